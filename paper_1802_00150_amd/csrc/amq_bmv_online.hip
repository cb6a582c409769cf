// The plain small-batch product for one batch entry whose operand vector it quantizes itself (amq_bmv_body.h): the output layer
// of a language model.
#include "amq_bmv_body.h"

namespace amq {

namespace {

// (The second launch bound keeps the results of the quantizer's matrix instructions in ordinary registers.)
template <int KW, int KA, int NSEG>
__global__ __launch_bounds__(256, 2) void bmv_online_kernel(BmvArgs a) {
  extern __shared__ uint4 xs[];
  __shared__ double sh[2 * kExchange<4>];
  __shared__ float bts[4];
  bmv_body<KW, KA, NSEG, 1, kEpiStore, true, true>(a, xs, sh, bts);
}

// Rows (row groups of four where there are many) per wave of a plain product.  Every workgroup quantizes the vector, so
// the grid is kept near two workgroups per compute unit rather than near the most parallelism.
int store_segments(long long m, int R) { return (m + R - 1) / R > 2048 ? 4 : 1; }

template <int KW, int KA>
hipError_t launch_k(const BmvArgs& a, hipStream_t s) {
  const size_t lds = (size_t)KA * ((a.blk[0].n + 127) / 128) * 16;
  const dim3 grid((unsigned)((a.lse_slots + 3) / 4));
  if (store_segments(a.m, 64 >> a.lg) == 4)
    hipLaunchKernelGGL((bmv_online_kernel<KW, KA, 4>), grid, dim3(256), lds, s, a);
  else
    hipLaunchKernelGGL((bmv_online_kernel<KW, KA, 1>), grid, dim3(256), lds, s, a);
  return hipGetLastError();
}

int lanes_log2(int n) {
  const int cpr = (n + 127) / 128;
  int lg = 0;
  while ((1 << lg) < cpr) ++lg;
  return lg;
}

long long store_waves(long long m, int n) {
  const int R = 64 >> lanes_log2(n);
  const long long per = (long long)store_segments(m, R) * R;
  return (m + per - 1) / per;
}

}  // namespace

// 2- and 3-bit codes and vectors of at most 2048 entries (8 slots per lane of the quantizer); the product also leaves the
// pairs of a log-softmax, which must fit.
bool bmv_online_supported(const BmvArgs& a, int k_w, int k_a) {
  if (a.batch != 1 || a.groups != 1 || k_w < 2 || k_w > 3 || k_a < 2 || k_a > 3 || a.blk[0].n > 2048) return false;
  const long long waves = store_waves(a.m, a.blk[0].n);
  return a.lse_part && waves <= kLseMaxSlots && waves <= a.lse_cap;
}

hipError_t launch_bmv_online(BmvArgs a, int k_w, int k_a, hipStream_t s, int* lse_slots) {
  a.lg = lanes_log2(a.blk[0].n);
  a.lse_slots = (int)store_waves(a.m, a.blk[0].n);
  *lse_slots = a.lse_slots;
  a.streaming = (long long)k_w * a.m * ((a.blk[0].n + 127) / 128) * 16 > kBmvStreamingBytes;
  if (k_w == 2) return k_a == 2 ? launch_k<2, 2>(a, s) : launch_k<2, 3>(a, s);
  return k_a == 2 ? launch_k<3, 2>(a, s) : launch_k<3, 3>(a, s);
}

}  // namespace amq
