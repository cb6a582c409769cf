// The small-batch product kernel for one batch entry whose operand vectors it quantizes itself (amq_bmv_body.h).
#include "amq_bmv_body.h"

namespace amq {

namespace {

// (The second launch bound keeps the results of the quantizer's matrix instructions in ordinary registers.)
template <int KW, int KA, int NSEG, int NBLK, int EPI>
__global__ __launch_bounds__(256, 2) void bmv_online_kernel(BmvArgs a) {
  extern __shared__ uint4 xs[];
  __shared__ double sh[2 * kExchange<4>];
  __shared__ float bts[NBLK][4];
  bmv_body<KW, KA, NSEG, NBLK, EPI, EPI == kEpiStore, true>(a, xs, sh, bts);
}

// Rows (row groups of four where there are many) per wave of a plain product.  Every workgroup quantizes the vector, so
// the grid is kept near two workgroups per compute unit rather than near the most parallelism.
int store_segments(long long m, int R) { return (m + R - 1) / R > 2048 ? 4 : 1; }

template <int KW, int KA>
hipError_t launch_k(BmvArgs a, int epi, hipStream_t s) {
  const int R = 64 >> a.lg;
  size_t lds = 0;
  for (int k = 0; k < (epi == kEpiStore ? 1 : 2); ++k) lds += (size_t)KA * ((a.blk[k].n + 127) / 128) * 16;
  if (epi == kEpiLstm) {
    const unsigned grid = (unsigned)(((a.H + R - 1) / R + 3) / 4);
    hipLaunchKernelGGL((bmv_online_kernel<KW, KA, 4, 2, kEpiLstm>), dim3(grid), dim3(256), lds, s, a);
  } else {
    const unsigned grid = (unsigned)((a.lse_slots + 3) / 4);
    if (store_segments(a.m, R) == 4)
      hipLaunchKernelGGL((bmv_online_kernel<KW, KA, 4, 1, kEpiStore>), dim3(grid), dim3(256), lds, s, a);
    else
      hipLaunchKernelGGL((bmv_online_kernel<KW, KA, 1, 1, kEpiStore>), dim3(grid), dim3(256), lds, s, a);
  }
  return hipGetLastError();
}

int lanes_log2(int n0, int n1) {
  const int cpr = ((n0 > n1 ? n0 : n1) + 127) / 128;
  int lg = 0;
  while ((1 << lg) < cpr) ++lg;
  return lg;
}

long long store_waves(long long m, int n) {
  const int R = 64 >> lanes_log2(n, 0);
  const long long per = (long long)store_segments(m, R) * R;
  return (m + per - 1) / per;
}

}  // namespace

// 2- and 3-bit codes and vectors of at most 2048 entries (8 slots per lane of the quantizer); a plain product also
// leaves the pairs of a log-softmax, which must fit.
bool bmv_online_supported(const BmvArgs& a, int k_w, int k_a, int epi) {
  if (a.batch != 1 || a.groups != 1 || k_w < 2 || k_w > 3 || k_a < 2 || k_a > 3 || a.blk[0].n > 2048) return false;
  if (epi == kEpiLstm) return a.blk[1].n <= 2048;
  const long long waves = store_waves(a.m, a.blk[0].n);
  return epi == kEpiStore && a.lse_part && waves <= kLseMaxSlots && waves <= a.lse_cap;
}

hipError_t launch_bmv_online(BmvArgs a, int k_w, int k_a, int epi, hipStream_t s, int* lse_slots) {
  a.lg = lanes_log2(a.blk[0].n, epi == kEpiStore ? 0 : a.blk[1].n);
  if (epi == kEpiStore) {
    a.lse_slots = (int)store_waves(a.m, a.blk[0].n);
    if (lse_slots) *lse_slots = a.lse_slots;
  }
  long long plane_bytes = (long long)k_w * a.m * ((a.blk[0].n + 127) / 128) * 16;
  if (epi != kEpiStore) plane_bytes += (long long)k_w * a.m * ((a.blk[1].n + 127) / 128) * 16;
  a.streaming = plane_bytes > kBmvStreamingBytes;
  if (k_w == 2) return k_a == 2 ? launch_k<2, 2>(a, epi, s) : launch_k<2, 3>(a, epi, s);
  return k_a == 2 ? launch_k<3, 2>(a, epi, s) : launch_k<3, 3>(a, epi, s);
}

}  // namespace amq
