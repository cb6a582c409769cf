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

// Row groups per wave.  Every workgroup quantizes the vector, and a compute unit holds two: what counts is the row groups of the
// unit that has the most, so the workgroups of four waves are to fill one or two per unit of 256.  Of equal splits the one that
// measured faster: with 3-bit activations two workgroups quantizing on a unit are more in each other's way (10000 x 650 W3/A3
// 14.8 us with one group per wave, 14.4 with two; 10000 x 1024 W2/A2 12.2 and 12.3).  us per language-model step, one group up
// to 2048 and four beyond / here: 42000 x 1024 W2/A2 14.1 / 13.7, W3/A3 17.4 / 16.7, 20000 x 1024 W3/A3 15.4 / 15.1, 42000 x 2048
// W3/A3 27.4 / 25.1, 20000 x 2048 W2/A2 15.0 / 14.5; on either side of each line no size is slower.
int store_segments(long long m, int R, int k_a) {
  const long long groups = (m + R - 1) / R;
  if (groups <= 1024) return 1;                 // a workgroup per unit
  if (groups <= 2048) return k_a == 3 ? 2 : 1;  // two with one group per wave, one with two
  if (groups <= 3072) return 3;                 // one (with two: two workgroups, four groups in all)
  if (groups <= 4096) return 4;                 // one
  if (groups <= 6144) return 3;                 // two (with four: two as well)
  if (groups <= 8192) return 4;                 // two
  return groups <= 12288 ? 6 : 4;               // two; more than two rounds
}

template <int KW, int KA>
hipError_t launch_k(const BmvArgs& a, hipStream_t s) {
  const size_t lds = (size_t)KA * ((a.blk[0].n + 127) / 128) * 16;
  const dim3 grid((unsigned)((a.lse_slots + 3) / 4));
  auto launch = [&](auto segments) {
    hipLaunchKernelGGL((bmv_online_kernel<KW, KA, decltype(segments)::value>), grid, dim3(256), lds, s, a);
  };
  switch (store_segments(a.m, 64 >> a.lg, KA)) {
    case 1: launch(std::integral_constant<int, 1>{}); break;
    case 2:
      if constexpr (KA == 3) launch(std::integral_constant<int, 2>{});
      break;
    case 3: launch(std::integral_constant<int, 3>{}); break;
    case 4: launch(std::integral_constant<int, 4>{}); break;
    default: launch(std::integral_constant<int, 6>{}); break;
  }
  return hipGetLastError();
}

int lanes_log2(int n) {
  const int cpr = (n + 127) / 128;
  int lg = 0;
  while ((1 << lg) < cpr) ++lg;
  return lg;
}

long long store_waves(long long m, int n, int k_a) {
  const int R = 64 >> lanes_log2(n);
  const long long per = (long long)store_segments(m, R, k_a) * R;
  return (m + per - 1) / per;
}

}  // namespace

// 2- and 3-bit codes and vectors of at most 2048 entries (8 slots per lane of the quantizer); the product also leaves the
// pairs of a log-softmax, which must fit.
bool bmv_online_supported(const BmvArgs& a, int k_w, int k_a) {
  if (a.batch != 1 || a.groups != 1 || k_w < 2 || k_w > 3 || k_a < 2 || k_a > 3 || a.blk[0].n > 2048) return false;
  const long long waves = store_waves(a.m, a.blk[0].n, k_a);
  return a.lse_part && waves <= kLseMaxSlots && waves <= a.lse_cap;
}

hipError_t launch_bmv_online(BmvArgs a, int k_w, int k_a, hipStream_t s, int* lse_slots) {
  a.lg = lanes_log2(a.blk[0].n);
  a.lse_slots = (int)store_waves(a.m, a.blk[0].n, k_a);
  *lse_slots = a.lse_slots;
  a.streaming = (long long)k_w * a.m * ((a.blk[0].n + 127) / 128) * 16 > kBmvStreamingBytes;
  if (k_w == 2) return k_a == 2 ? launch_k<2, 2>(a, s) : launch_k<2, 3>(a, s);
  return k_a == 2 ? launch_k<3, 2>(a, s) : launch_k<3, 3>(a, s);
}

}  // namespace amq
