// The quantizer kernel and its launch rules, shared by the quantizer proper (RECON false: packed codes and coefficients)
// and the training-side form that leaves the reconstruction instead (RECON).
#pragma once
#include "amq_launch.h"
#include "amq_quantize_body.h"

namespace amq {

namespace {

// The second launch bound is the waves per SIMD that the registers shall allow.
template <int K>
constexpr int kQuantWaves = K == 4 ? 3 : 4;

template <int K, int NJ, int NW, bool ONLINE, bool RECON>
__global__ __launch_bounds__(64 * NW, NW < 16 ? kQuantWaves<K> : 4)
void quantize_kernel(QuantArgs a) {
  __shared__ double sh[2 * kExchange<NW>];
  asm volatile("" ::AMQ_ARG(a.seg[0].X), AMQ_ARG(a.seg[0].ld), AMQ_ARG(a.seg[0].n), AMQ_ARG(a.seg[0].count),
               AMQ_ARG(a.seg[0].planes), AMQ_ARG(a.seg[0].coef), AMQ_ARG(a.seg[1].X), AMQ_ARG(a.seg[1].ld),
               AMQ_ARG(a.seg[1].n), AMQ_ARG(a.seg[1].count), AMQ_ARG(a.seg[1].planes), AMQ_ARG(a.seg[1].coef),
               AMQ_ARG(a.T), AMQ_ARG(a.gather.count));
  quantize_block<K, NJ, NW, ONLINE, RECON>(a, blockIdx.x, sh);
}

template <int K, int NJ, int NW, bool ONLINE, bool RECON>
void launch_one(QuantArgs a, int total, hipStream_t s) {
  AMQ_PHASE_ATTACH(a);
  hipLaunchKernelGGL((quantize_kernel<K, NJ, NW, ONLINE, RECON>), dim3(total), dim3(64 * NW), 0, s, a);
}

// Waves per vector.  Many vectors (throughput): as few waves as hold the vector with at most 16 slots per lane --
// what a wave does once per vector (reductions, solves, code tables) is then paid by few waves, and 16 slots keep
// the registers at about 100; then the smallest register form that holds the share.  Few vectors (the on-line case,
// latency): at most 4 slots per lane over at least 4 waves, and the form of the algorithm made for that.
template <int K, bool RECON>
hipError_t launch_k(const QuantArgs& a, int max_n, hipStream_t s) {
  const int nvec = a.seg[0].count + a.seg[1].count;
  const int total = nvec + a.gather.count;  // one workgroup per vector, one per gathered row
  if (total == 0) return hipSuccess;
  const int nslots = nvec ? 2 * ((max_n + 127) / 128) : 1;
  if (nslots > 256) return hipErrorInvalidValue;
  if (nvec < 1024 && nslots <= 64) {
    if (nslots <= 2) launch_one<K, 2, 1, true, RECON>(a, total, s);
    else if (nslots <= 16) launch_one<K, 4, 4, true, RECON>(a, total, s);
    else if (nslots <= 32) launch_one<K, 4, 8, true, RECON>(a, total, s);
    else launch_one<K, 4, 16, true, RECON>(a, total, s);
    return hipGetLastError();
  }
  int nw = 1;
  while (nw < 16 && (nslots + nw - 1) / nw > 16) nw *= 2;
  const int nj = (nslots + nw - 1) / nw;
  switch (nw * 32 + (nj + 1) / 2 * 2) {
    case 32 + 2: launch_one<K, 2, 1, false, RECON>(a, total, s); break;
    case 32 + 4: launch_one<K, 4, 1, false, RECON>(a, total, s); break;
    case 32 + 6: launch_one<K, 6, 1, false, RECON>(a, total, s); break;
    case 32 + 8: launch_one<K, 8, 1, false, RECON>(a, total, s); break;
    case 32 + 10: launch_one<K, 10, 1, false, RECON>(a, total, s); break;
    case 32 + 12: launch_one<K, 12, 1, false, RECON>(a, total, s); break;
    case 32 + 14: launch_one<K, 14, 1, false, RECON>(a, total, s); break;
    case 32 + 16: launch_one<K, 16, 1, false, RECON>(a, total, s); break;
    case 64 + 10: launch_one<K, 10, 2, false, RECON>(a, total, s); break;
    case 64 + 12: launch_one<K, 12, 2, false, RECON>(a, total, s); break;
    case 64 + 14: launch_one<K, 14, 2, false, RECON>(a, total, s); break;
    case 64 + 16: launch_one<K, 16, 2, false, RECON>(a, total, s); break;
    case 128 + 10: launch_one<K, 10, 4, false, RECON>(a, total, s); break;
    case 128 + 12: launch_one<K, 12, 4, false, RECON>(a, total, s); break;
    case 128 + 14: launch_one<K, 14, 4, false, RECON>(a, total, s); break;
    case 128 + 16: launch_one<K, 16, 4, false, RECON>(a, total, s); break;
    default:
      if (nw == 8) launch_one<K, 16, 8, false, RECON>(a, total, s);
      else launch_one<K, 16, 16, false, RECON>(a, total, s);
  }
  return hipGetLastError();
}

template <bool RECON>
hipError_t launch_bits(const QuantArgs& a, int k, hipStream_t s) {
  const int max_n = a.seg[1].count > 0 && a.seg[1].n > a.seg[0].n ? a.seg[1].n : a.seg[0].n;
  switch (k) {
    case 1: return launch_k<1, RECON>(a, max_n, s);
    case 2: return launch_k<2, RECON>(a, max_n, s);
    case 3: return launch_k<3, RECON>(a, max_n, s);
    case 4: return launch_k<4, RECON>(a, max_n, s);
  }
  return hipErrorInvalidValue;
}

}  // namespace

}  // namespace amq
