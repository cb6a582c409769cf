// The quantizer kernel and its launch rules, shared by the quantizer proper (RECON false: packed codes and coefficients)
// and the training-side form that leaves the reconstruction instead (RECON).
#pragma once
#include "amq_launch.h"
#include "amq_quantize_body.h"

namespace amq {

namespace {

// The second launch bound is the waves per SIMD that the registers shall allow.
constexpr int quant_waves(int k, int nj, bool online) {
  if (k == 4 && nj <= 4 && !online) return 5;  // (98 registers otherwise: 42000 vectors of 200 entries 96.7 against 92.3 us)
  return k == 4 && nj > 16 ? 2 : k == 4 || nj > 24 ? 3 : 4;
}

template <int K, int NJ, int NW, bool ONLINE, bool RECON>
__global__ __launch_bounds__(64 * NW, NW < 16 ? quant_waves(K, NJ, ONLINE) : 4)
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

// Wide forms: 20 to 32 slots per lane, vectors of 1025 .. 2048 entries on one wave and up to 4096 on two.  What a wave does once
// per vector (reductions, solves, code tables) takes as long as 20 slots' work at k = 2, 30 to 50 beyond, so half the waves
// per vector win over the registers that the slots take (three or two waves per SIMD) -- given enough vectors to fill the
// chip.  Measured, us, 16384 vectors, 16 slots / here: k = 2 of 1100 / 1500 / 2048 / 3000 / 4096 entries 29.7 / 31.3 / 34.0 /
// 56.6 / 67.2 -> 22.6 / 25.2 / 27.7 / 51.6 / 65.6, k = 3 59.4 / 62.3 / 65.1 / 116 / 126 -> 40.5 / 45.3 / 55.0 / 96.8 / 121,
// k = 4 131 / 139 / 148 / 267 / 290 -> 83.6 / 93.2 / 129 / 208 / 284; reconstruction k = 3 54.5 / 62.2 / 66.4 / 120 / 132 ->
// 41.5 / 47.3 / 60.2 / 104 / 115.  At k = 3 on one wave 32 slots spill (84 bytes per lane, reconstruction 64) and are ahead all the
// same (1540 / 2300 / 4096 / 16384 vectors of 2048 entries 5 / 4 / 11 / 15 %, reconstruction -1 / -3 / 3 / 9 %); the others of
// these forms spill nothing worth the name.  Where they are ahead:
constexpr bool wide_ahead(int k, bool recon, int nw, int nj, int vectors) {
  if (recon && k == 2 && nj > (nw == 1 ? 24 : 20)) return false;  // (bound by its stores: 16384 x 1700 36.1 against 37.1)
  if (nw == 2 && nj > 24)  // (4096 entries, k = 2: 8192 vectors 33.6 against 33.8, 4096 19.2 against 20.0)
    return vectors >= (recon ? 4096 : k == 3 ? 8192 : 12288);
  // (2500 vectors of 2900 entries are 5 % behind at k = 2, of 2816 and 3072, whose slots are all full, 5 to 13 % ahead)
  // Rounds of two waves per SIMD against two waves per vector in rounds of three: 1536 vectors are one of the latter (18.7 against
  // 17.0 at 2048 entries), 2048 one of the former, and some more leave its second nearly empty (2200 29.6 against 27.4)
  if (k == 4 && nw == 1 && nj > (recon ? 28 : 24)) return (vectors > 1536 && vectors <= 2048) || vectors >= 2700;
  return vectors >= 1536;  // (1100 vectors of 1700 entries, k = 3: 9.6 against 10.4; 2000 11.2 against 10.5)
}

template <int K, bool RECON>
bool launch_wide(const QuantArgs& a, int total, int nw, int nj, hipStream_t s) {
  constexpr bool kAll = !(RECON && K == 2);
  switch (nw * 64 + (nj + 3) / 4 * 4) {
    case 64 + 20: launch_one<K, 20, 1, false, RECON>(a, total, s); return true;
    case 64 + 24: launch_one<K, 24, 1, false, RECON>(a, total, s); return true;
    case 128 + 20: launch_one<K, 20, 2, false, RECON>(a, total, s); return true;
  }
  if constexpr (kAll) {
    switch (nw * 64 + (nj + 3) / 4 * 4) {
      case 64 + 28: launch_one<K, 28, 1, false, RECON>(a, total, s); return true;
      case 64 + 32: launch_one<K, 32, 1, false, RECON>(a, total, s); return true;
      case 128 + 24: launch_one<K, 24, 2, false, RECON>(a, total, s); return true;
      case 128 + 28: launch_one<K, 28, 2, false, RECON>(a, total, s); return true;
      case 128 + 32: launch_one<K, 32, 2, false, RECON>(a, total, s); return true;
    }
  }
  return false;
}

// Waves per vector.  Many vectors (throughput): the wide forms above where they are ahead, otherwise as few waves as hold
// the vector with at most 16 slots per lane, which keep the registers at about 100; then the smallest register form that
// holds the share.  Few vectors (the on-line case, latency): at most 4 slots per lane over 4 or 8 waves, and the form of
// the algorithm made for that.  It buys its short chain with every wave of a vector solving the same small systems, so it
// ends where those waves no longer fit the chip side by side: about two vectors per compute unit, three at k = 3.  Beyond
// 2048 entries it would take 16 waves per vector, whose exchange costs more than the slots that they save, already at one
// vector (but for one range of lengths at k = 3, below).  Both give the same codes and coefficients, to the bit.  Measured, us, latency / throughput form, 512 and 700
// vectors: 300 entries k = 2 3.48 / 3.06 (reconstruction) and 3.97 / 3.11, k = 4 7.97 / 6.06 and 10.3 / 6.1; 650 entries k = 2
// 3.64 / 3.67 and 4.17 / 3.78, k = 3 at 700 5.18 / 5.38 and at 1000 6.03 / 5.42, k = 4 8.67 / 9.26 and 10.9 / 9.3; 2048 entries
// k = 2 4.71 / 4.82 and 5.76 / 4.88.  4096 entries, 1 and 512 vectors: k = 2 4.37 / 3.92 and 8.05 / 4.98, k = 3 6.17 / 5.94 and
// 11.6 / 7.6, k = 4 13.2 / 10.1, reconstruction k = 3 6.46 / 5.95 and 12.8 / 8.4.  A wave on its own whose 16 slots are not all
// full is slow enough for the line of k = 3 at k = 1 and in reconstructions too (680 vectors of 1000 entries k = 1 2.82 / 2.97, of
// 1024 2.80 / 2.56, reconstruction k = 3 6.2 / 6.45).
constexpr int online_vectors(int k, bool recon, int n) {
  const bool partly = n > 896 && n < 1024 && (k == 1 || k == 3);
  return (k == 3 && !recon) || partly ? 768 : 600;
}

template <int K, bool RECON>
hipError_t launch_k(const QuantArgs& a, int max_n, hipStream_t s) {
  const int nvec = a.seg[0].count + a.seg[1].count;
  const int total = nvec + a.gather.count;  // one workgroup per vector, one per gathered row
  if (total == 0) return hipSuccess;
  const int nslots = nvec ? 2 * ((max_n + 127) / 128) : 1;
  if (nslots > 256) return hipErrorInvalidValue;
  if (nslots <= 32 && nvec < online_vectors(K, RECON, max_n)) {
    if (nslots <= 2) launch_one<K, 2, 1, true, RECON>(a, total, s);
    else if (nslots <= 16) launch_one<K, 4, 4, true, RECON>(a, total, s);
    else launch_one<K, 4, 8, true, RECON>(a, total, s);
    return hipGetLastError();
  }
  if constexpr (K == 3 && !RECON) {
    // As long as every vector has a compute unit, and 16 slots of four waves are not all full: 16 and 250 vectors of 3840 entries
    // 6.77 / 7.33 and 7.12 / 7.5, 300 11.7 / 7.9; 16 of 4096 6.66 / 6.43
    if (nslots > 56 && nslots <= 64 && max_n < 4096 && nvec <= 256) {
      launch_one<K, 4, 16, true, RECON>(a, total, s);
      return hipGetLastError();
    }
  }
  if constexpr (K >= 2) {
    const int nw = nslots <= 32 ? 1 : 2, nj = (nslots + nw - 1) / nw;
    if (nslots > 16 && nslots <= 64 && wide_ahead(K, RECON, nw, nj, nvec) && launch_wide<K, RECON>(a, total, nw, nj, s))
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
