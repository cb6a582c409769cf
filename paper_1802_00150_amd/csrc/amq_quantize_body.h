// Body of the quantizer kernel for one workgroup (Alg. 2 on one vector held in registers, or the copy
// of one row of a quantized table), shared by the stand-alone quantizer kernel and the front kernel of
// the split recurrent step.
#pragma once
#include "amq_launch.h"
#include "amq_quantize_core.h"

namespace amq {

// One workgroup copies row ids[g] of a quantized table (all K planes and coefficients) to
// position g of the output operand; an index outside the table gives the zero vector.
template <int K>
__device__ __forceinline__ void gather_row(const GatherSeg& t, int g, int nthreads) {
  const int wpr = 4 * ((t.n + 127) >> 7);
  const long long id = t.ids[g];
  const bool ok = id >= 0 && id < t.vocab;
  const long long row = ok ? id : 0;
#pragma unroll
  for (int i = 0; i < K; ++i) {
    const uint32_t* src = t.table + ((long long)i * t.vocab + row) * wpr;
    uint32_t* dst = t.planes + ((long long)i * t.count + g) * wpr;
    for (int w = threadIdx.x; w < wpr; w += nthreads) dst[w] = ok ? src[w] : 0u;
  }
  if (threadIdx.x < K) t.coef[(long long)g * K + threadIdx.x] = ok ? t.table_coef[row * K + threadIdx.x] : 0.0f;
}

// Entries (base + j) * 64 + lane of a vector of n entries, 0.0 beyond its end or beyond slot nj.  Straight-line
// loads (the index is clamped), so that they all go out before the first is waited for.
template <int NJ>
__device__ __forceinline__ void load_slots(const float* x, int n, int base, int nj, float (&w)[NJ]) {
  const int lane = lane_id();
  if (nj == NJ && (base + NJ) * 64 <= n) {
#pragma unroll
    for (int j = 0; j < NJ; ++j) w[j] = x[(base + j) * 64 + lane];
  } else {
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      const int e = (base + j) * 64 + lane;
      w[j] = x[e < n ? e : n - 1];
    }
#pragma unroll
    for (int j = 0; j < NJ; ++j) w[j] = (j < nj && (base + j) * 64 + lane < n) ? w[j] : 0.0f;
  }
}

// f(number of slots to hold in registers, a constant).  The latency-bound form computes every slot it holds, so there the
// number follows the share of the wave closely: 2, 3, 4, 6 or 8, as far as NJ goes.
template <int NJ, bool ONLINE, typename F>
__device__ __forceinline__ void with_slots(int nj, F f) {
  auto call = [&](auto slots) { f(slots); };
  if constexpr (ONLINE && NJ == 4) {
    if (nj <= 2) call(std::integral_constant<int, 2>{});
    else if (nj == 3) call(std::integral_constant<int, 3>{});
    else call(std::integral_constant<int, 4>{});
  } else if constexpr (ONLINE && NJ == 8) {
    if (nj <= 2) call(std::integral_constant<int, 2>{});
    else if (nj <= 4) call(std::integral_constant<int, 4>{});
    else if (nj <= 6) call(std::integral_constant<int, 6>{});
    else call(std::integral_constant<int, 8>{});
  } else {
    call(std::integral_constant<int, NJ>{});
  }
}

// vec: index of this workgroup's vector over both segments (then over the gathered rows).  sh:
// 2 * kExchange<NW> doubles of LDS.  Every wave of the workgroup (NW of them) must call this.
template <int K, int NJ, int NW, bool ONLINE, bool RECON = false>
__device__ __forceinline__ void quantize_block(const QuantArgs& a, int vec, double* sh) {
  int phase = 0;
  const int lane = lane_id(), wv = __builtin_amdgcn_readfirstlane(wave_id());
  AMQ_PHASE(AMQ_PHASE_OF(a), 0);
  if (vec >= a.seg[0].count + a.seg[1].count) {
    // workgroups past the vectors to quantize copy table rows by index
    gather_row<K>(a.gather, vec - a.seg[0].count - a.seg[1].count, 64 * NW);
    return;
  }
  const int which = (vec >= a.seg[0].count) ? 1 : 0;
  if (which) vec -= a.seg[0].count;
  const float* X = which ? a.seg[1].X : a.seg[0].X;
  const long long ld = which ? a.seg[1].ld : a.seg[0].ld;
  const int n = which ? a.seg[1].n : a.seg[0].n;
  const int count = which ? a.seg[1].count : a.seg[0].count;
  uint32_t* planes = which ? a.seg[1].planes : a.seg[0].planes;
  float* coef = which ? a.seg[1].coef : a.seg[0].coef;

  const int wpr = 4 * ((n + 127) >> 7);
  const int nslots = wpr >> 1;            // 64-entry slots per row, padding included
  const int nj = (nslots + NW - 1) / NW;  // slots per wave; host guarantees nj <= NJ
  const int base = wv * nj;
  const float* x = X + (long long)vec * ld;

  float alpha[K];
  unsigned long long mym[K];
  AMQ_PHASE(AMQ_PHASE_OF(a), 1);
  with_slots<NJ, ONLINE>(nj, [&](auto slots) {
    float w[slots()];
    load_slots<slots()>(x, n, base, nj, w);
    if constexpr (RECON && !ONLINE) {
      float v[slots()];
      quantize_core<K, slots(), NW, ONLINE, true>(w, n, base, nj, a.T, alpha, mym, sh, phase, AMQ_PHASE_OF(a), v);
      float* out = a.recon + (long long)vec * a.recon_ld + base * 64 + lane;
      const int left = min(n - base * 64, nj * 64) - lane;
#pragma unroll
      for (int j = 0; j < slots(); ++j)
        if (j * 64 < left) out[j * 64] = v[j];
    } else {
      quantize_core<K, slots(), NW, ONLINE>(w, n, base, nj, a.T, alpha, mym, sh, phase, AMQ_PHASE_OF(a));
    }
  });

  if constexpr (RECON) {
    if (!ONLINE) return;
    // left to right over the planes, as launch_dequantize forms it; the mask of a slot sits in the slot's lane
    float* out = a.recon + (long long)vec * a.recon_ld + base * 64 + lane;
    const int left = min(n - base * 64, nj * 64) - lane;
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      float v = 0.0f;
#pragma unroll
      for (int i = 0; i < K; ++i) {
        const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(mym[i] & 0xffffffffull), j);
        const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(mym[i] >> 32), j);
        const float term = lane_bit(((unsigned long long)hi << 32) | lo) ? alpha[i] : -alpha[i];
        v = (i == 0) ? term : v + term;
      }
      if (j * 64 < left) out[j * 64] = v;
    }
    return;
  }
#pragma unroll
  for (int i = 0; i < K; ++i)
    if (lane < nj && base + lane < nslots)
      reinterpret_cast<unsigned long long*>(planes + ((long long)i * count + vec) * wpr)[base + lane] = mym[i];
  if (threadIdx.x == 0) {
#pragma unroll
    for (int i = 0; i < K; ++i) coef[(long long)vec * K + i] = alpha[i];
  }
  AMQ_PHASE(AMQ_PHASE_OF(a), 31);
}

}  // namespace amq
