// What the two kernels of resident batched sequences share (amq_seqw.hip: one batch tile per workgroup, amq_seqw_tiles.hip: several):
// the exchange, the products of a row block with a tile, the cell.
#pragma once
#include "amq_launch.h"
#include "amq_quantize_body.h"

namespace amq {

namespace {

constexpr int kWBlocks = 4;             // row blocks per workgroup
constexpr int kWWaves = 2 * kWBlocks;   // waves per workgroup: one per row block and operand block
constexpr int kBlocksPad = kWBlocks + 1;
constexpr int kWTurn = 9;       // 16-byte units per row in the LDS piece that turns rows into operands (128 B + 16 B pad)

// Pairs that the codes and coefficients of one batch entry take in the exchange buffer: whole cache lines of 16.
__host__ __device__ constexpr int seqw_entry_pairs(int k_a, int wpr) { return (k_a * (wpr + 1) + 15) & ~15; }

__device__ __forceinline__ void put_pair(unsigned long long* p, unsigned value, unsigned tag) {
  __hip_atomic_store(p, ((unsigned long long)tag << 32) | value, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ unsigned long long get_pair(const unsigned long long* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// One failed poll: counts it, and decides whether to give up (too many, or somebody else has).
__device__ __forceinline__ bool poll_again(unsigned& spins, unsigned limit, unsigned* flag) {
  ++spins;
  if (spins > limit) {
    __hip_atomic_store(flag, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return false;
  }
  return (spins & 63u) != 0 || __hip_atomic_load(flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == 0u;
}

// Products of one wave's row block (16 rows) with one batch tile: packed weights in operand layout, activations as the
// expanded image in LDS (see amq_pair_body.h for both layouts).  The accumulators start at minus the contribution of
// the positions past the end of the vectors, so they end as the dot products of the codes.
template <int KW, int KA, int NC>
__device__ __forceinline__ void contract(const uint4 (&araw)[NC][KW][2], const uint4* image, int l16, int l4, int n,
                                         v4f (&acc)[KW][KA]) {
  constexpr int kAllSteps = NC * kSteps;
  const int halves = (n + 511) >> 9;
  const float start = (float)(n - halves * 512);
#pragma unroll
  for (int i = 0; i < KW; ++i)
#pragma unroll
    for (int j = 0; j < KA; ++j) acc[i][j] = v4f{start, start, start, start};
  const uint4* const my = image + 16 * l4;
  auto b_operand = [&](int j, int t) { return my[(j * kAllSteps + t) * 64 + (l16 ^ ((l4 << 1) | (((t >> 2) & 1) << 3)))]; };
  uint4 aop[KW], anx[KW], bop[KA], bnx[KA];
#pragma unroll
  for (int j = 0; j < KA; ++j) bop[j] = b_operand(j, 0);
#pragma unroll
  for (int i = 0; i < KW; ++i) aop[i] = expand4_signed(word_of(araw[0][i], 0));
#pragma unroll
  for (int half = 0; half < 2 * NC; ++half) {
    if (half > 0 && half >= halves) break;  // (uniform)
#pragma unroll
    for (int t = 4 * half; t < 4 * half + 4; ++t) {
      if (t + 1 < kAllSteps) {
#pragma unroll
        for (int j = 0; j < KA; ++j) bnx[j] = b_operand(j, t + 1);
#pragma unroll
        for (int i = 0; i < KW; ++i) anx[i] = expand4_signed(word_of(araw[(t + 1) / kSteps][i], (t + 1) % kSteps));
      }
#pragma unroll
      for (int i = 0; i < KW; ++i)
#pragma unroll
        for (int j = 0; j < KA; ++j) acc[i][j] = mfma_fp4(aop[i], bop[j], acc[i][j]);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = 0; i < KW; ++i) aop[i] = anx[i];
#pragma unroll
      for (int j = 0; j < KA; ++j) bop[j] = bnx[j];
    }
  }
  settle_accumulators<16>();
#pragma unroll
  for (int i = 0; i < KW; ++i)
#pragma unroll
    for (int j = 0; j < KA; ++j) asm volatile("" : "+v"(acc[i][j]));
}

// Keeps the compiler from expanding these words once, ahead of the loop over the steps, and holding the result.
template <int NC, int KW>
__device__ __forceinline__ void keep_packed(uint4 (&w)[NC][KW][2]) {
#pragma unroll
  for (int ch = 0; ch < NC; ++ch)
#pragma unroll
    for (int i = 0; i < KW; ++i)
#pragma unroll
      for (int v = 0; v < 2; ++v) asm volatile("" : "+v"(w[ch][i][v].x), "+v"(w[ch][i][v].y), "+v"(w[ch][i][v].z), "+v"(w[ch][i][v].w));
}

// y_r = sum_i alpha_ri sum_j beta_j d_ij of this lane's four rows (the gates of its hidden unit) and batch entry.
template <int KW, int KA>
__device__ __forceinline__ void weigh(const v4f (&acc)[KW][KA], const float (&al)[4][KW], const float (&bt)[KA],
                                      float (&y)[4]) {
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    float s = 0.0f;
#pragma unroll
    for (int i = 0; i < KW; ++i) {
      float inner = 0.0f;
#pragma unroll
      for (int j = 0; j < KA; ++j) inner = fmaf(bt[j], acc[i][j][r], inner);
      s = fmaf(al[r][i], inner, s);
    }
    y[r] = s;
  }
}

// Eq. 6 on one unit's sums; bias0 / bias1 as the per-step kernels take them.  h: h_{t-1} in, h_t out.
template <int EPI>
__device__ __forceinline__ void cell(const float (&yx)[4], const float (&yh)[4], const float (&b0)[4], const float (&b1)[4],
                                     float& h, float& c) {
  if constexpr (EPI == kEpiLstm) {
    const float gi = sigmoidf_dev(yx[0] + yh[0] + b0[0]);
    const float gf = sigmoidf_dev(yx[1] + yh[1] + b0[1]);
    const float go = sigmoidf_dev(yx[2] + yh[2] + b0[2]);
    const float gg = tanhf_dev(yx[3] + yh[3] + b0[3]);
    c = fmaf(gf, c, gi * gg);
    h = go * tanhf_dev(c);
  } else {
    const float rg = sigmoidf_dev(yx[0] + yh[0] + b0[0] + b1[0]);
    const float z = sigmoidf_dev(yx[1] + yh[1] + b0[1] + b1[1]);
    const float nn = tanhf_dev(fmaf(rg, yh[2] + b1[2], yx[2] + b0[2]));
    h = fmaf(z, h - nn, nn);
  }
}

// Whether the weights stay in registers as matrix operands (32 registers per plane and stretch) or packed: as far as the
// registers go.
template <int KW, int KA, int NC>
constexpr bool kExpandedOnce = NC == 1 && KW * KA < 9;

template <int KW, int KA, int NC>
constexpr size_t seqw_lds() {
  return sizeof(uint4) * (2 * KA * NC * kSteps * 64);
}

}  // namespace

}  // namespace amq
