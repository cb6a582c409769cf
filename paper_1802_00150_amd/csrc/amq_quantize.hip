// Alternating multi-bit quantization (Alg. 2) on gfx950: one workgroup of NW wavefronts per vector, the vector
// held in registers, every stage of the algorithm in this one kernel (amq_quantize_core.h), and the two staged
// hooks (Eq. 5 alone, Alg. 1 alone).
#include "amq_quantize_kernels.h"

namespace amq {

namespace {

// Staged hooks on one vector per workgroup: Eq. 5 with the codes given (a.mode == kQuantLsOnly), or Alg. 1 with
// the coefficients given.
template <int K, int NJ, int NW>
__global__ __launch_bounds__(64 * NW) void quantize_stage_kernel(QuantArgs a) {
  __shared__ double sh[2][16 * kMaxRed];
  int phase = 0;
  const int lane = lane_id(), wv = __builtin_amdgcn_readfirstlane(wave_id());
  const long long vec = blockIdx.x;
  const int n = a.seg[0].n, count = a.seg[0].count;
  const int wpr = 4 * ((n + 127) >> 7);
  const int nslots = wpr >> 1;
  const int nj = (nslots + NW - 1) / NW;
  const int base = wv * nj;
  float* coef = a.seg[0].coef + vec * K;
  const bool holds = lane < nj && base + lane < nslots;
  float w[NJ];
  load_slots<NJ>(a.seg[0].X + vec * a.seg[0].ld, n, base, nj, w);
  auto masks_of = [&](int i) {
    return reinterpret_cast<unsigned long long*>(a.seg[0].planes + ((long long)i * count + vec) * wpr) + base + lane;
  };
  float alpha[K];
#pragma unroll
  for (int i = 0; i < K; ++i) alpha[i] = coef[i];
  unsigned long long mym[K];
  if (a.mode == kQuantLsOnly) {
    constexpr int NP = K * (K - 1) / 2;
    double red[K + NP];
#pragma unroll
    for (int i = 0; i < K; ++i) {
      mym[i] = holds ? *masks_of(i) : 0ull;
      const int lo = (int)(mym[i] & 0xffffffffull), hi = (int)(mym[i] >> 32);
      double q = 0.0;
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        if (j < nj) {
          const unsigned long long mk = ((unsigned long long)(unsigned)__builtin_amdgcn_readlane(hi, j) << 32) |
                                        (unsigned)__builtin_amdgcn_readlane(lo, j);
          q += ((mk >> lane) & 1ull) ? (double)w[j] : -(double)w[j];
        }
      }
      red[i] = q;
    }
    int t = K;
#pragma unroll
    for (int i = 0; i < K; ++i)
#pragma unroll
      for (int j = i + 1; j < K; ++j) red[t++] = (double)__popcll(mym[i] ^ mym[j]);
    block_totals<NW, K + NP>(red, sh, phase);
    double qq[K];
#pragma unroll
    for (int i = 0; i < K; ++i) qq[i] = red[i];
    ls_solve_f64<K>(n, red + K, qq, alpha);
    if (threadIdx.x == 0) {
#pragma unroll
      for (int i = 0; i < K; ++i) coef[i] = alpha[i];
    }
  } else {
    constexpr int H = 1 << (K - 1);
#pragma unroll
    for (int i = 0; i < K; ++i) mym[i] = 0ull;
    CodeTable<K> ct;
    if constexpr (K > 1) {
      code_table_any_order<K>(alpha, ct);
    } else {
      // the upper code is +alpha or, for a negative coefficient, -alpha
      ct.bm[0] = __ballot(alpha[0] < 0.0f) != 0ull ? 0u : 1u;
    }
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      if (j < nj) {
        const float xc = w[j] + 0.0f;
        const unsigned b = __float_as_uint(xc);
        const int u = (int)min(b, b + 0x7fffffffu);
        int m = 0;
        if constexpr (K > 1) {
#pragma unroll
          for (int t = 0; t < H - 1; ++t) m += (u >= ct.thr[t]) ? 1 : 0;
        }
        const unsigned long long in = lanes_inside(n, base + j);
#pragma unroll
        for (int i = 0; i < K; ++i)
          keep_in_lane(mym[i], __ballot((((ct.bm[i] >> m) & 1u) != 0u) != (xc < 0.0f)) & in, j);
      }
    }
#pragma unroll
    for (int i = 0; i < K; ++i)
      if (holds) *masks_of(i) = mym[i];
  }
}

template <int K>
hipError_t launch_stage(const QuantArgs& a, int nslots, hipStream_t s) {
  const dim3 grid((unsigned)a.seg[0].count);
  if (nslots <= 16) hipLaunchKernelGGL((quantize_stage_kernel<K, 4, 4>), grid, dim3(256), 0, s, a);
  else if (nslots <= 64) hipLaunchKernelGGL((quantize_stage_kernel<K, 16, 4>), grid, dim3(256), 0, s, a);
  else hipLaunchKernelGGL((quantize_stage_kernel<K, 16, 16>), grid, dim3(1024), 0, s, a);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_quantize(const QuantArgs& a, int k, hipStream_t s) {
  if (a.mode == kQuantFull) return launch_bits<false>(a, k, s);
  const int nslots = 2 * ((a.seg[0].n + 127) / 128);
  if (a.seg[0].count == 0) return hipSuccess;
  if (nslots > 256) return hipErrorInvalidValue;
  switch (k) {
    case 1: return launch_stage<1>(a, nslots, s);
    case 2: return launch_stage<2>(a, nslots, s);
    case 3: return launch_stage<3>(a, nslots, s);
    case 4: return launch_stage<4>(a, nslots, s);
  }
  return hipErrorInvalidValue;
}

}  // namespace amq
