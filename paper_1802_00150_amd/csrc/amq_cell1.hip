// One LSTM or GRU step of one batch entry in one launch (Eq. 6 at batch 1): every workgroup quantizes the operand vectors itself
// while its weights are under way, multiplies the rows of its hidden units (amq_unit_lanes.h) and applies the cell.
//
// Against a quantizer launch of its own that is about a microsecond of arithmetic in every workgroup instead of a launch (2.5 us
// on the host, 1.6 to 3.4 us between dependent kernels).  Bound: latency -- the vectors' cold loads, Alg. 2, the cell.  So
// nothing that a later part needs is asked for late: vectors first (loads return in order), then weights, coefficients,
// biases and the previous state, then the row of the table whose index arrived meanwhile.  Two vectors are quantized side by
// side, each by half of the waves: with at most 8 slots of 64 entries per lane that is 4 waves up to 1024 entries, 8 beyond.
//
// Measured, us per call, before (a wave held all gates of its units, two vectors one after the other, state asked for at the
// end) -> here: LSTM step 300 units W2/A2 / W3/A3 7.6 / 12.1 -> 4.7 / 5.7, 1024 units 7.8 / 12.5 -> 4.4 / 5.7; language-model
// step of 1024 units and 42000 words W2/A2 17.3 -> 14.5; GRU step (two launches before) with its output layer 14.6 -> 11.8.
#include "amq_launch.h"
#include "amq_quantize_body.h"
#include "amq_unit_lanes.h"

namespace amq {

namespace {

enum { kLookUp = 0, kBoth = 1 };  // x is a row of a quantized table; x and h are quantized here

// WG: waves of a workgroup.
template <int KW, int KA, int EPI, int OPS, int WG>
__global__ __launch_bounds__(64 * WG, 8 / WG) void cell1_kernel(BmvArgs a) {
  constexpr int NG = EPI == kEpiGru ? 3 : 4;
  constexpr int kChunks = 16;
  constexpr int NW = OPS == kBoth ? WG / 2 : WG;  // waves per vector
  constexpr int NJ = OPS == kBoth ? 8 : 4;        // slots per lane
  __shared__ double sh[WG / NW * 2 * kExchange<NW>];
  __shared__ __attribute__((aligned(16))) uint4 codes[2][KA][kChunks];
  __shared__ float coef[2][KA];
  asm volatile("" ::AMQ_ARG(a.blk[0].Wp), AMQ_ARG(a.blk[0].alpha), AMQ_ARG(a.blk[0].Xp), AMQ_ARG(a.blk[0].beta),
               AMQ_ARG(a.blk[0].n), AMQ_ARG(a.blk[1].Wp), AMQ_ARG(a.blk[1].alpha), AMQ_ARG(a.blk[1].n), AMQ_ARG(a.H),
               AMQ_ARG(a.bias0), AMQ_ARG(a.bias1), AMQ_ARG(a.c_prev), AMQ_ARG(a.h_prev), AMQ_ARG(a.raw[0]), AMQ_ARG(a.raw[1]),
               AMQ_ARG(a.row_of), AMQ_ARG(a.lg));
  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int I = a.blk[0].n, H = (int)a.H;
  const int cprI = (I + 127) >> 7, cprH = (H + 127) >> 7;

  // ---- the vectors
  const int mine = OPS == kBoth ? wv / NW : 1;  // which vector this wave works on
  const int n = mine ? H : I, nslots = (n + 63) / 64, nj = (nslots + NW - 1) / NW, base = (wv & (NW - 1)) * nj;
  float raw[NJ];
  load_slots<NJ>(a.raw[mine], n, base, nj, raw);
  long long id = 0;
  if constexpr (OPS == kLookUp) id = a.row_of[0];

  // ---- weights, biases, previous state
  const UnitLanes l(a.lg, lane);
  const int unit = ((int)blockIdx.x * WG + wv) * l.per + l.uo;
  UnitWeights<KW, 1> q;
  load_unit_weights<KW, 1, NG>(q, l, unit, a.blk[0].Wp, a.blk[0].alpha, I, a.blk[1].Wp, a.blk[1].alpha, H);
  const bool cell = l.c == 0 && l.gate == 0 && unit < H;
  const int uc = unit < H ? unit : 0;
  float b0[NG], b1[NG];
#pragma unroll
  for (int r = 0; r < NG; ++r) {
    b0[r] = a.bias0 ? a.bias0[r * H + uc] : 0.0f;
    b1[r] = (EPI == kEpiGru && a.bias1) ? a.bias1[r * H + uc] : 0.0f;
  }
  float h = EPI == kEpiGru ? a.h_prev[uc] : 0.0f, c = EPI == kEpiLstm ? a.c_prev[uc] : 0.0f;

  // ---- the row of the table: one 16-byte piece and one coefficient per thread
  uint4 piece = make_uint4(0, 0, 0, 0);
  float piece_coef = 0.0f;
  if constexpr (OPS == kLookUp) {
    const bool there = id >= 0 && id < a.rows_of;
    const long long r = there ? id : 0;
    const int t = tid < KA * cprI ? tid : 0, j = t / cprI;
    const uint4 got = reinterpret_cast<const uint4*>(a.blk[0].Xp)[(j * a.rows_of + r) * cprI + (t - j * cprI)];
    const float gc = a.blk[0].beta[r * KA + (tid < KA ? tid : 0)];
    if (there) {
      piece = got;
      piece_coef = gc;
    }
  }

  // ---- Alg. 2
  {
    int phase = 0;
    float alpha[KA];
    unsigned long long mym[KA];
    with_slots<NJ, true>(nj, [&](auto slots) {
      float x[slots()];
#pragma unroll
      for (int j = 0; j < slots(); ++j) x[j] = raw[j];
      quantize_core<KA, slots(), NW, true>(x, n, base, nj, a.T, alpha, mym, sh + (OPS == kBoth ? mine * 2 * kExchange<NW> : 0),
                                           phase);
    });
    const int cpr = mine ? cprH : cprI;
    if (lane < (base + nj >= nslots ? 2 * cpr - base : nj)) {
#pragma unroll
      for (int j = 0; j < KA; ++j) reinterpret_cast<unsigned long long*>(codes[mine][j])[base + lane] = mym[j];
    }
    if ((wv & (NW - 1)) == 0 && lane == 0) {
#pragma unroll
      for (int j = 0; j < KA; ++j) coef[mine][j] = alpha[j];
    }
  }
  if constexpr (OPS == kLookUp) {
    if (tid < KA * cprI) codes[0][tid / cprI][tid % cprI] = piece;
    if (tid < KA) coef[0][tid] = piece_coef;
  }
  lds_barrier();

  // ---- products and cell
  float p[2][1];
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    const int cpr = k ? cprH : cprI;
    uint4 x[KA];
    float bt[KA];
#pragma unroll
    for (int j = 0; j < KA; ++j) {
      const uint4 t = codes[k][j][l.c < cpr ? l.c : 0];
      x[j] = l.c < cpr ? t : make_uint4(0, 0, 0, 0);
      bt[j] = coef[k][j];
    }
    p[k][0] = unit_dot(q, k, 0, x, bt);
  }
  unit_cell<EPI, 1, true, NG>(l, p[0], p[1], b0, b1, h, c);
  if (cell) {
    a.h_out[unit] = h;
    if constexpr (EPI == kEpiLstm) a.c_out[unit] = c;
    if (a.hs_out) a.hs_out[unit] = h;
  }
}

template <int KW, int KA, int EPI, int OPS, int WG>
hipError_t run(const BmvArgs& a, hipStream_t s) {
  const int units = WG * (16 >> a.lg);
  hipLaunchKernelGGL((cell1_kernel<KW, KA, EPI, OPS, WG>), dim3((unsigned)((a.H + units - 1) / units)), dim3(64 * WG), 0, s, a);
  return hipGetLastError();
}

template <int KW, int KA>
hipError_t run_k(const BmvArgs& a, int epi, hipStream_t s) {
  const bool longer = a.lg == 4;
  if (epi == kEpiGru) return longer ? run<KW, KA, kEpiGru, kBoth, 8>(a, s) : run<KW, KA, kEpiGru, kBoth, 4>(a, s);
  if (!a.raw[0]) return longer ? run<KW, KA, kEpiLstm, kLookUp, 8>(a, s) : run<KW, KA, kEpiLstm, kLookUp, 4>(a, s);
  return longer ? run<KW, KA, kEpiLstm, kBoth, 8>(a, s) : run<KW, KA, kEpiLstm, kBoth, 4>(a, s);
}

}  // namespace

// 2- and 3-bit codes and vectors of at most 2048 entries.
bool cell1_supported(const BmvArgs& a, int k_w, int k_a, int epi) {
  return a.batch == 1 && a.groups == 1 && k_w >= 2 && k_w <= 3 && k_a >= 2 && k_a <= 3 && a.blk[0].n <= 2048 &&
         a.blk[1].n <= 2048 && a.raw[1] && (a.raw[0] || (epi == kEpiLstm && a.row_of));
}

hipError_t launch_cell1(BmvArgs a, int k_w, int k_a, int epi, hipStream_t s) {
  const int n = a.blk[0].n > a.blk[1].n ? a.blk[0].n : a.blk[1].n;
  a.lg = 0;
  while ((128 << a.lg) < n) ++a.lg;
  if (k_w == 2) return k_a == 2 ? run_k<2, 2>(a, epi, s) : run_k<2, 3>(a, epi, s);
  return k_a == 2 ? run_k<3, 2>(a, epi, s) : run_k<3, 3>(a, epi, s);
}

}  // namespace amq
