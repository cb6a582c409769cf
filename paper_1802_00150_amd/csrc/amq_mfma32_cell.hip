// Recurrent steps of large batches on the 32 x 32 form of the fp4 matrix instruction (see amq_mfma32_body.h for what that form
// buys): a wave forms, for 8 hidden units x all gates and 32 batch entries, the x-side and the h-side sums one after the other
// and applies the LSTM or GRU cell (Eq. 6) to them in registers.
//
// The 32 rows of a wave are ordered unit by unit, four rows each (the GRU's fourth stays unused), so that the C layout (lane =
// column l % 32, register r = row 8 (r / 4) + 4 (l / 32) + r % 4) leaves all gates of a unit in four adjacent registers: lane
// half kb holds units 2 q + kb of its column.  State and results pass between the halves with two shuffles so that each lane
// loads and stores 16 adjacent bytes, in one request where the tensors of the state are aligned to them.  The activation operands of the workgroup's 32 entries are staged in LDS as in the plain
// kernel, both blocks at once where they fit, otherwise one after the other; weight pieces go from memory to registers two
// ahead of their use.
//
// Bound: matrix cores for large steps (2048 units at batch 256, W2/A2: 69 GFLOP), otherwise the latency of one pass.
#include "amq_mfma32_body.h"

namespace amq {

namespace {

using mfma32::kMaxLds;
using mfma32::kTileN;
using mfma32::kXcds;
using mfma32::v16f;

constexpr int kUnits = 8;  // hidden units of a wave

// Pieces per k-block; the contraction takes them in pairs, so their number is made even.
__host__ __device__ constexpr int pieces_per_half(int n) { return (((n + 127) >> 7) + 1) / 2; }
__host__ __device__ constexpr int even_half_pieces(int n) { return (pieces_per_half(n) + 1) / 2 * 2; }
__host__ __device__ constexpr size_t cell_image_bytes(int ka, int n) { return (size_t)ka * even_half_pieces(n) * 4 * 1024; }
// Private to a wave: [block][plane][row] coefficients, [bias][row]; with more than four plane products also what the
// accumulators leave no registers for: the x-side sums and the previous state, [5][64 lanes] of 16 bytes
__host__ __device__ constexpr bool cell_parks(int kw, int ka) { return kw * ka > 4; }
__host__ __device__ constexpr int cell_wave_floats(int kw, int ka) { return kTileN * (2 * kw + 2) + (cell_parks(kw, ka) ? 5 * 64 * 4 : 0); }

template <int KW, int KA, int EPI, int WV>
__global__ __launch_bounds__(64 * WV, 8 / WV) void mfma32_cell_kernel(BmvArgs a, int rowblocks, int tiles, int per_xcd,
                                                                       int together, int aligned) {
  constexpr int NG = EPI == kEpiGru ? 3 : 4;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  asm volatile("" ::AMQ_ARG(a.blk[0].Wp), AMQ_ARG(a.blk[0].alpha), AMQ_ARG(a.blk[0].Xp), AMQ_ARG(a.blk[0].beta),
               AMQ_ARG(a.blk[0].n), AMQ_ARG(a.blk[1].Wp), AMQ_ARG(a.blk[1].alpha), AMQ_ARG(a.blk[1].Xp), AMQ_ARG(a.blk[1].beta),
               AMQ_ARG(a.blk[1].n), AMQ_ARG(a.H), AMQ_ARG(a.batch), AMQ_ARG(a.bias0), AMQ_ARG(a.bias1), AMQ_ARG(rowblocks),
               AMQ_ARG(tiles), AMQ_ARG(per_xcd), AMQ_ARG(together), AMQ_ARG(aligned));
  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, kb = lane >> 5;
  const int task = (blockIdx.x % kXcds) * per_xcd + blockIdx.x / kXcds;
  const int rb0 = task / tiles * WV;
  if (rb0 >= rowblocks) return;  // (the whole workgroup)
  const int rb = rb0 + wv, col0 = task % tiles * kTileN;
  const int H = (int)a.H, batch = a.batch;
  const int nn[2] = {a.blk[0].n, a.blk[1].n};
  const int np[2] = {even_half_pieces(nn[0]), even_half_pieces(nn[1])};

  // ---- weight pieces of this wave's rows (rows, gates and pieces past the end are clamped: their results are never used, or
  // meet zeros of the staged operand); index counts through the pieces of both blocks
  const int my_unit = min(rb * kUnits + (l32 >> 2), H - 1), my_gate = min(l32 & 3, NG - 1);
  const int my_row = my_gate * H + my_unit;
  // Pieces asked for together: adjacent ones share a cache line, which the first-level cache does not hold until a later
  // request comes (31.4 -> 27.9 us at 2048 units, batch 256, W2/A2).  Nine plane products leave no registers for more than one.
  constexpr int D = KW * KA < 9 ? 2 : 1;
  typedef uint4 Pieces[D][KW];
  Pieces cur, nxt;
  const int all = (np[0] + np[1]) / D;
  auto request = [&](int index, Pieces& to) {
    const int p0 = min(index, all - 1) * D, k = p0 < np[0] ? 0 : 1, p = k ? p0 - np[0] : p0;
    const int wq = (nn[k] + 127) >> 7;
    const uint4* row = reinterpret_cast<const uint4*>(k ? a.blk[1].Wp : a.blk[0].Wp) + (unsigned)(my_row * wq);
    const size_t plane = (size_t)NG * H * wq;
#pragma unroll
    for (int d = 0; d < D; ++d) {
      const int g = kb * np[k] + p + d;
#pragma unroll
      for (int i = 0; i < KW; ++i) to[d][i] = row[i * plane + (g < wq ? g : 0)];
    }
  };

  // ---- activation operands of block k into `image`: item -> (plane, piece, k-block, column); kBatch items per thread at a time
  constexpr int kBatch = 4;
  auto ask = [&](int k, int e0, uint4 (&xw)[kBatch]) {
    const uint4* Xp4 = reinterpret_cast<const uint4*>(k ? a.blk[1].Xp : a.blk[0].Xp);
    const int wq = (nn[k] + 127) >> 7, h = np[k], items = KA * h * 64;
#pragma unroll
    for (int v = 0; v < kBatch; ++v) {
      const unsigned e = min(e0 + tid + v * 64 * WV, items - 1);
      const unsigned q = e >> 6, p = q % (unsigned)h, j = q / (unsigned)h;
      const int c = col0 + (int)(e & 31), g = (int)(((e >> 5) & 1) * h + p);
      xw[v] = Xp4[((size_t)j * batch + (c < batch ? c : batch - 1)) * wq + (g < wq ? g : 0)];
    }
  };
  auto put = [&](int k, int e0, uint4* image, const uint4 (&xw)[kBatch]) {
    const int n = nn[k], h = np[k], items = KA * h * 64;
#pragma unroll
    for (int v = 0; v < kBatch; ++v) {
      const unsigned e = e0 + tid + v * 64 * WV;
      if (e < (unsigned)items) {
        const unsigned q = e >> 6, p = q % (unsigned)h, j = q / (unsigned)h;
        const int g = (int)(((e >> 5) & 1) * h + p);
        const uint32_t ws[4] = {xw[v].x, xw[v].y, xw[v].z, xw[v].w};
        uint4* d = image + (j * 4 * h + 4 * p) * 64 + (e & 63);
        if (128 * (g + 1) <= n) {
#pragma unroll
          for (int s = 0; s < 4; ++s) d[s * 64] = expand4_signed(ws[s]);
        } else {
#pragma unroll
          for (int s = 0; s < 4; ++s) {
            const int left = n - 32 * (4 * g + s);
            const uint32_t valid = left >= 32 ? 0xffffffffu : left <= 0 ? 0u : ((1u << left) - 1u);
            d[s * 64] = expand4_signed_valid(ws[s], valid);
          }
        }
      }
    }
  };
  auto stage_rest = [&](int k, int e0, uint4* image) {
    for (; e0 < KA * np[k] * 64; e0 += kBatch * 64 * WV) {  // (uniform)
      uint4 xw[kBatch];
      ask(k, e0, xw);
      put(k, e0, image, xw);
    }
  };
  uint4 x0[kBatch], x1[kBatch];
  ask(0, 0, x0);
  if (together) ask(1, 0, x1);
  request(0, cur);
  request(1, nxt);
  uint4* const image0 = reinterpret_cast<uint4*>(smem);
  uint4* const image1 = reinterpret_cast<uint4*>(smem + (together ? cell_image_bytes(KA, nn[0]) : 0));
  const size_t images = together ? cell_image_bytes(KA, nn[0]) + cell_image_bytes(KA, nn[1])
                                 : max(cell_image_bytes(KA, nn[0]), cell_image_bytes(KA, nn[1]));
  float* const mine = reinterpret_cast<float*>(smem + images) + wv * cell_wave_floats(KW, KA);
  constexpr bool kParks = cell_parks(KW, KA);
  float4* const parked = reinterpret_cast<float4*>(mine + kTileN * (2 * KW + 2)) + lane;

  // ---- coefficients and biases of this wave's rows, row = 4 * unit + gate; state of its columns
  constexpr int kCoef = (kTileN * KW + 63) / 64;
  float coef[2][kCoef], bias;
#pragma unroll
  for (int k = 0; k < 2; ++k)
#pragma unroll
    for (int v = 0; v < kCoef; ++v) {
      const int e = min(v * 64 + lane, kTileN * KW - 1), g = e / (kUnits * KW), r = e % (kUnits * KW);
      const int u = min(rb * kUnits + r / KW, H - 1);
      coef[k][v] = (k ? a.blk[1].alpha : a.blk[0].alpha)[(size_t)(min(g, NG - 1) * H + u) * KW + r % KW];
    }
  {
    const float* from = kb == 0 ? a.bias0 : EPI == kEpiGru ? a.bias1 : nullptr;
    const int u = min(rb * kUnits + (l32 & 7), H - 1);
    bias = from ? from[min(l32 >> 3, NG - 1) * H + u] : 0.0f;
  }
  const int col = col0 + l32, bc = min(col, batch - 1);
  float beta[2][KA];
#pragma unroll
  for (int k = 0; k < 2; ++k)
#pragma unroll
    for (int j = 0; j < KA; ++j) beta[k][j] = (k ? a.blk[1].beta : a.blk[0].beta)[bc * KA + j];
  const int u4 = rb * kUnits + 4 * kb;  // the four adjacent units this lane loads and stores
  const bool vec = aligned && (H & 3) == 0 && u4 + 4 <= H;
  const size_t at = (size_t)bc * H + u4;
  float prev[4];
  {
    const float* from = EPI == kEpiGru ? a.h_prev : a.c_prev;
    if (vec) {
      const float4 t = *reinterpret_cast<const float4*>(from + at);
      prev[0] = t.x; prev[1] = t.y; prev[2] = t.z; prev[3] = t.w;
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) prev[e] = from[(size_t)bc * H + min(u4 + e, H - 1)];
    }
  }

  put(0, 0, image0, x0);
  stage_rest(0, kBatch * 64 * WV, image0);
  if (together) {
    put(1, 0, image1, x1);
    stage_rest(1, kBatch * 64 * WV, image1);
  }
  lds_barrier();

  // ---- products: y[k][4 q + g] = gate g of unit 2 q + kb
  float y[2][16];
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    const uint4* const img = (k ? image1 : image0) + lane;
    const int steps = 4 * np[k], first = k ? np[0] : 0;
    if (k == 1 && !together) {
      lds_barrier();
      stage_rest(1, 0, image1);
      lds_barrier();
    }
    uint4 bop[KA], bnx[KA], aop[KW], anx[KW];
    auto fetch = [&](int step, uint4 (&b)[KA]) {
#pragma unroll
      for (int j = 0; j < KA; ++j) b[j] = img[(j * steps + step) * 64];
    };
    auto expand = [&](const uint4 (&from)[KW], int word, uint4 (&to)[KW]) {
#pragma unroll
      for (int i = 0; i < KW; ++i)
        to[i] = expand4_signed(word == 0 ? from[i].x : word == 1 ? from[i].y : word == 2 ? from[i].z : from[i].w);
    };
    v16f acc[KW][KA];
#pragma unroll
    for (int i = 0; i < KW; ++i)
#pragma unroll
      for (int j = 0; j < KA; ++j) acc[i][j] = v16f{};
    fetch(0, bop);
    expand(cur[0], 0, aop);
    auto step = [&](int index, auto s_c, const uint4 (&cur)[KW], const uint4 (&nxt)[KW]) {
      constexpr int s = decltype(s_c)::value;
      fetch(index + 1 == steps ? 0 : index + 1, bnx);
      if constexpr (s < 3) expand(cur, s + 1, anx); else expand(nxt, 0, anx);
#pragma unroll
      for (int i = 0; i < KW; ++i)
#pragma unroll
        for (int j = 0; j < KA; ++j) acc[i][j] = mfma32::mfma32_fp4(aop[i], bop[j], acc[i][j]);
      constexpr int kValu = (7 * KW + KW * KA - 1) / (KW * KA);
      __builtin_amdgcn_sched_group_barrier(0x100, KA, 0);
#pragma unroll
      for (int g = 0; g < KW * KA; ++g) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x002, kValu, 0);
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int j = 0; j < KA; ++j) bop[j] = bnx[j];
#pragma unroll
      for (int i = 0; i < KW; ++i) aop[i] = anx[i];
    };
    auto piece = [&](int p, const uint4 (&cur)[KW], const uint4 (&nxt)[KW]) {
      step(4 * p, std::integral_constant<int, 0>{}, cur, nxt);
      step(4 * p + 1, std::integral_constant<int, 1>{}, cur, nxt);
      step(4 * p + 2, std::integral_constant<int, 2>{}, cur, nxt);
      step(4 * p + 3, std::integral_constant<int, 3>{}, cur, nxt);
    };
    for (int p = 0; p < np[k]; p += D) {
#pragma unroll
      for (int d = 0; d < D; ++d) piece(p + d, cur[d], d + 1 < D ? cur[d + 1 < D ? d + 1 : d] : nxt[0]);
#pragma unroll
      for (int d = 0; d < D; ++d)
#pragma unroll
        for (int i = 0; i < KW; ++i) cur[d][i] = nxt[d][i];
      request((first + p) / D + 2, nxt);
    }
    // (pinned in uniform control flow: the compiler takes a matrix instruction for lane-local)
    settle_accumulators<32>();
#pragma unroll
    for (int i = 0; i < KW; ++i)
#pragma unroll
      for (int j = 0; j < KA; ++j) asm volatile("" : "+v"(acc[i][j]));
    if (k == 0) {  // (a wave's own piece of LDS, which serves its accesses in order)
#pragma unroll
      for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int v = 0; v < kCoef; ++v) {
          const int e = v * 64 + lane, g = e / (kUnits * KW), r = e % (kUnits * KW);
          if (kTileN * KW % 64 == 0 || e < kTileN * KW) mine[(b * KW + r % KW) * kTileN + 4 * (r / KW) + g] = coef[b][v];
        }
      mine[(2 * KW + kb) * kTileN + 4 * (l32 & 7) + (l32 >> 3)] = bias;
      if constexpr (kParks) parked[4 * 64] = make_float4(prev[0], prev[1], prev[2], prev[3]);
      __builtin_amdgcn_wave_barrier();
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      float4 al[KW];
#pragma unroll
      for (int i = 0; i < KW; ++i) al[i] = *reinterpret_cast<const float4*>(&mine[(k * KW + i) * kTileN + 8 * q + 4 * kb]);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        float s = 0.0f;
#pragma unroll
        for (int i = 0; i < KW; ++i) {
          float inner = 0.0f;
#pragma unroll
          for (int j = 0; j < KA; ++j) inner = fmaf(beta[k][j], acc[i][j][4 * q + r], inner);
          s = fmaf(r == 0 ? al[i].x : r == 1 ? al[i].y : r == 2 ? al[i].z : al[i].w, inner, s);
        }
        y[k][4 * q + r] = s;
      }
      if (kParks && k == 0) parked[q * 64] = make_float4(y[0][4 * q], y[0][4 * q + 1], y[0][4 * q + 2], y[0][4 * q + 3]);
    }
  }
  if constexpr (kParks) {
    const float4 t = parked[4 * 64];
    prev[0] = t.x; prev[1] = t.y; prev[2] = t.z; prev[3] = t.w;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const float4 v = parked[q * 64];
      y[0][4 * q] = v.x; y[0][4 * q + 1] = v.y; y[0][4 * q + 2] = v.z; y[0][4 * q + 3] = v.w;
    }
  }

  // ---- the cell.  From the four adjacent units a lane holds to every second one, and back: the halves of the wave swap two
  auto swap = [&](float x) { return __shfl_xor(x, 32, kWave); };
  float st[4];
  {
    const float r0 = swap(kb ? prev[0] : prev[1]), r1 = swap(kb ? prev[2] : prev[3]);
    st[0] = kb ? r0 : prev[0];
    st[1] = kb ? r1 : prev[2];
    st[2] = kb ? prev[1] : r0;
    st[3] = kb ? prev[3] : r1;
  }
  float hv[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const float4 b0 = *reinterpret_cast<const float4*>(&mine[2 * KW * kTileN + 8 * q + 4 * kb]);
    const float* yx = &y[0][4 * q];
    const float* yh = &y[1][4 * q];
    if constexpr (EPI == kEpiLstm) {
      const float gi = sigmoidf_dev(yx[0] + yh[0] + b0.x);
      const float gf = sigmoidf_dev(yx[1] + yh[1] + b0.y);
      const float go = sigmoidf_dev(yx[2] + yh[2] + b0.z);
      const float gg = tanhf_dev(yx[3] + yh[3] + b0.w);
      st[q] = fmaf(gf, st[q], gi * gg);
      hv[q] = go * tanhf_dev(st[q]);
    } else {
      const float4 b1 = *reinterpret_cast<const float4*>(&mine[(2 * KW + 1) * kTileN + 8 * q + 4 * kb]);
      const float rg = sigmoidf_dev(yx[0] + yh[0] + b0.x + b1.x);
      const float z = sigmoidf_dev(yx[1] + yh[1] + b0.y + b1.y);
      const float nw = tanhf_dev(fmaf(rg, yh[2] + b1.z, yx[2] + b0.z));
      hv[q] = fmaf(z, st[q] - nw, nw);
    }
  }
  const bool mine_to_store = rb < rowblocks && col < batch;
  auto store = [&](float* to, const float (&v)[4]) {
    const float r0 = swap(kb ? v[0] : v[2]), r1 = swap(kb ? v[1] : v[3]);
    const float4 o = kb ? make_float4(r0, v[2], r1, v[3]) : make_float4(v[0], r0, v[1], r1);
    if (!mine_to_store) return;
    if (vec) {
      *reinterpret_cast<float4*>(to + at) = o;
    } else {
      const float e[4] = {o.x, o.y, o.z, o.w};
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (u4 + i < H) to[at + i] = e[i];
    }
  };
  store(a.h_out, hv);
  if constexpr (EPI == kEpiLstm) store(a.c_out, st);
  if (a.hs_out) store(a.hs_out, hv);
}

template <int KW, int KA, int EPI, int WV>
hipError_t run(const BmvArgs& a, hipStream_t s) {
  const int rowblocks = (int)((a.H + kUnits - 1) / kUnits), tiles = (a.batch + kTileN - 1) / kTileN;
  const int groups = (rowblocks + WV - 1) / WV * tiles, per_xcd = (groups + kXcds - 1) / kXcds;
  const size_t i0 = cell_image_bytes(KA, a.blk[0].n), i1 = cell_image_bytes(KA, a.blk[1].n), co = (size_t)WV * cell_wave_floats(KW, KA) * sizeof(float);
  const bool together = i0 + i1 + co <= (size_t)kMaxLds;
  const uintptr_t state = reinterpret_cast<uintptr_t>(EPI == kEpiGru ? a.h_prev : a.c_prev) | reinterpret_cast<uintptr_t>(a.h_out) |
                          reinterpret_cast<uintptr_t>(EPI == kEpiGru ? nullptr : a.c_out) | reinterpret_cast<uintptr_t>(a.hs_out);
  static std::atomic<unsigned long long> configured{0};
  const hipError_t e = ensure_dynamic_lds(reinterpret_cast<const void*>(&mfma32_cell_kernel<KW, KA, EPI, WV>), kMaxLds, configured);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((mfma32_cell_kernel<KW, KA, EPI, WV>), dim3((unsigned)(per_xcd * kXcds)), dim3(64 * WV),
                     (together ? i0 + i1 : i0 > i1 ? i0 : i1) + co, s, a, rowblocks, tiles, per_xcd, together ? 1 : 0,
                     (state & 15) == 0 ? 1 : 0);
  return hipGetLastError();
}

// Workgroups have four waves as long as every one of them gets a compute unit of its own, otherwise eight.
constexpr int kCompute = 256;
struct Groups {
  bool few;
  long long rounds;  // of workgroups on the chip
};
Groups groups_of(long long H, long long batch) {
  const long long rowblocks = (H + kUnits - 1) / kUnits, tiles = (batch + kTileN - 1) / kTileN;
  if ((rowblocks + 3) / 4 * tiles <= kCompute) return Groups{true, 1};
  return Groups{false, ((rowblocks + 7) / 8 * tiles + kCompute - 1) / kCompute};
}

template <int KW, int KA>
hipError_t run_k(const BmvArgs& a, int epi, hipStream_t s) {
  const bool few = groups_of(a.H, a.batch).few;
  if (epi == kEpiGru) return few ? run<KW, KA, kEpiGru, 4>(a, s) : run<KW, KA, kEpiGru, 8>(a, s);
  return few ? run<KW, KA, kEpiLstm, 4>(a, s) : run<KW, KA, kEpiLstm, 8>(a, s);
}

}  // namespace

// Steps of 2- and 3-bit codes and vectors of at most 2048 entries.  Both this kernel and those on 16 x 16 tiles take as long as
// the compute unit with the most to do: here a round of workgroups, of four waves or of eight, there `other` workgroups of 16
// units and 16 entries.  Measured, us per step with its quantizer, 16 x 16 / here, LSTM:
//   - a vector above 1024 entries.  16 x 16 takes 4.2 (W2/A2) to 6.1 (W3/A3) per workgroup and 5 to 6 more, whatever the lengths up
//     to 2048; here a round takes as long as the vectors are.  2048 units, batch 64 / 128 / 160 / 256 / 272 / 400 W2/A2 13.3 / 18.0,
//     20.9 / 19.2, 26.3 / 25.4, 38.2 / 28.7, 42.3 / 44.3, 59.1 / 47.4, W3/A2 15.8 / 21.7, 25.5 / 23.7, 32.1 / 33.8, 47.3 / 42.0,
//     53.8 / 64.0, 74.7 / 69.1, W3/A3 18.9 / 29.5, 30.2 / 32.2, 37.9 / 40.3, 55.9 / 48.1, 63.1 / 76.2, 89.1 / 81.4; 300 and 2000 entries
//     batch 128 W3/A3 32.8 / 24.5, 1100 units batch 256 W2/A2 24.1 / 19.5;
//   - up to 1024 entries the 16 x 16 kernel takes two batch tiles per wave at four plane products and stays ahead (1024 units
//     batch 256 11.9 / 13.5).  Six: 1024 units batch 256 W2/A3 21.4 / 16.6, 512 28.9 / 23.0, 650 units batch 256 15.6 / 17.4, 1024
//     38.2 / 39.3; nine: 1024 units batch 256 20.9 / 19.4, 512 33.3 / 27.2, 650 units batch 200 20.8 / 20.0, 900 units batch 140
//     14.6 / 20.0, 1024 units batch 128 12.2 / 18.0.  A second round wants to be filled more than at longer vectors: batch 600
//     900 units W2/A3 31.2 / 39.3, 1024 units W3/A2 33.2 / 38.0, W3/A3 40.9 / 45.2.
bool mfma32_cell_supported(const BmvArgs& a, int k_w, int k_a, int epi) {
  if (epi != kEpiLstm && epi != kEpiGru) return false;
  if (a.groups > 1 || k_w < 2 || k_w > 3 || k_a < 2 || k_a > 3) return false;
  const int nmax = a.blk[0].n > a.blk[1].n ? a.blk[0].n : a.blk[1].n;
  if (nmax > 2048) return false;  // (one block's image fits LDS)
  if (a.m * ((nmax + 127) / 128) * k_w >= (1LL << 28) || (long long)a.batch * a.H >= (1LL << 29)) return false;
  const int products = k_w * k_a, np = even_half_pieces(a.blk[0].n) + even_half_pieces(a.blk[1].n);
  const Groups g = groups_of(a.H, a.batch);
  const long long work = (a.H + 15) / 16 * ((a.batch + 15) / 16), other = (work + kCompute - 1) / kCompute;
  const long long past = other - 8 * (g.rounds - 1);  // (a full round of eight waves is eight of those)
  if (nmax > 1024) {
    const bool light = np <= 10 || (np <= 12 && k_a == 2);
    if (g.few) return other >= (light ? 3 : np <= 12 || k_a == 2 ? 4 : 5);
    if (light || g.rounds > 2) return true;
    if (g.rounds == 1) return other >= (products == 9 && np > 12 ? 6 : 5);
    return past >= (products == 4 ? 1 : np <= 12 ? 2 : 3);
  }
  const bool padded = even_half_pieces(a.blk[0].n) != pieces_per_half(a.blk[0].n) ||
                      even_half_pieces(a.blk[1].n) != pieces_per_half(a.blk[1].n);
  if (products == 4) return false;
  if (g.few) return products == 6 ? (a.H + kUnits - 1) / kUnits * ((a.batch + kTileN - 1) / kTileN) > 768 : work >= 528;
  if (products == 6 && padded && g.rounds > 1) return false;
  if (g.rounds != 2) return true;
  const bool gru = epi == kEpiGru;  // (the 16 x 16 kernel leaves a quarter of a GRU's tiles empty, too)
  return past >= (products == 6 ? (gru ? 4 : 5) : gru && !padded ? 1 : 3);
}

hipError_t launch_mfma32_cell(const BmvArgs& a, int k_w, int k_a, int epi, hipStream_t s) {
  if (k_w == 2) return k_a == 2 ? run_k<2, 2>(a, epi, s) : run_k<2, 3>(a, epi, s);
  return k_a == 2 ? run_k<3, 2>(a, epi, s) : run_k<3, 3>(a, epi, s);
}

}  // namespace amq
