// Large batched binary matrix products on the fp4 matrix cores of gfx950 (Fig. 3 right):
// Y = (sum_i alpha_i B_i)(sum_j beta_j x_j) for many rows and 32 or more columns (mfma4w_kernel),
// and the recurrent steps for batches of 128 and more (mfma4wc_kernel, further down).
//
// Same matrix instruction as the kernel in amq_mfma4.hip (codes as E2M1 nibbles,
// v_mfma_f32_16x16x128_f8f6f4), different work split.  There a wave owns one 16 x 16 output tile
// per pass, and per pass it spends about 350 vector instructions (1400 cycles) on addressing, expanding
// the weight words, popcounts and the coefficient epilogue against k_w k_a 8 matrix instructions (900
// cycles at W2/A3): the vector unit, not the matrix core, bounds it.  Here a wave owns 16 rows x NBT batch
// tiles, so that everything on the weight side (loads, expansion, row coefficients) is paid once per NBT
// tiles and only the per-output epilogue grows with the tile count.  A workgroup of 8 waves stages NBT * 16
// batch entries (all planes) in LDS once and its waves walk over row blocks.  mfma4w_kernel works on
// {-1, +1} codes (the staged activations hold 0.0 beyond the end of a vector), so its accumulators are the
// dot products of the codes and no popcount enters, and so does mfma4wc_kernel.
#include <type_traits>

#include "amq_device.h"
#include "amq_launch.h"
#include "amq_pair_body.h"

namespace amq {

namespace {

constexpr int kWaves = 8;
constexpr int kTurn = 9;  // 16-byte units per row in the piece of LDS that turns weight rows into operands (128 B + 16 B pad)

// Contraction of one operand block of a row block with NBT staged batch tiles: units u = (k-step t,
// tile bt); the LDS reads (and, when the step changes, the weight expansion) of unit u + 1 are
// issued under the matrix instructions of unit u.  `tile` points at this lane's 16 bytes of step 0
// of the block's first tile and plane ([tile][plane][kPlaneBytes] layout).
template <int KW, int KA, int NBT>
__device__ __forceinline__ void contract_tiles(const uint4 (&araw)[KW][2], const unsigned char* tile,
                                               v4f (&acc)[NBT][KW][KA]) {
  // (the staged tiles hold 0.0 beyond the end of a vector, so the accumulators are the dot products of the codes)
#pragma unroll
  for (int bt = 0; bt < NBT; ++bt)
#pragma unroll
    for (int i = 0; i < KW; ++i)
#pragma unroll
      for (int j = 0; j < KA; ++j) acc[bt][i][j] = v4f{0.f, 0.f, 0.f, 0.f};
  uint4 bop[KA], bnx[KA], aop[KW], anx[KW];
#pragma unroll
  for (int j = 0; j < KA; ++j) bop[j] = *reinterpret_cast<const uint4*>(tile + j * kPlaneBytes);
#pragma unroll
  for (int i = 0; i < KW; ++i) aop[i] = expand4_signed(word_of(araw[i], 0));
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int u = 0; u < kSteps * NBT; ++u) {
    const int bt = u % NBT;
    const int tn = (u + 1) / NBT, bn = (u + 1) % NBT;
    if (u + 1 < kSteps * NBT) {
#pragma unroll
      for (int j = 0; j < KA; ++j)
        bnx[j] = *reinterpret_cast<const uint4*>(tile + (bn * KA + j) * kPlaneBytes + tn * kTileB * 64);
      if (bn == 0) {
#pragma unroll
        for (int i = 0; i < KW; ++i) anx[i] = expand4_signed(word_of(araw[i], tn));
      }
    }
#pragma unroll
    for (int i = 0; i < KW; ++i)
#pragma unroll
      for (int j = 0; j < KA; ++j)
        acc[bt][i][j] = mfma_fp4(aop[i], bop[j], acc[bt][i][j]);
    __builtin_amdgcn_sched_group_barrier(0x100, KA, 0);
#pragma unroll
    for (int g = 0; g < KW * KA; ++g) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x002, 3, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int j = 0; j < KA; ++j) bop[j] = bnx[j];
    if (bn == 0) {
#pragma unroll
      for (int i = 0; i < KW; ++i) aop[i] = anx[i];
    }
  }
  // An MFMA reads its operands from all 64 lanes, but the compiler treats it as lane-local and
  // would sink it into the divergent branches that guard the stores of the epilogues, where lanes
  // of padded batch columns -- which still supply weight rows -- are masked off.  Pin the
  // accumulators here, in uniform control flow.
  settle_accumulators<16>();
#pragma unroll
  for (int bt = 0; bt < NBT; ++bt)
#pragma unroll
    for (int i = 0; i < KW; ++i)
#pragma unroll
      for (int j = 0; j < KA; ++j) asm volatile("" : "+v"(acc[bt][i][j]));
}

// The packed activation words of one operand block (NBT * 16 batch entries from bg0 on, KA planes): requests, and then, staged
// in LDS as {-1, +1} 4-bit codes with 0.0 at the positions from nlen on, [tile][plane][step][batch entry][k-block][16 B].
template <int KA, int NBT, int NTHREADS>
__device__ __forceinline__ void load_activation_words(const uint32_t* Xp, int batch, int bg0, int wq,
                                                      uint4 (&xw)[(NBT * KA * kTileB * 8 + NTHREADS - 1) / NTHREADS]) {
  constexpr int kGroupB = NBT * kTileB;
  constexpr int kItems = NBT * KA * kTileB * 8;
  constexpr int kIter = (kItems + NTHREADS - 1) / NTHREADS;
  const uint4* Xp4 = reinterpret_cast<const uint4*>(Xp);
#pragma unroll
  for (int it = 0; it < kIter; ++it) {
    const int e = threadIdx.x + it * NTHREADS;
    const int q = e & 7, nn = (e >> 3) % kGroupB, j = (e >> 3) / kGroupB;
    const bool valid = e < kItems && bg0 + nn < batch && q < wq;
    const int bb = bg0 + nn < batch ? bg0 + nn : batch - 1;
    const uint4 v = Xp4[((e < kItems ? j : 0) * batch + bb) * wq + (q < wq ? q : 0)];
    xw[it] = valid ? v : make_uint4(0, 0, 0, 0);
  }
}
template <int KA, int NBT, int NTHREADS>
__device__ __forceinline__ void stage_activation_words(const uint4 (&xw)[(NBT * KA * kTileB * 8 + NTHREADS - 1) / NTHREADS],
                                                       unsigned char* btile, int nlen) {
  constexpr int kGroupB = NBT * kTileB;
  constexpr int kItems = NBT * KA * kTileB * 8;
  constexpr int kIter = (kItems + NTHREADS - 1) / NTHREADS;
#pragma unroll
  for (int it = 0; it < kIter; ++it) {
    const int e = threadIdx.x + it * NTHREADS;
    const int q = e & 7, nn = (e >> 3) % kGroupB, j = (e >> 3) / kGroupB;
    const int bt = nn >> 4, n16 = nn & 15;
    const uint4 w4 = xw[it];
    if (e < kItems) {
      // words 4q .. 4q+3 of the row: k-block q >> 1, steps 4 * (q & 1) + 0..3
      uint4* dst = reinterpret_cast<uint4*>(btile + (bt * KA + j) * kPlaneBytes + ((4 * (q & 1)) * kTileB + n16) * 64 +
                                            (q >> 1) * 16);
      // word 4q + c of the row holds positions 32 (4q + c) .. + 31
      auto inside = [&](int c) {
        const int left = nlen - 32 * (4 * q + c);
        return left >= 32 ? 0xffffffffu : left <= 0 ? 0u : ((1u << left) - 1u);
      };
      dst[0 * kTileB * 4] = expand4_signed_valid(w4.x, inside(0));
      dst[1 * kTileB * 4] = expand4_signed_valid(w4.y, inside(1));
      dst[2 * kTileB * 4] = expand4_signed_valid(w4.z, inside(2));
      dst[3 * kTileB * 4] = expand4_signed_valid(w4.w, inside(3));
    }
  }
}

// FIRST: a wave in its contraction has precedence (launch_one).
template <int KW, int KA, int NBT, bool FIRST>
__global__ __launch_bounds__(64 * kWaves) void mfma4w_kernel(BmvArgs a, int rb_per_wg, int rowblocks) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  constexpr int kGroupB = NBT * kTileB;               // batch entries per workgroup
  constexpr int kIter = (NBT * KA * kTileB * 8 + 64 * kWaves - 1) / (64 * kWaves);
  unsigned char* btile = smem;                                           // [tile][plane][kPlaneBytes]

  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, l4 = lane >> 4;
  const int bg0 = blockIdx.y * kGroupB;
  const int batch = a.batch;
  const int m = (int)a.m;
  const int nlen = a.blk[0].n;
  const int wq = (nlen + 127) >> 7;  // 16-byte groups per row
  const uint4* Wp4 = reinterpret_cast<const uint4*>(a.blk[0].Wp);
  const float* alpha = a.blk[0].alpha;
  const int rb_first = blockIdx.x * rb_per_wg;
  int rb_end = rb_first + rb_per_wg;
  if (rb_end > rowblocks) rb_end = rowblocks;

  // ---- packed activation words, 16 bytes per thread and round, coalesced.  Item e: group q = e % 8 of the row of batch entry
  // (e / 8) % kGroupB of plane e / (8 kGroupB).  Staged while the coefficients are under way, before the first weights are asked for;
  // with nine products per tile after that (W3/A3 20000 x 900 batch 70 10.2 us, 10.9), with twelve at once, or the words would be spilled
  // (W4/A3 4096 x 512 batch 256 9.1, 9.8).
  constexpr bool kWeightsFirst = KW * KA == 9, kAtOnce = KW * KA >= 12;
  uint4 xw[kIter];
  load_activation_words<KA, NBT, 64 * kWaves>(a.blk[0].Xp, batch, bg0, wq, xw);
  if constexpr (kAtOnce) {
    stage_activation_words<KA, NBT, 64 * kWaves>(xw, btile, nlen);
    lds_barrier();
  }

  // coefficients of this lane's batch column, one column per tile
  int bcol[NBT];
  bool bok[NBT];
  float btv[NBT][KA];
#pragma unroll
  for (int bt = 0; bt < NBT; ++bt) {
    bcol[bt] = bg0 + bt * kTileB + l16;
    bok[bt] = bcol[bt] < batch;
    const int bc = bok[bt] ? bcol[bt] : batch - 1;
#pragma unroll
    for (int j = 0; j < KA; ++j) btv[bt][j] = a.blk[0].beta[bc * KA + j];
  }

  // optional: the output row whose value is wanted on its own, per batch column
  long long tg[NBT];
#pragma unroll
  for (int bt = 0; bt < NBT; ++bt) tg[bt] = (a.tgt && bok[bt]) ? a.tgt[bcol[bt]] : -1;

  float lse_m[NBT], lse_s[NBT];  // running (max, sum exp) of this lane's outputs, per tile
#pragma unroll
  for (int bt = 0; bt < NBT; ++bt) {
    lse_m[bt] = kLseLow;
    lse_s[bt] = 0.0f;
  }
  float* const lse_part = a.lse_part;
  const unsigned char* tile = btile + l16 * 64 + l4 * 16;

  // Requests of a row block: its packed weight words in the A-operand view (lane = (tile row l16, k-block
  // l4)) and its row coefficients and bias, one value per lane.  Every request is unconditional on a
  // clamped row (results of rows outside the matrix are masked or never stored), and those of the next row
  // block of this wave go out before the contraction of the current one.
  const int plane = m * wq;
  auto request_rowblock = [&](int rb, uint4 (&raw)[KW][2], float& coef, float& bs) {
    const int rbc = rb < rowblocks ? rb : rowblocks - 1;
    const int wrow = rbc * 16 + l16;
    const int base = (wrow < m ? wrow : m - 1) * wq;
#pragma unroll
    for (int i = 0; i < KW; ++i)
#pragma unroll
      for (int v = 0; v < 2; ++v) {
        const int g = 2 * l4 + v;
        raw[i][v] = Wp4[base + i * plane + (g < wq ? g : 0)];
      }
    // lane l < 16 KW: coefficient l % KW of row rb * 16 + l / KW; lane l < 16: bias of row rb * 16 + l
    const int ci = rbc * 16 * KW + (lane < 16 * KW ? lane : 0);
    coef = alpha[ci < m * KW ? ci : m * KW - 1];
    const int bi = rbc * 16 + l16;
    bs = a.bias0 ? a.bias0[bi < m ? bi : m - 1] : 0.0f;
  };
  uint4 anext[KW][2];
  float coef_next, bias_next;
  if constexpr (kWeightsFirst) request_rowblock(rb_first + wv, anext, coef_next, bias_next);
  if constexpr (!kAtOnce) stage_activation_words<KA, NBT, 64 * kWaves>(xw, btile, nlen);
  if constexpr (!kWeightsFirst) request_rowblock(rb_first + wv, anext, coef_next, bias_next);
  if constexpr (!kAtOnce) lds_barrier();  // (the weights under way are not waited for)

  for (int rb = rb_first + wv; rb < rb_end; rb += kWaves) {
    // ---- weight side of the row block, shared by all tiles
    const int wrow_a = rb * 16 + l16;
    const bool wok = wrow_a < m;
    uint4 araw[KW][2];
#pragma unroll
    for (int i = 0; i < KW; ++i)
#pragma unroll
      for (int v = 0; v < 2; ++v)
        araw[i][v] = (wok && 2 * l4 + v < wq) ? anext[i][v] : make_uint4(0, 0, 0, 0);
    const float coef_req = coef_next, bias_req = bias_next;
    request_rowblock(rb + kWaves, anext, coef_next, bias_next);
    // C view: rows 4 * l4 + r
    int crow0 = rb * 16 + 4 * l4;
    bool cok[4];
    float alr[4][KW], bias[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      cok[r] = crow0 + r < m;
#pragma unroll
      for (int i = 0; i < KW; ++i) alr[r][i] = __shfl(coef_req, (4 * l4 + r) * KW + i, kWave);
      bias[r] = __shfl(bias_req, 4 * l4 + r, kWave);
    }
    // ---- contraction with all tiles
    v4f acc[NBT][KW][KA];
    if constexpr (FIRST) __builtin_amdgcn_s_setprio(2);
    contract_tiles<KW, KA, NBT>(araw, tile, acc);
    if constexpr (FIRST) __builtin_amdgcn_s_setprio(0);

    // ---- epilogue per tile, lane = (batch column l16, row quad l4): the accumulators are the dot products
    // d_ij of the codes (integers, exact in binary32);  y = sum_i alpha_i sum_j beta_j d_ij
#pragma unroll
    for (int bt = 0; bt < NBT; ++bt) {
      float yv[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        float y = 0.0f;
#pragma unroll
        for (int i = 0; i < KW; ++i) {
          float inner = 0.0f;
#pragma unroll
          for (int j = 0; j < KA; ++j) inner = fmaf(btv[bt][j], acc[bt][i][j][r], inner);
          y = fmaf(alr[r][i], inner, y);
        }
        yv[r] = y + bias[r];
      }
      if (a.tgt_out && bok[bt]) {  // (no accumulation in this use)
        const long long d = tg[bt] - crow0;
        if (d >= 0 && d < 4) {
          const float yt = d == 0 ? yv[0] : d == 1 ? yv[1] : d == 2 ? yv[2] : yv[3];
          if (crow0 + d < m) a.tgt_out[bcol[bt]] = yt;
        }
      }
      if (a.Y && bok[bt]) {
        float* yp = a.Y + (long long)bcol[bt] * m + crow0;
        if (a.accumulate) {
#pragma unroll
          for (int r = 0; r < 4; ++r)
            if (cok[r]) yv[r] += yp[r];
        }
        if ((m & 3) == 0 && cok[3]) {
          // the four rows of this lane are consecutive in Y[b][.]: one aligned 16-byte store
          *reinterpret_cast<float4*>(yp) = make_float4(yv[0], yv[1], yv[2], yv[3]);
        } else {
#pragma unroll
          for (int r = 0; r < 4; ++r)
            if (cok[r]) yp[r] = yv[r];
        }
      }
      if (lse_part) {  // uniform: fold this row block's outputs into the running (max, sum)
        float mx = lse_m[bt];
#pragma unroll
        for (int r = 0; r < 4; ++r) mx = fmaxf(mx, cok[r] ? yv[r] : kLseLow);
        float sm = lse_s[bt] * __expf(lse_m[bt] - mx);
#pragma unroll
        for (int r = 0; r < 4; ++r) sm += cok[r] ? __expf(yv[r] - mx) : 0.0f;
        lse_m[bt] = mx;
        lse_s[bt] = sm;
      }
    }
  }

  if (lse_part) {  // uniform
    // One slot per workgroup and batch column: every wave merges its four row quads (lanes 16
    // apart) and leaves the pair in LDS (the staged activations are no longer needed once all
    // waves are past their contractions); wave 0 merges the eight and writes.  A wave that had
    // no row block contributes the neutral pair.
    float2* xch = reinterpret_cast<float2*>(smem);  // [wave][tile][column]
    __syncthreads();
#pragma unroll
    for (int bt = 0; bt < NBT; ++bt) {
      float mm = lse_m[bt], ss = lse_s[bt];
#pragma unroll
      for (int o = 16; o <= 32; o <<= 1) {
        const float m2 = __shfl_xor(mm, o, kWave), s2 = __shfl_xor(ss, o, kWave);
        lse_merge(mm, ss, m2, s2);
      }
      if (l4 == 0) xch[(wv * NBT + bt) * kTileB + l16] = make_float2(mm, ss);
    }
    __syncthreads();
    if (tid < NBT * kTileB) {
      const int b = bg0 + tid;  // tid = tile * 16 + column
      float mm = kLseLow, ss = 0.0f;
#pragma unroll
      for (int w = 0; w < kWaves; ++w) {
        const float2 p = xch[w * NBT * kTileB + tid];
        lse_merge(mm, ss, p.x, p.y);
      }
      if (b < batch) {
        float* dst = lse_part + ((long long)b * a.lse_slots + blockIdx.x) * 2;
        dst[0] = mm;
        dst[1] = ss;
      }
    }
  }
}

// The recurrent steps (Eq. 6 and the GRU) in the same work split, for batches of 128 and more: a
// wave owns 4 hidden units x all gates (the 16 tile rows are 4 units x 4 gates, so that in the C
// layout one lane holds every gate of one unit for one batch entry) x NBT batch tiles x both operand
// blocks, one block after the other, and applies the cell in registers.  Both blocks' activation
// tiles are staged in LDS.  The pre-activations are formed from the exact integer dot products
// (h_t goes back into the on-line quantizer, where a difference in the last digits can move an
// entry across an interval boundary), in the same order as the one-tile kernel.
template <int KW, int KA, int NBT, int EPI, int NWV>
__global__ __launch_bounds__(64 * NWV) void mfma4wc_kernel(BmvArgs a, int rb_per_wg, int rowblocks) {
  static_assert(EPI == kEpiLstm || EPI == kEpiGru, "cell modes only");
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  constexpr int NG = (EPI == kEpiGru) ? 3 : 4;
  constexpr int kGroupB = NBT * kTileB;
  constexpr int kBlockBytes = NBT * KA * kPlaneBytes;
  constexpr int kIter = (NBT * KA * kTileB * 8 + 64 * NWV - 1) / (64 * NWV);
  unsigned char* btile = smem;                                        // [block][tile][plane][kPlaneBytes]

  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  uint4* const mine = reinterpret_cast<uint4*>(smem + 2 * kBlockBytes) + wv * (kTileB * kTurn);  // this wave's piece
  const int l16 = lane & 15, l4 = lane >> 4;
  const int bg0 = blockIdx.y * kGroupB;
  const int batch = a.batch;
  const int m = (int)a.m, H = (int)a.H;
  int nlen[2], wq[2];
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    nlen[k] = a.blk[k].n;
    wq[k] = (nlen[k] + 127) >> 7;
  }
  const int rb_first = blockIdx.x * rb_per_wg;
  int rb_end = rb_first + rb_per_wg;
  if (rb_end > rowblocks) rb_end = rowblocks;

  uint4 xw[2][kIter];
#pragma unroll
  for (int k = 0; k < 2; ++k) load_activation_words<KA, NBT, 64 * NWV>(a.blk[k].Xp, batch, bg0, wq[k], xw[k]);

  // Requests of a row block, all unconditional on clamped rows and units (what a row outside the matrix gives is not used, a piece
  // past the end of a row meets 0.0 of the staged operand): weight words, whole rows of 128 bytes by 8 adjacent lanes (16 bytes of
  // 64 rows per request keep the memory pipe busy four times as long), to be turned into the A view through LDS; row coefficients
  // and biases, one value per lane (lane l < 16 KW: coefficient l % KW of tile row l / KW); previous state in the C view (lane =
  // (unit l4, batch column l16)).  Those of the first row block go out between the staging of the activations and the barrier, those
  // of the next one before the contraction of the current: asked for where they were used, the weights of either operand block and
  // the coefficients cost a trip to memory each.  us per LSTM step on packed operands, where they were used / all before the staging,
  // which they delay / here: W2/A2 600 units batch 600 12.6 / 10.2 / 9.6, 1024 batch 256 8.2 / 8.35 / 7.6, W1/A2 6.7 / 7.1 / 6.5, W4/A1 9.5 /
  // 10.0 / 8.5, W2/A3 1000 units batch 160 11.0 / 10.2 / 9.3.  Of 78 combinations of size and bits none is slower than the first.
  // With four planes in a workgroup of eight waves only block 0 is asked for a row block ahead, block 1 when its row block begins: both
  // are 256 registers with 9 spilled (W4/A1 LSTM), block 0 is 240 and none.
  constexpr bool kBothBlocks = KW < 4 || NWV < 8;
  struct Row {
    uint4 w[2][KW][2];
    float coef[2], bias[2], prev[NBT];
  };
  auto matrix_row = [&](int rb, int tile_row) {
    const int unit = rb * 4 + (tile_row >> 2), gate = tile_row & 3;
    return (gate < NG ? gate : 0) * H + (unit < H ? unit : H - 1);
  };
  auto request_weights = [&](int rb, int k, Row& r) {
    rb = rb < rowblocks ? rb : rowblocks - 1;
    const int rows[2] = {matrix_row(rb, lane >> 3), matrix_row(rb, 8 + (lane >> 3))};
    const uint4* const Wp4 = reinterpret_cast<const uint4*>(a.blk[k].Wp) + ((lane & 7) < wq[k] ? (lane & 7) : 0);
    const int plane = m * wq[k];
#pragma unroll
    for (int i = 0; i < KW; ++i)
#pragma unroll
      for (int v = 0; v < 2; ++v) r.w[k][i][v] = Wp4[rows[v] * wq[k] + i * plane];
  };
  auto request = [&](int rb, Row& r) {
    request_weights(rb, 0, r);
    if constexpr (kBothBlocks) request_weights(rb, 1, r);
    rb = rb < rowblocks ? rb : rowblocks - 1;
    const int row = matrix_row(rb, l16);
    const int cl = lane < 16 * KW ? lane : 0, crow = matrix_row(rb, cl / KW);
#pragma unroll
    for (int k = 0; k < 2; ++k) r.coef[k] = a.blk[k].alpha[crow * KW + cl % KW];
    r.bias[0] = a.bias0 ? a.bias0[row] : 0.0f;
    r.bias[1] = (EPI == kEpiGru && a.bias1) ? a.bias1[row] : 0.0f;
    const int unit = rb * 4 + l4;
#pragma unroll
    for (int bt = 0; bt < NBT; ++bt) {
      const int col = bg0 + bt * kTileB + l16;
      const int t = (col < batch ? col : batch - 1) * H + (unit < H ? unit : H - 1);
      r.prev[bt] = (EPI == kEpiLstm) ? a.c_prev[t] : a.h_prev[t];
    }
  };

  // per batch column of this lane (one per tile) and operand block: beta_j
  int bcol[NBT];
  bool bok[NBT];
  float btv[2][NBT][KA];
#pragma unroll
  for (int bt = 0; bt < NBT; ++bt) {
    bcol[bt] = bg0 + bt * kTileB + l16;
    bok[bt] = bcol[bt] < batch;
    const int bc = bok[bt] ? bcol[bt] : batch - 1;
#pragma unroll
    for (int k = 0; k < 2; ++k)
#pragma unroll
      for (int j = 0; j < KA; ++j) btv[k][bt][j] = a.blk[k].beta[bc * KA + j];
  }
#pragma unroll
  for (int k = 0; k < 2; ++k)
    stage_activation_words<KA, NBT, 64 * NWV>(xw[k], btile + k * kBlockBytes, nlen[k]);
  Row next;
  request(rb_first + wv, next);
  lds_barrier();  // (the requests under way are not waited for)

  for (int rb = rb_first + wv; rb < rb_end; rb += NWV) {
    Row now = next;
    if constexpr (!kBothBlocks) request_weights(rb, 1, now);
    if (rb + NWV < rb_end) request(rb + NWV, next);
    // C view: this lane's hidden unit, rows r = gate r
    const int unit_c = rb * 4 + l4;
    const bool uok = unit_c < H;
    float bias0[4], bias1[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      bias0[r] = __shfl(now.bias[0], 4 * l4 + r, kWave);
      bias1[r] = EPI == kEpiGru ? __shfl(now.bias[1], 4 * l4 + r, kWave) : 0.0f;
    }

    float ysum[2][NBT][4];
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      float alr[4][KW];
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int i = 0; i < KW; ++i) alr[r][i] = __shfl(now.coef[k], (4 * l4 + r) * KW + i, kWave);
      // (lane = (tile row l16 = 4 * unit + gate, k-block l4); LDS serves the accesses of a wave in order)
#pragma unroll
      for (int i = 0; i < KW; ++i) {
#pragma unroll
        for (int v = 0; v < 2; ++v) mine[(8 * v + (lane >> 3)) * kTurn + (lane & 7)] = now.w[k][i][v];
#pragma unroll
        for (int v = 0; v < 2; ++v) now.w[k][i][v] = mine[l16 * kTurn + 2 * l4 + v];
      }
      v4f acc[NBT][KW][KA];
      contract_tiles<KW, KA, NBT>(now.w[k], btile + k * kBlockBytes + l16 * 64 + l4 * 16, acc);
      // the accumulators are the dot products d_ij of the codes (integers, exact in binary32):
      // y = sum_i alpha_i sum_j beta_j d_ij
#pragma unroll
      for (int bt = 0; bt < NBT; ++bt)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          float y = 0.0f;
#pragma unroll
          for (int i = 0; i < KW; ++i) {
            float inner = 0.0f;
#pragma unroll
            for (int j = 0; j < KA; ++j) inner = fmaf(btv[k][bt][j], acc[bt][i][j][r], inner);
            y = fmaf(alr[r][i], inner, y);
          }
          ysum[k][bt][r] = y;
        }
    }

    // (no early exit for padded batch columns or units: every lane stays active through the
    // loop, the stores are predicated instead)
#pragma unroll
    for (int bt = 0; bt < NBT; ++bt) {
      const int t = bcol[bt] * H + unit_c;
      if constexpr (EPI == kEpiLstm) {
        const float gi = sigmoidf_dev(ysum[0][bt][0] + ysum[1][bt][0] + bias0[0]);
        const float gf = sigmoidf_dev(ysum[0][bt][1] + ysum[1][bt][1] + bias0[1]);
        const float go = sigmoidf_dev(ysum[0][bt][2] + ysum[1][bt][2] + bias0[2]);
        const float gg = tanhf_dev(ysum[0][bt][3] + ysum[1][bt][3] + bias0[3]);
        const float c = fmaf(gf, now.prev[bt], gi * gg);
        const float h = go * tanhf_dev(c);
        if (bok[bt] && uok) {
          a.c_out[t] = c;
          a.h_out[t] = h;
          if (a.hs_out) a.hs_out[t] = h;
        }
      } else {
        const float rg = sigmoidf_dev(ysum[0][bt][0] + ysum[1][bt][0] + bias0[0] + bias1[0]);
        const float z = sigmoidf_dev(ysum[0][bt][1] + ysum[1][bt][1] + bias0[1] + bias1[1]);
        const float nn = tanhf_dev(fmaf(rg, ysum[1][bt][2] + bias1[2], ysum[0][bt][2] + bias0[2]));
        if (bok[bt] && uok) a.h_out[t] = fmaf(z, now.prev[bt] - nn, nn);
      }
    }
  }
}

// The recurrent steps when there are too few row-block x batch-tile tasks to give every SIMD more than
// one wave: one workgroup of pair_body per (row-block group, batch group).
template <int KW, int KA, int NBT, int EPI, int NWV, int NC>
__global__ __launch_bounds__(64 * NWV) void mfma4p_kernel(BmvArgs a, int rowblocks) {
  __shared__ float4 xch[(NWV / 2) * NBT * 64];  // [pair][tile][lane]: the h-side sums on their way to the x wave
  extern __shared__ __attribute__((aligned(16))) uint4 turn[];
  asm volatile("" ::AMQ_ARG(a.blk[0].Wp), AMQ_ARG(a.blk[0].alpha), AMQ_ARG(a.blk[0].Xp), AMQ_ARG(a.blk[0].beta),
               AMQ_ARG(a.blk[0].n), AMQ_ARG(a.blk[1].Wp), AMQ_ARG(a.blk[1].alpha), AMQ_ARG(a.blk[1].Xp),
               AMQ_ARG(a.blk[1].beta), AMQ_ARG(a.blk[1].n), AMQ_ARG(a.m), AMQ_ARG(a.H), AMQ_ARG(a.batch), AMQ_ARG(a.bias0),
               AMQ_ARG(a.bias1), AMQ_ARG(a.c_prev), AMQ_ARG(a.h_prev), AMQ_ARG(a.h_out), AMQ_ARG(a.c_out),
               AMQ_ARG(a.hs_out), AMQ_ARG(rowblocks));
  pair_body<KW, KA, NBT, EPI, NWV, kPairBoth, NC>(a, rowblocks, blockIdx.x, blockIdx.y, turn, xch);
}

// Tiles per wave: as many as keep the accumulators within about 100 registers.
constexpr int max_tiles(int kw, int ka) { return 24 / (kw * ka) > 4 ? 4 : 24 / (kw * ka); }

// Row blocks of a workgroup: about one workgroup per compute unit (registers and the staged activations allow no second one);
// in multiples of 4, so that its four SIMDs (waves w and w + 4 share one) get the same number of passes.
int blocks_each(int rowblocks, int groups) {
  const int splits = groups < 256 ? 256 / groups : 1;
  const int per = ((rowblocks + splits - 1) / splits + 3) / 4 * 4;
  return per < kWaves ? kWaves : per;
}

// Of the two waves of a SIMD the one in its contraction goes first (by age, a wave in its epilogue keeps the matrix cores from the
// younger one), from more than four row blocks per wave on: us, 10000 x 900 W2/A2 batch 1000 25.0 -> 23.7, 20000 x 300 W4/A3 batch 1000
// 93 -> 83; with two or three 0 to 2 % slower (10000 x 1024 W3/A3 batch 128 12.7 / 12.9).  A form of its own, as the branch splits the
// contraction's scheduling (W4/A3 18 registers spilled, 6).
template <int KW, int KA, int NBT>
hipError_t launch_one(BmvArgs a, hipStream_t s, int* lse_slots) {
  if constexpr (NBT > max_tiles(KW, KA) || NBT < 2) {
    return hipErrorInvalidValue;
  } else {
    const int rowblocks = (int)((a.m + 15) / 16);
    const int groups = (a.batch + NBT * kTileB - 1) / (NBT * kTileB);
    const int per = blocks_each(rowblocks, groups);
    const bool first = per > 4 * kWaves;
    const auto kernel = first ? &mfma4w_kernel<KW, KA, NBT, true> : &mfma4w_kernel<KW, KA, NBT, false>;
    constexpr size_t lds = (size_t)NBT * KA * kPlaneBytes;
    static std::atomic<unsigned long long> configured[2] = {{0}, {0}};
    {
      hipError_t e = ensure_dynamic_lds(reinterpret_cast<const void*>(kernel), (int)lds, configured[first]);
      if (e != hipSuccess) return e;
    }
    dim3 grid((unsigned)((rowblocks + per - 1) / per), (unsigned)groups);
    const long long slots = grid.x;  // one per workgroup of a batch group
    if (slots > kLseMaxSlots || slots > a.lse_cap) a.lse_part = nullptr;
    a.lse_slots = (int)slots;
    if (lse_slots) *lse_slots = a.lse_part ? (int)slots : 0;
    hipLaunchKernelGGL(kernel, grid, dim3(64 * kWaves), lds, s, a, per, rowblocks);
    return hipGetLastError();
  }
}

template <int KW, int KA>
hipError_t launch_tiles(const BmvArgs& a, int nbt, hipStream_t s, int* lse_slots) {
  switch (nbt) {
    case 2: return launch_one<KW, KA, 2>(a, s, lse_slots);
    case 3: return launch_one<KW, KA, 3>(a, s, lse_slots);
    case 4: return launch_one<KW, KA, 4>(a, s, lse_slots);
  }
  return hipErrorInvalidValue;
}

template <int KW>
hipError_t launch_ka(const BmvArgs& a, int k_a, int nbt, hipStream_t s, int* lse_slots) {
  switch (k_a) {
    case 1: return launch_tiles<KW, 1>(a, nbt, s, lse_slots);
    case 2: return launch_tiles<KW, 2>(a, nbt, s, lse_slots);
    case 3: return launch_tiles<KW, 3>(a, nbt, s, lse_slots);
    case 4: return launch_tiles<KW, 4>(a, nbt, s, lse_slots);
  }
  return hipErrorInvalidValue;
}

// Batch tiles per wave for this product: the register budget's maximum, lowered so that the
// batch groups come out even (5 tiles -> 3 + 2 rather than 4 + 1).
int tiles_per_wave(int k_w, int k_a, int batch) {
  const int cap = max_tiles(k_w, k_a);
  if (cap < 2) return 0;
  const int tiles = (batch + kTileB - 1) / kTileB;
  const int groups = (tiles + cap - 1) / cap;
  const int nbt = (tiles + groups - 1) / groups;
  return nbt < 2 ? 0 : nbt;
}

// Cell modes: tiles per wave bounded by the accumulators (as above) and by the LDS that both
// operand blocks' activation tiles take (2 * NBT * KA * 8 KiB <= 144 KiB, of 160 with the waves' pieces of 2.25).  With at most four
// plane pairs, two tiles per wave in 8-wave workgroups fit 256 registers and keep two waves on
// every SIMD (each hides the other's load latencies: measured faster than four tiles per wave
// with one wave per SIMD); beyond that, 4-wave workgroups with up to 512 registers per wave.
constexpr int max_cell_tiles(int kw, int ka) {
  if (kw * ka <= 4) return 2;
  int c = max_tiles(kw, ka);
  return 9 / ka < c ? 9 / ka : c;
}
constexpr int cell_waves(int kw, int ka) { return kw * ka <= 4 ? 8 : 4; }
int cell_tiles_per_wave(int k_w, int k_a, int batch) {
  const int cap = max_cell_tiles(k_w, k_a);
  if (cap < 2) return 0;
  const int tiles = (batch + kTileB - 1) / kTileB;
  const int groups = (tiles + cap - 1) / cap;
  const int nbt = (tiles + groups - 1) / groups;
  return nbt < 2 ? 0 : nbt;
}

template <int KW, int KA, int NBT, int EPI>
hipError_t launch_cell_one(const BmvArgs& a, hipStream_t s) {
  if constexpr (NBT > max_cell_tiles(KW, KA) || NBT < 2) {
    return hipErrorInvalidValue;
  } else {
    constexpr int NWV = cell_waves(KW, KA);
    const int rowblocks = (int)((a.H + 3) / 4);
    const int groups = (a.batch + NBT * kTileB - 1) / (NBT * kTileB);
    // about one workgroup per compute unit; row blocks per workgroup in multiples of 4, so that
    // its four SIMDs get the same number of passes
    int splits = 256 / groups;
    if (splits < 1) splits = 1;
    int per = (rowblocks + splits - 1) / splits;
    per = (per + 3) / 4 * 4;
    if (per < NWV) per = NWV;
    const size_t lds = (size_t)2 * NBT * KA * kPlaneBytes + sizeof(uint4) * NWV * kTileB * kTurn;
    static std::atomic<unsigned long long> configured{0};
    {
      hipError_t e = ensure_dynamic_lds(reinterpret_cast<const void*>(&mfma4wc_kernel<KW, KA, NBT, EPI, NWV>), (int)lds,
                                        configured);
      if (e != hipSuccess) return e;
    }
    dim3 grid((unsigned)((rowblocks + per - 1) / per), (unsigned)groups);
    hipLaunchKernelGGL((mfma4wc_kernel<KW, KA, NBT, EPI, NWV>), grid, dim3(64 * NWV), lds, s, a, per, rowblocks);
    return hipGetLastError();
  }
}

template <int KW, int KA, int EPI>
hipError_t launch_cell_tiles(const BmvArgs& a, int nbt, hipStream_t s) {
  switch (nbt) {
    case 2: return launch_cell_one<KW, KA, 2, EPI>(a, s);
    case 3: return launch_cell_one<KW, KA, 3, EPI>(a, s);
    case 4: return launch_cell_one<KW, KA, 4, EPI>(a, s);
  }
  return hipErrorInvalidValue;
}

template <int KW, int EPI>
hipError_t launch_cell_ka(const BmvArgs& a, int k_a, int nbt, hipStream_t s) {
  switch (k_a) {
    case 1: return launch_cell_tiles<KW, 1, EPI>(a, nbt, s);
    case 2: return launch_cell_tiles<KW, 2, EPI>(a, nbt, s);
    case 3: return launch_cell_tiles<KW, 3, EPI>(a, nbt, s);
    case 4: return launch_cell_tiles<KW, 4, EPI>(a, nbt, s);
  }
  return hipErrorInvalidValue;
}

template <int EPI>
hipError_t launch_cell_kw(const BmvArgs& a, int k_w, int k_a, int nbt, hipStream_t s) {
  switch (k_w) {
    case 1: return launch_cell_ka<1, EPI>(a, k_a, nbt, s);
    case 2: return launch_cell_ka<2, EPI>(a, k_a, nbt, s);
    case 3: return launch_cell_ka<3, EPI>(a, k_a, nbt, s);
    case 4: return launch_cell_ka<4, EPI>(a, k_a, nbt, s);
  }
  return hipErrorInvalidValue;
}

// Measured on config 3 (256 row blocks x 4 batch tiles, W3/A3), whole step: one tile per wave in
// workgroups of 8 waves 12.4 us; two tiles per wave in workgroups of 4 (one wave per SIMD, weights
// fetched half as often, activation operands shared by two row blocks instead of four) 13.0 us; two
// tiles, 8 waves (half the compute units) 14.3 us.
template <int KW, int KA, int EPI, int NC>
hipError_t launch_pair_one(const BmvArgs& a, hipStream_t s) {
  if constexpr (KW > 3 || KW * KA > 9) {
    return hipErrorInvalidValue;
  } else {
    constexpr int NBT = 1, NWV = 8;
    const int rowblocks = (int)((a.H + 3) / 4);
    const int groups = (a.batch + NBT * kTileB - 1) / (NBT * kTileB);
    dim3 grid((unsigned)((rowblocks + NWV / 2 - 1) / (NWV / 2)), (unsigned)groups);
    BmvArgs b = a;
    AMQ_PHASE_ATTACH(b);
    constexpr size_t lds = pair_body_lds<KW, KA, NBT, NWV, kPairBoth, NC>();
    static std::atomic<unsigned long long> configured{0};
    {
      hipError_t e = ensure_dynamic_lds(reinterpret_cast<const void*>(&mfma4p_kernel<KW, KA, NBT, EPI, NWV, NC>), (int)lds,
                                        configured);
      if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL((mfma4p_kernel<KW, KA, NBT, EPI, NWV, NC>), grid, dim3(64 * NWV), lds, s, b, rowblocks);
    return hipGetLastError();
  }
}

template <int KW, int KA, int EPI>
hipError_t launch_pair_nc(const BmvArgs& a, hipStream_t s) {
  return a.blk[0].n > 1024 || a.blk[1].n > 1024 ? launch_pair_one<KW, KA, EPI, 2>(a, s) : launch_pair_one<KW, KA, EPI, 1>(a, s);
}

template <int KW, int EPI>
hipError_t launch_pair_ka(const BmvArgs& a, int k_a, hipStream_t s) {
  switch (k_a) {
    case 1: return launch_pair_nc<KW, 1, EPI>(a, s);
    case 2: return launch_pair_nc<KW, 2, EPI>(a, s);
    case 3: return launch_pair_nc<KW, 3, EPI>(a, s);
    case 4: return launch_pair_nc<KW, 4, EPI>(a, s);
  }
  return hipErrorInvalidValue;
}

template <int EPI>
hipError_t launch_pair_kw(const BmvArgs& a, int k_w, int k_a, hipStream_t s) {
  switch (k_w) {
    case 1: return launch_pair_ka<1, EPI>(a, k_a, s);
    case 2: return launch_pair_ka<2, EPI>(a, k_a, s);
    case 3: return launch_pair_ka<3, EPI>(a, k_a, s);
  }
  return hipErrorInvalidValue;
}

}  // namespace

// Recurrent steps at batch 2 and more with vectors of at most 2048 entries.  Where the several-tiles cell kernel
// applies (at most 1024 entries), up to two row-block x tile tasks per SIMD of the chip.
// Batches 2 / 4 / 8 / 16 of longer vectors, LSTM step on packed operands, us, small-batch kernel against this one:
// 1500 units W2/A2 6.4 / 9.4 / 15.4 / 27.4 against 4.9 / 4.8 / 4.9 / 5.0, 2048 units W3/A3 8.7 / 13.7 / 23.8 / 43.7
// against 7.2 / 7.1 / 7.1 / 7.2.  The two add in another order (binary32 partial sums per 128 entries there, exact
// integer sums here), so their last digits differ; against binary64 sums this one is the closer (root mean square error
// of c at 1100 to 2048 units 4.1e-8 to 4.8e-8, there 4.4e-8 to 5.4e-8).
bool mfma4_pair_supported(const BmvArgs& a, int k_w, int k_a, int epi) {
  if (epi != kEpiLstm && epi != kEpiGru) return false;
  const long long nmax = a.blk[0].n > a.blk[1].n ? a.blk[0].n : a.blk[1].n;
  if (nmax > 2048) return false;
  if (k_w > 3 || k_w * k_a > 9) return false;
  const long long tiles = (a.batch + kTileB - 1) / kTileB;
  const long long rowblocks = (a.H + 3) / 4;
  if (a.batch < 2 || tiles > 65535) return false;
  if (nmax <= 1024 && rowblocks * tiles > 2048) return false;
  const long long pieces = (nmax + 127) / 128;
  if (a.m * pieces * k_w >= (1LL << 28)) return false;  // byte offsets within a plane in 32 bits
  if (a.batch * pieces >= (1LL << 28)) return false;
  if ((long long)a.batch * a.H >= (1LL << 29)) return false;
  return true;
}

hipError_t launch_mfma4_pair(const BmvArgs& a, int k_w, int k_a, int epi, hipStream_t s) {
  if (epi == kEpiLstm) return launch_pair_kw<kEpiLstm>(a, k_w, k_a, s);
  if (epi == kEpiGru) return launch_pair_kw<kEpiGru>(a, k_w, k_a, s);
  return hipErrorInvalidValue;
}

// Plain products (no integer hook) with vectors of at most 1024 entries, at least two batch tiles,
// and enough row-block tasks to give every SIMD of the chip two of them; sizes whose element
// offsets fit 32 bits.
bool mfma4w_supported(const BmvArgs& a, int k_w, int k_a) {
  if (a.D || a.groups > 1 || a.blk[0].n > 1024 || (!a.Y && !(a.tgt && a.tgt_out))) return false;
  const int nbt = tiles_per_wave(k_w, k_a, a.batch);
  if (nbt == 0) return false;
  if (a.batch > 65535 * nbt * kTileB) return false;
  if (a.m * 8 * k_w >= (1LL << 31)) return false;  // weight offsets in 16-byte units
  if ((long long)a.batch * a.m >= (1LL << 31)) return false;
  const long long rowblocks = (a.m + 15) / 16;
  const long long groups = (a.batch + nbt * kTileB - 1) / (nbt * kTileB);
  return rowblocks * groups >= 2048;
}

int mfma4w_most_tasks(const BmvArgs& a, int k_w, int k_a) {
  if (!mfma4w_supported(a, k_w, k_a)) return 0;
  const int nbt = tiles_per_wave(k_w, k_a, a.batch);
  return blocks_each((int)((a.m + 15) / 16), (a.batch + nbt * kTileB - 1) / (nbt * kTileB)) / 4 * nbt;
}

hipError_t launch_mfma4w(const BmvArgs& a, int k_w, int k_a, hipStream_t s, int* lse_slots) {
  if (lse_slots) *lse_slots = 0;
  const int nbt = tiles_per_wave(k_w, k_a, a.batch);
  switch (k_w) {
    case 1: return launch_ka<1>(a, k_a, nbt, s, lse_slots);
    case 2: return launch_ka<2>(a, k_a, nbt, s, lse_slots);
    case 3: return launch_ka<3>(a, k_a, nbt, s, lse_slots);
    case 4: return launch_ka<4>(a, k_a, nbt, s, lse_slots);
  }
  return hipErrorInvalidValue;
}

// Recurrent steps with vectors of at most 1024 entries, at least 8 batch tiles, and more row-block x
// batch-tile tasks than the paired-wave form of the one-tile kernel is used for.
bool mfma4w_cell_supported(const BmvArgs& a, int k_w, int k_a, int epi) {
  if (epi != kEpiLstm && epi != kEpiGru) return false;
  if (a.blk[0].n > 1024 || a.blk[1].n > 1024) return false;
  const long long tiles = (a.batch + kTileB - 1) / kTileB;
  const long long rowblocks = (a.H + 3) / 4;
  if (tiles < 8 || rowblocks * tiles <= 2048) return false;
  const int nbt = cell_tiles_per_wave(k_w, k_a, a.batch);
  if (nbt == 0) return false;
  if (a.batch > 65535LL * nbt * kTileB) return false;
  if (a.m * 8 * k_w >= (1LL << 31)) return false;  // weight offsets in 16-byte units
  if ((long long)a.batch * a.H >= (1LL << 31)) return false;
  return true;
}

hipError_t launch_mfma4w_cell(const BmvArgs& a, int k_w, int k_a, int epi, hipStream_t s) {
  const int nbt = cell_tiles_per_wave(k_w, k_a, a.batch);
  if (epi == kEpiLstm) return launch_cell_kw<kEpiLstm>(a, k_w, k_a, nbt, s);
  if (epi == kEpiGru) return launch_cell_kw<kEpiGru>(a, k_w, k_a, nbt, s);
  return hipErrorInvalidValue;
}

}  // namespace amq
