// Whole recurrent sequences of a batch in one launch, spread over the chip (Eq. 6 over a sequence, Sec. 4).
//
// With two launches per step (amq_step.hip) a step of a 1024-unit LSTM at batch 64 costs 9.4 us, of which the matrix
// work is half a microsecond: the rest is launch gaps, the cold misses every new kernel starts with, weights fetched
// and turned into operand layout again at every step, and state that goes through memory.  Here the grid stays
// resident for the whole sequence:
//   - a workgroup of 8 waves owns one batch tile (16 entries) and 4 row blocks (16 hidden units, all gates), one wave
//     per row block and operand block; its weights, coefficients, biases and cell state stay in registers, the
//     weights already in operand layout;
//   - the inputs do not depend on the recurrence: their codes are all formed (or looked up) before this launch, and the
//     x-side sums of step t are formed while the codes of h_{t-1} are under way;
//   - per step two exchanges: every workgroup publishes its h_t; the workgroup in charge of a batch entry (one of
//     those of its tile) gathers the entry's whole h_t, quantizes it (the shared quantizer core on 4 waves) and
//     publishes its codes, which all workgroups of the tile gather as matrix operands (both kinds of wave, where the x side
//     leaves time).  What is published goes through LDS to the x side's waves, which store it: a wave's loads are counted
//     behind its stores, and a store takes 1500 cycles until it is acknowledged, which the polls of the h side's waves would
//     otherwise wait for.
// What is exchanged are 8-byte {value, step tag} pairs, each written with one device-scope store; the readers poll
// the pairs they need until all carry the tag of the step (one way across the chip: about 0.55 us measured), so the
// data is its own arrival signal: no barrier, no ordering between locations.  Two buffers in turn suffice: whoever
// writes the pairs of step t + 2 has seen data of step t + 1 that depend on every reader of step t.
//
// The arithmetic and its order are those of the per-step kernels: the results are the same bit for bit.
//
// All workgroups must be resident at once: the host launches this only where the grid fits the chip, and such launches
// share it by a count kept on the device (amq_resident.h: the reset kernel claims room, the recovery kernel gives it
// back).  Should the chip be shared in a way this cannot see, the waits are bounded: a workgroup that gives up raises a flag, everyone
// leaves, and the launch that always follows (seqw_recover_kernel) computes the piece again from the saved initial
// state, one workgroup per batch entry, with no exchange between workgroups -- slow, but it depends on nobody; without
// the flag it returns at once.
#include <atomic>
#include <mutex>

#include "amq_seqw_body.h"

namespace amq {

namespace {

// How long a workgroup that quantizes waits before it asks for h_{t-1} for the first time, in units of 64 cycles.  A store is seen
// elsewhere after about 1400 cycles, and a gather that comes too early is a whole trip (1600 to 1900 cycles) before the next.  Measured
// with 0 / 10 / 12 / 14 / 16, us per 35 steps: 1024 units batch 64 W2/A2 180 / 181 / 178 / 177 / 178, GRU 187 / 181 / 179 / 178 / 178,
// W3/A3 235 / 230 / 228 / 226 / 226, 650 units batch 20 166 / 160 / 158 / 159 / 159, 2000 units batch 5 228 / 216 / 215 / 216 / 217.  (The
// codes are asked for at once: any delay there is lost, 4 units 2 us, 12 units 8 us.)
// Up to kFewWorkgroups workgroups per tile, no more than there are dies, finish close together and are seen sooner.  Measured there with
// 0 / 4 / 8 / 14: 20 units batch 5 W2/A2 233 / 234 / 238 / 244, 64 batch 5 171 / 172 / 175 / 180, GRU 8 batch 2 158 / 160 / 164 / 170, 100 units with
// inputs of 600 batch 8 189 / 187 / 187 / 192; over 24 kinds of call each, the mean (the least) of the speed without any wait or later store: 20
// units 1.008 / 1.008 / 1.002 / 0.983 (0.988 / 0.988 / 0.967 / 0.924), 64 1.010 / 1.017 / 1.030 / 1.011 (0.981 / 0.992 / 0.973 / 0.935), 100 1.011 /
// 1.017 / 1.029 / 1.021 (0.981 / 0.985 / 0.993 / 0.976); beyond, 160 1.018 / 1.026 / 1.034 / 1.035 (0.994 / 1.001 / 1.002 / 1.014).
constexpr int kFirstPoll = 14, kFirstPollFew = 4, kFewWorkgroups = 8;

// Whether the two waves of a row block share the contraction of its h side, half of K each (the x side's wave has nothing else to do
// then).  The matrix instructions of a compute unit's SIMD are the same either way; what two waves halve is the expansion of weights that
// do not stay expanded in registers, at the price of the partial sums' way through LDS and a barrier.  us per 35 steps, alone / shared: two
// stretches W2/A2 2048 units batch 16 222.9 / 219.3, 1500 batch 20 204.0 / 200.5, W3/A3 334.6 / 325.4, 288.7 / 287.9, GRU 2048 batch 5 331.8 /
// 301.8 (fewer registers spilled as well), W1/A1 1500 143.8 / 139.2, W2/A1 153.0 / 146.6, W1/A2 191.1 / 189.6, W1/A3 237.0 / 232.2; six plane
// products W2/A3 250.1 / 252.7, W3/A2 216.1 / 221.5; W3/A1 161.1 / 158.6, but 2048 units 177.6 / 196.8.  On one stretch it lost 2 to 4 % where that was
// tried, before the x waves gathered codes: W2/A2 180 / 188, W3/A3 228 / 232.
template <int KW, int KA, int NC>
constexpr bool kSharedK = NC == 2 && KW * KA != 6 && !(KW == 3 && KA == 1);

// `contract` over a stretch of K: halves of 512 positions first, first + 1 (first even) of the `halves` that the vectors have, weights
// packed in operand layout, a word per k-step.  The sums begin at `start`.
template <int KW, int KA, int NC>
__device__ __forceinline__ void contract_part(const uint4 (&araw)[2][KW], const uint4* image, int l16, int l4, int first, int halves,
                                              float start, v4f (&acc)[KW][KA]) {
  constexpr int kAllSteps = NC * kSteps;
#pragma unroll
  for (int i = 0; i < KW; ++i)
#pragma unroll
    for (int j = 0; j < KA; ++j) acc[i][j] = v4f{start, start, start, start};
  const uint4* const my = image + 16 * l4 + first * 4 * 64;
  auto b_operand = [&](int j, int t) { return my[(j * kAllSteps + t) * 64 + (l16 ^ ((l4 << 1) | (((t >> 2) & 1) << 3)))]; };
  auto word = [](const uint4& q, int t) { return (t & 3) == 0 ? q.x : (t & 3) == 1 ? q.y : (t & 3) == 2 ? q.z : q.w; };
  uint4 aop[KW], anx[KW], bop[KA], bnx[KA];
#pragma unroll
  for (int j = 0; j < KA; ++j) bop[j] = b_operand(j, 0);
#pragma unroll
  for (int i = 0; i < KW; ++i) aop[i] = expand4_signed(araw[0][i].x);
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    if (h > 0 && first + h >= halves) break;  // (uniform)
#pragma unroll
    for (int t = 4 * h; t < 4 * h + 4; ++t) {
      if (t + 1 < 8) {
#pragma unroll
        for (int j = 0; j < KA; ++j) bnx[j] = b_operand(j, t + 1);
#pragma unroll
        for (int i = 0; i < KW; ++i) anx[i] = expand4_signed(word(araw[(t + 1) / 4][i], t + 1));
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

// Partial sums from one wave to another through LDS, [piece][lane]: integers of at most 1024 in binary32, so the sums are the same in
// whatever order they are formed.
template <int KW, int KA>
constexpr int kPartPieces = KW * KA;  // pieces of 16 bytes per lane

template <int KW, int KA>
__device__ __forceinline__ void put_part(const v4f (&acc)[KW][KA], float4* part, int lane) {
#pragma unroll
  for (int q = 0; q < KW * KA; ++q) {
    const v4f& v = acc[q / KA][q % KA];
    part[q * 64 + lane] = make_float4(v[0], v[1], v[2], v[3]);
  }
}

template <int KW, int KA>
__device__ __forceinline__ void add_part(v4f (&acc)[KW][KA], const float4* part, int lane) {
#pragma unroll
  for (int q = 0; q < KW * KA; ++q) {
    const float4 v = part[q * 64 + lane];
    acc[q / KA][q % KA] += v4f{v.x, v.y, v.z, v.w};
  }
}

template <int KW>
__device__ __forceinline__ void keep_packed_part(uint4 (&w)[2][KW]) {
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int i = 0; i < KW; ++i) asm volatile("" : "+v"(w[h][i].x), "+v"(w[h][i].y), "+v"(w[h][i].z), "+v"(w[h][i].w));
}

// NC: stretches of 1024 entries of the longer operand block (1 or 2).  Waves 0 .. 3 take the h side, the cell and the
// quantizer, waves 4 .. 7 the x side of the next step.  BOTH: the x waves gather half of the codes as well (both_gather).
template <int KW, int KA, int EPI, int NC, bool BOTH>
__device__ __forceinline__ void seqw_body(const SeqWArgs& a) {
  constexpr int NG = (EPI == kEpiGru) ? 3 : 4;
  constexpr int kImage = KA * NC * kSteps * 64;
  constexpr int NJ = 4 * NC;  // slots per lane of the quantizer
  __shared__ double sh[2 * kExchange<kWBlocks>];
  __shared__ int dead;
  __shared__ uint32_t codes[KA * 32 * NC + KA];            // codes of one entry, then its coefficients
  __shared__ float hout[kTileB][4 * kBlocksPad];           // h_t of the workgroup's units
  __shared__ float4 xsum[2][kWBlocks][64];  // x-side sums of two consecutive steps
  constexpr bool kShared = kSharedK<KW, KA, NC>;
  __shared__ float4 part[kShared ? kWBlocks : 1][kShared ? kPartPieces<KW, KA> * 64 : 1];  // h-side sums over the second half of K
  extern __shared__ __attribute__((aligned(16))) uint4 lds[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const bool xwave = wv >= kWBlocks;
  const int blk = wv & (kWBlocks - 1);            // row block of the workgroup
  uint4* const image = lds + (xwave ? kImage : 0);  // activations of this wave's side
  static_assert(kWBlocks * kTileB * kWTurn <= 2 * kImage, "the pieces that turn the weights borrow the images");
  const int l16 = lane & 15, l4 = lane >> 4;
  const int H = a.H, batch = a.batch, G = gridDim.x, bx = blockIdx.x, tile = blockIdx.y;
  const int b0 = tile * kTileB;
  const int ncols = batch - b0 < kTileB ? batch - b0 : kTileB;
  const int rb = bx * kWBlocks + blk;
  const int unit = rb * 4 + l4;
  const bool uok = unit < H, bok = l16 < ncols;
  const int col = bok ? l16 : ncols - 1;         // this lane's batch entry (clamped)
  const int uc = uok ? unit : 0;
  const bool own = uok && bok && !xwave;
  unsigned* const flag = a.flag;
  const int n = xwave ? a.x.n : H;               // vector length of this wave's side
  const int wq = (n + 127) >> 7;                 // 16-byte pieces per row
  const int piece0 = lane & 7;

  // ---- once: this wave's weights in operand layout (rows through a padded piece of LDS, amq_pair_body.h; four waves
  // at a time), coefficients, state.  Where K is shared: the x waves also take the second stretch of the h side (two halves of
  // 512 positions), and the h waves keep the first.
  uint4 w[NC][KW][2], wh[2][KW];
  {
    int u = rb * 4 + ((lane >> 3) & 3);
    u = u < H ? u : H - 1;
    const char* Wb = reinterpret_cast<const char*>(xwave ? a.x.Wp : a.h.Wp);
    const size_t plane = (size_t)NG * H * wq * 16;
#pragma unroll
    for (int v = 0; v < 2; ++v) {
      int g = 2 * v + (lane >> 5);
      g = g < NG ? g : NG - 1;
#pragma unroll
      for (int ch = 0; ch < NC; ++ch) {
        const int p = 8 * ch + piece0;
        const unsigned off = (unsigned)((g * H + u) * wq + (p < wq ? p : 0)) * 16u;
#pragma unroll
        for (int i = 0; i < KW; ++i) w[ch][i][v] = *reinterpret_cast<const uint4*>(Wb + i * plane + off);
      }
    }
  }
  if (tid == 0) dead = 0;
  float al[4][KW], bs0[4], bs1[4];
  {
    const float* alpha = xwave ? a.x.alpha : a.h.alpha;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int row = (r < NG ? r : NG - 1) * H + uc;
#pragma unroll
      for (int i = 0; i < KW; ++i) al[r][i] = alpha[row * KW + i];
      bs0[r] = a.bias0 ? a.bias0[row] : 0.0f;
      bs1[r] = (EPI == kEpiGru && a.bias1) ? a.bias1[row] : 0.0f;
    }
  }
  const size_t state = (size_t)(b0 + col) * H + uc;
  float h = a.h0[state], c = EPI == kEpiLstm ? a.c0[state] : 0.0f;
  if (own) {
    a.save_h[state] = h;
    if (EPI == kEpiLstm) a.save_c[state] = c;
  }
  const int hhalves = (H + 511) >> 9;          // halves that the h side's vectors have
  const bool shared_k = kShared && hhalves > 2;  // (otherwise the x waves have no part in the h side)
#pragma unroll
  for (int side = 0; side < 2; ++side) {
    if (xwave == (side == 1)) {
      uint4* const mine = lds + blk * (kTileB * kWTurn);
      const int row = 4 * ((lane >> 3) & 3) + (lane >> 5);
      auto turn = [&](uint4 (&t)[2], uint32_t keep) {
#pragma unroll
        for (int v = 0; v < 2; ++v)
          mine[(row + 2 * v) * kWTurn + piece0] = make_uint4(t[v].x & keep, t[v].y & keep, t[v].z & keep, t[v].w & keep);
#pragma unroll
        for (int v = 0; v < 2; ++v) t[v] = mine[l16 * kWTurn + l4 + 4 * v];
      };
#pragma unroll
      for (int ch = 0; ch < NC; ++ch) {
        const uint32_t keep = 8 * ch + piece0 < wq ? 0xffffffffu : 0u;
#pragma unroll
        for (int i = 0; i < KW; ++i) turn(w[ch][i], keep);
      }
      if (side == 0 && kShared) {
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
          for (int i = 0; i < KW; ++i) wh[h][i] = w[0][i][h];
      } else if (side == 1 && shared_k) {
        int u = rb * 4 + ((lane >> 3) & 3);
        u = u < H ? u : H - 1;
        const int wqh = (H + 127) >> 7;
        const size_t plane = (size_t)NG * H * wqh * 16;
#pragma unroll
        for (int i = 0; i < KW; ++i) {
          uint4 t[2];
          const int p = 8 + piece0;
#pragma unroll
          for (int v = 0; v < 2; ++v) {
            int g = 2 * v + (lane >> 5);
            g = g < NG ? g : NG - 1;
            t[v] = *reinterpret_cast<const uint4*>(reinterpret_cast<const char*>(a.h.Wp) + i * plane +
                                                   (unsigned)((g * H + u) * wqh + (p < wqh ? p : 0)) * 16u);
          }
          turn(t, p < wqh ? 0xffffffffu : 0u);
#pragma unroll
          for (int h = 0; h < 2; ++h) wh[h][i] = t[h];
        }
      }
    }
    lds_barrier();
  }

  if (*flag != 0u) return;  // (there was no room)

  // ---- codes of the inputs (x waves), [plane][step * batch + entry][piece]: the tile is KA * NC * 2 requests of 1 KiB
  // (plane, stretch, half of the tile; lane -> entry, 16-byte piece), dealt to the four x waves in turn
  constexpr int kReq = KA * NC * 2;
  constexpr int kPer = (kReq + kWBlocks - 1) / kWBlocks;
  uint4 xw[kPer];
  float beta_next = 0.0f;
  auto request_inputs = [&](int t) {
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
      int idx = blk + q * kWBlocks;
      idx = idx < kReq ? idx : kReq - 1;
      const int v = idx & 1, ch = (idx >> 1) % NC, j = (idx >> 1) / NC;
      int cc = 8 * v + (lane >> 3);
      cc = cc < ncols ? cc : ncols - 1;
      const int p = 8 * ch + piece0;
      const char* src = reinterpret_cast<const char*>(a.x.Xp) + ((size_t)j * a.rows + (size_t)t * batch + b0) * wq * 16;
      xw[q] = *reinterpret_cast<const uint4*>(src + (unsigned)(cc * wq + (p < wq ? p : 0)) * 16u);
    }
    beta_next = a.x.beta[((size_t)t * batch + b0 + col) * KA + (l4 < KA ? l4 : KA - 1)];
  };
  auto expand_inputs = [&]() {
    const int pb = piece0 & 3, th = piece0 >> 2;
    const int swz = (pb << 1) | (th << 3);
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
      int idx = blk + q * kWBlocks;
      idx = idx < kReq ? idx : kReq - 1;
      const int ch = (idx >> 1) % NC;
      const uint32_t keep = 8 * ch + piece0 < wq ? 0xffffffffu : 0u;
      uint4* dst = image + ((idx >> 1) * kSteps + 4 * th) * 64 + 16 * pb + ((8 * (idx & 1) + (lane >> 3)) ^ swz);
      dst[0 * 64] = expand4_signed(xw[q].x & keep);
      dst[1 * 64] = expand4_signed(xw[q].y & keep);
      dst[2 * 64] = expand4_signed(xw[q].z & keep);
      dst[3 * 64] = expand4_signed(xw[q].w & keep);
    }
  };
  // this wave's sums of its row block and tile from its image
  auto sums = [&](float beta, float (&y)[4]) {
    v4f acc[KW][KA];
    float bt[KA];
#pragma unroll
    for (int j = 0; j < KA; ++j) bt[j] = __shfl(beta, 16 * j + l16, kWave);
    if (kShared && !xwave) {
      if constexpr (KW * KA > 4) keep_packed_part(wh);
      contract_part<KW, KA, NC>(wh, image, l16, l4, 0, hhalves, (float)(H - hhalves * 512), acc);
      if (shared_k) {
        lds_barrier();
        add_part<KW, KA>(acc, part[blk], lane);
      }
    } else {
      if constexpr (NC == 1 && KW * KA == 9) {
        // the first half's weights stay expanded, for which there are registers (us per 35 steps when it was introduced, none / these:
        // 1024 units batch 64 227.3 / 224.1, GRU 228.0 / 222.2, 512 units batch 30 191.5 / 185.5)
#pragma unroll
        for (int i = 0; i < KW; ++i) asm volatile("" : "+v"(w[0][i][1].x), "+v"(w[0][i][1].y), "+v"(w[0][i][1].z), "+v"(w[0][i][1].w));
      } else if constexpr (!kExpandedOnce<KW, KA, NC>) {
        keep_packed(w);
      }
      contract<KW, KA, NC>(w, image, l16, l4, n, acc);
    }
    weigh<KW, KA>(acc, al, bt, y);
  };

  // ---- which entries of its tile this workgroup quantizes: spread over the workgroups of the tile
  const int spread = G / ncols;
  const int q_first = spread > 0 ? (bx % spread == 0 ? bx / spread : ncols) : bx;
  const int q_next = spread > 0 ? ncols : G;
  const int wprH = 4 * ((H + 127) >> 7);
  const int nslots = wprH >> 1;
  const int nj = (nslots + kWBlocks - 1) / kWBlocks;
  const int base = blk * nj;
  const size_t hhalf = (size_t)batch * H;
  const int centry = seqw_entry_pairs(KA, wprH);
  const size_t chalf = (size_t)gridDim.y * kTileB * centry;
  int phase = 0;
  // publishing h_t (x waves): thread -> entry and unit
  const int hp_unit = 4 * kWBlocks * bx + (tid & 15), hp_col = (tid >> 4) & 15;
  const bool hp_ok = hp_unit < H && hp_col < ncols;
  const size_t hp_at = (size_t)(b0 + (hp_ok ? hp_col : 0)) * H + (hp_ok ? hp_unit : 0);

  // ---- gathering the codes of a step, by the h waves or (BOTH) half of the tile's entries by either kind: thread -> word of the row
  // and entry; the same bytes land where expand_inputs puts those of the inputs
  constexpr int kWords = 32 * NC;                              // words of a row, padding included
  constexpr int kColsPer = 64 * kWBlocks / kWords;             // entries per request
  constexpr int kColReq = kTileB / kColsPer / (BOTH ? 2 : 1);  // requests per plane
  constexpr int kGather = KA * kColReq;
  const int gt = tid & (64 * kWBlocks - 1);
  const int gw = gt & (kWords - 1), gc = (BOTH && xwave ? kTileB / 2 : 0) + gt / kWords;
  const bool gok = gw < wprH;
  unsigned goff[kColReq];
#pragma unroll
  for (int k = 0; k < kColReq; ++k) {
    const int cc = k * kColsPer + gc;
    goff[k] = (unsigned)((cc < ncols ? cc : ncols - 1) * centry + (gok ? gw : 0)) * 8u;
  }
  const unsigned gboff = (unsigned)(col * centry + KA * wprH + (l4 < KA ? l4 : KA - 1)) * 8u;
  const int gdst = ((gw >> 5) * kSteps + 4 * ((gw >> 4) & 1) + (gw & 3)) * 64 + 16 * ((gw >> 2) & 3);
  const int gswz = (((gw >> 2) & 3) << 1) | (((gw >> 4) & 1) << 3);
  // returns this lane's coefficient (h waves)
  auto gather_codes = [&](int t) {
    const unsigned tag = (unsigned)t + 1u;
    const char* src = reinterpret_cast<const char*>(a.cbuf + (t & 1) * chalf + (size_t)tile * kTileB * centry);
    auto at = [](const char* base, unsigned off) { return reinterpret_cast<const unsigned long long*>(base + off); };
    unsigned long long v[kGather], bv = (unsigned long long)tag << 32;
    unsigned spins = 0;
    for (;;) {
      if (!xwave) bv = get_pair(at(src, gboff));
#pragma unroll
      for (int q = 0; q < kGather; ++q) v[q] = get_pair(at(src + (q / kColReq) * wprH * 8, goff[q % kColReq]));
      bool ready = (unsigned)(bv >> 32) == tag;
#pragma unroll
      for (int q = 0; q < kGather; ++q) ready = ready && (unsigned)(v[q] >> 32) == tag;
      if (__all(ready)) break;
      if (!poll_again(spins, a.limit, flag)) {
        dead = 1;
        break;
      }
    }
#pragma unroll
    for (int q = 0; q < kGather; ++q)
      lds[(q / kColReq) * NC * kSteps * 64 + gdst + ((q % kColReq * kColsPer + gc) ^ gswz)] =
          expand4_signed(gok ? (uint32_t)(v[q] & 0xffffffffull) : 0u);
    return __uint_as_float((unsigned)(bv & 0xffffffffull));
  };

  // ---- x side of step u: its inputs into the image (one barrier before they are used), the sums into xsum
  float xbeta = 0.0f;
  auto stage_inputs = [&](int u) {
    if (u >= a.steps) return;
    expand_inputs();
    xbeta = beta_next;
    if (u + 1 < a.steps) request_inputs(u + 1);
  };
  auto x_side = [&](int u) {
    float y[4];
    sums(xbeta, y);
    xsum[u & 1][blk][lane] = make_float4(y[0], y[1], y[2], y[3]);
  };
  // ---- a step of the x waves and of the h waves, with the same barriers in both; true: somebody waits in vain, so all
  // leave and the piece is done again.  Each kind has its own loop over the steps, so that what only one of them keeps
  // takes no registers in the other.  With one loop for both the forms needed up to 256 registers (W3/A3 on two
  // stretches 32 more, spilled), now 15 to 40 fewer; 240 are allowed (kResidentRegisters), which leaves W3/A3 on two
  // stretches 13 to 47 spilled and four other forms up to 4.
  auto x_step = [&](int t) {
    const unsigned tag = (unsigned)t + 1u;
    stage_inputs(t + 1);
    for (int e = q_first; e < ncols; e += q_next) {
      for (int i = quantize_exchanges<KA>(a.T) + 1; i > 0; --i) lds_barrier();
      if (gt < KA * (wprH + 1))
        put_pair(a.cbuf + (t & 1) * chalf + ((size_t)tile * kTileB + e) * centry + gt, codes[gt], tag);
    }
    lds_barrier();
    // x side of step t + 1, while the codes are under way
    x_side(t + 1);
    if constexpr (BOTH) gather_codes(t);
    lds_barrier();
    const int gone = dead;
    if (shared_k) {
      v4f acc[KW][KA];
      if constexpr (KW * KA > 4) keep_packed_part(wh);
      contract_part<KW, KA, NC>(wh, lds, l16, l4, 2, hhalves, 0.0f, acc);
      put_part<KW, KA>(acc, part[blk], lane);
      lds_barrier();
    }
    lds_barrier();
    // h_t, through LDS: 16 units are one cache line
    if (hp_ok) {
      const float ht = hout[(tid >> 4) & 15][tid & 15];
      if (t + 1 < a.steps) put_pair(a.hbuf + (t & 1) * hhalf + hp_at, __float_as_uint(ht), tag);
      if (a.hs) a.hs[(size_t)t * hhalf + hp_at] = ht;
    }
    return __builtin_amdgcn_readfirstlane(gone) != 0;
  };
  auto h_step = [&](int t) {
    // ---- quantize h_{t-1} of the entries in this workgroup's charge
    if (t > 0 && q_first < ncols) {
      __builtin_amdgcn_s_sleep(kFirstPollFew);
      if (G > kFewWorkgroups) __builtin_amdgcn_s_sleep(kFirstPoll - kFirstPollFew);
    }
    for (int e = q_first; e < ncols; e += q_next) {
      float v[NJ];
      if (t == 0) {
        load_slots<NJ>(a.h0 + (size_t)(b0 + e) * H, H, base, nj, v);
      } else {
        const unsigned long long* src = a.hbuf + ((t - 1) & 1) * hhalf + (size_t)(b0 + e) * H;
        unsigned long long p[NJ];
        unsigned spins = 0;
        for (;;) {
          bool ready = true;
#pragma unroll
          for (int j = 0; j < NJ; ++j) {
            const int idx = (base + j) * 64 + lane;
            p[j] = (unsigned long long)(unsigned)t << 32;
            if (j < nj && idx < H) p[j] = get_pair(src + idx);
          }
#pragma unroll
          for (int j = 0; j < NJ; ++j) ready = ready && (unsigned)(p[j] >> 32) == (unsigned)t;
          if (__all(ready)) break;
          if (!poll_again(spins, a.limit, flag)) {
            dead = 1;
            break;
          }
        }
#pragma unroll
        for (int j = 0; j < NJ; ++j) v[j] = __uint_as_float((unsigned)(p[j] & 0xffffffffull));
      }
      float beta[KA];
      unsigned long long mym[KA];
      with_slots<NJ, true>(nj, [&](auto slots) {
        float w2[slots()];
#pragma unroll
        for (int j = 0; j < slots(); ++j) w2[j] = v[j];
        quantize_core<KA, slots(), kWBlocks, true>(w2, H, base, nj, a.T, beta, mym, sh, phase);
      });
      // through LDS, so that whole cache lines are written at once
      if (lane < nj && base + lane < nslots) {
#pragma unroll
        for (int i = 0; i < KA; ++i)
          reinterpret_cast<unsigned long long*>(codes + i * wprH)[base + lane] = mym[i];
      }
      if (tid == 0) {
#pragma unroll
        for (int i = 0; i < KA; ++i) codes[KA * wprH + i] = __float_as_uint(beta[i]);
      }
      lds_barrier();
    }

    lds_barrier();

    // ---- codes of h_{t-1}
    const float beta = gather_codes(t);
    lds_barrier();
    const int gone = dead;

    // ---- h side and cell
    float y[4];
    sums(beta, y);
    const float4 x4 = xsum[t & 1][blk][lane];
    const float yx[4] = {x4.x, x4.y, x4.z, x4.w};
    cell<EPI>(yx, y, bs0, bs1, h, c);
    hout[l16][4 * blk + l4] = h;
    lds_barrier();
    return __builtin_amdgcn_readfirstlane(gone) != 0;
  };

  if (!xwave) {
    lds_barrier();
    lds_barrier();
    for (int t = 0; t < a.steps; ++t)
      if (h_step(t)) return;
    if (own) {
      a.h0[state] = h;
      if (EPI == kEpiLstm) a.c0[state] = c;
    }
    return;
  }
  request_inputs(0);
  stage_inputs(0);
  lds_barrier();
  x_side(0);
  lds_barrier();  // (the image may be overwritten)
  for (int t = 0; t < a.steps; ++t)
    if (x_step(t)) return;
}

template <int KW, int KA, int EPI, int NC>
__global__ __launch_bounds__(64 * kWWaves, 2) __attribute__((amdgpu_num_vgpr(kResidentRegisters / 2))) void
seqw_kernel(SeqWArgs a) {
  seqw_body<KW, KA, EPI, NC, true>(a);
}
template <int KW, int KA, int EPI>
__global__ __launch_bounds__(64 * kWWaves, 2) __attribute__((amdgpu_num_vgpr(kResidentRegisters / 2))) void
seqw_apart_kernel(SeqWArgs a) {
  seqw_body<KW, KA, EPI, 2, false>(a);
}

// Whether the x waves gather half of the codes.  They do so once their x side is done, which must be before the codes arrive.  The x side
// takes the longer the more planes the weights have and with a fourth half of 512 inputs; the codes come the sooner the shorter the state
// is (slots per lane of the quantizer).  Three such reasons are one too many.  Time of the h waves alone / both, mean (range) of 16 to 70
// kinds of call for each: 1-bit weights 1.035 to 1.043 whatever the lengths (1.00 to 1.08), 1.01 up to 256 units; 2 bits 1.035 (1.00 to
// 1.06), up to 1024 units 1.025, with longer inputs 1.020, both 0.992 (0.95 to 1.04), up to 256 units 0.992 and 0.966; 3 bits 1.017 (0.98 to
// 1.05), up to 1024 units 0.979, with longer inputs 0.982, both 0.949.  us per 35 steps, LSTMs batch 16, inputs of 1536 and 1600: 1200
// units W2/A2 200.4 / 190.8 and 200.5 / 192.6, W3/A3 286.1 / 282.9 and 292.6 / 297.6, 1024 units W2/A3 224.5 / 221.4 and 225.6 / 227.7, W3/A2
// 191.0 / 193.5 and 196.4 / 204.7.  Nine plane products of a GRU with inputs of two stretches are slower with both throughout, 0.95
// (0.92 to 0.99): 1500 units batch 20 278.5 / 283.2; with inputs of 300 273.7 / 269.6.
constexpr bool both_gather(int k_w, int k_a, bool gru, long long I, long long H) {
  if (gru && k_w * k_a == 9 && I > 1024) return false;
  return k_w + (I > 1536) + (H <= 1024) + (H <= 256) <= 3;
}

// Before a launch: room for it (without it the flag is raised at once), no tags.
constexpr unsigned kNoRoom = 2u;  // (any other value but 0: a wait gave up)

__global__ __launch_bounds__(256) void seqw_reset_kernel(unsigned* flag, ResidentClaim claim, unsigned long long* pairs,
                                                         unsigned count) {
  const unsigned t = blockIdx.x * blockDim.x + threadIdx.x, nt = gridDim.x * blockDim.x;
  for (unsigned i = t; i < count; i += nt) pairs[i] = 0ull;
  if (t == 0) *flag = take_resident_share(claim) ? 0u : kNoRoom;
}

// The piece again from the saved state if the launch before gave up: one workgroup per batch entry.
template <int KA>
__global__ __launch_bounds__(64 * kWBlocks) void seqw_recover_kernel(SeqWArgs a, int KW, int gru, ResidentClaim claim, int clear) {
  __shared__ double sh[2 * kExchange<kWBlocks>];
  __shared__ float hcur[2][2048];
  __shared__ uint32_t codes[KA * 64];
  __shared__ float hbeta[KA];
  const unsigned why = *a.flag;
  if (blockIdx.x == 0 && threadIdx.x == 0 && why != kNoRoom) give_resident_share(claim);
  if (why == 0u) return;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int H = a.H, b = blockIdx.x, NG = gru ? 3 : 4;
  const int wprI = 4 * ((a.x.n + 127) >> 7), wprH = 4 * ((H + 127) >> 7);
  const int nslots = wprH >> 1, nj = (nslots + kWBlocks - 1) / kWBlocks, base = wv * nj;
  const long long m = (long long)NG * H;
  int phase = 0;
  for (int u = tid; u < H; u += 64 * kWBlocks) {
    hcur[0][u] = a.save_h[(size_t)b * H + u];
    if (!gru) a.c0[(size_t)b * H + u] = a.save_c[(size_t)b * H + u];
  }
  __syncthreads();
  for (int t = 0; t < a.steps; ++t) {
    const float* hp = hcur[t & 1];
    float w[8], beta[KA];
    unsigned long long mym[KA];
    load_slots<8>(hp, H, base, nj, w);
    quantize_core<KA, 8, kWBlocks, false>(w, H, base, nj, a.T, beta, mym, sh, phase);
#pragma unroll
    for (int i = 0; i < KA; ++i) {
      if (lane < nj && base + lane < nslots) {
        codes[i * 64 + 2 * (base + lane)] = (uint32_t)(mym[i] & 0xffffffffull);
        codes[i * 64 + 2 * (base + lane) + 1] = (uint32_t)(mym[i] >> 32);
      }
      if (tid == 0) hbeta[i] = beta[i];
    }
    __syncthreads();
    const long long row = (long long)t * a.batch + b;
    for (int u = tid; u < H; u += 64 * kWBlocks) {
      float y[2][4] = {};
      for (int s = 0; s < 2; ++s) {
        const BmvBlock& k = s ? a.h : a.x;
        const int wpr = s ? wprH : wprI;
        for (int g = 0; g < NG; ++g) {
          float sum = 0.0f;
          for (int i = 0; i < KW; ++i) {
            const uint32_t* wp = k.Wp + (i * m + (long long)g * H + u) * wpr;
            float inner = 0.0f;
            for (int j = 0; j < KA; ++j) {
              const uint32_t* xp = s ? codes + j * 64 : k.Xp + ((long long)j * a.rows + row) * wpr;
              int differ = 0;
              for (int q = 0; q < wpr; ++q) differ += __popc(wp[q] ^ xp[q]);
              inner = fmaf(s ? hbeta[j] : k.beta[row * KA + j], (float)(k.n - 2 * differ), inner);
            }
            sum = fmaf(k.alpha[((long long)g * H + u) * KW + i], inner, sum);
          }
          y[s][g] = sum;
        }
      }
      float b0[4], b1[4], h = hp[u], c = 0.0f;
      for (int g = 0; g < 4; ++g) {
        b0[g] = (g < NG && a.bias0) ? a.bias0[(long long)g * H + u] : 0.0f;
        b1[g] = (g < NG && gru && a.bias1) ? a.bias1[(long long)g * H + u] : 0.0f;
      }
      const size_t state = (size_t)b * H + u;
      if (gru) {
        cell<kEpiGru>(y[0], y[1], b0, b1, h, c);
      } else {
        c = a.c0[state];
        cell<kEpiLstm>(y[0], y[1], b0, b1, h, c);
        a.c0[state] = c;
      }
      hcur[(t + 1) & 1][u] = h;
      if (a.hs) a.hs[(size_t)t * a.batch * H + state] = h;
    }
    __syncthreads();
  }
  for (int u = tid; u < H; u += 64 * kWBlocks) a.h0[(size_t)b * H + u] = hcur[a.steps & 1][u];
  if (clear && tid == 0) *a.flag = 0u;  // (one workgroup: nobody else reads it)
}

hipError_t launch_recover(const SeqWArgs& a, int k_w, int k_a, int epi, const ResidentClaim& claim, hipStream_t s, int clear = 0) {
  const dim3 grid((unsigned)a.batch), block(64 * kWBlocks);
  const int gru = epi == kEpiGru;
  switch (k_a) {
    case 1: hipLaunchKernelGGL((seqw_recover_kernel<1>), grid, block, 0, s, a, k_w, gru, claim, clear); break;
    case 2: hipLaunchKernelGGL((seqw_recover_kernel<2>), grid, block, 0, s, a, k_w, gru, claim, clear); break;
    default: hipLaunchKernelGGL((seqw_recover_kernel<3>), grid, block, 0, s, a, k_w, gru, claim, clear); break;
  }
  return hipGetLastError();
}

template <int KW, int KA, int EPI, int NC, bool BOTH>
constexpr auto kernel_of() {
  if constexpr (BOTH) return &seqw_kernel<KW, KA, EPI, NC>;
  else return &seqw_apart_kernel<KW, KA, EPI>;
}

// Workgroups of an instantiation that the current device holds at once (asked for once per device).
template <int KW, int KA, int EPI, int NC, bool BOTH>
int resident_grid() {
  static std::atomic<int> known[64];
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return 0;
  const bool tracked = dev >= 0 && dev < 64;
  if (tracked) {
    const int k = known[dev].load(std::memory_order_acquire);
    if (k > 0) return k - 1;
  }
  constexpr size_t lds = seqw_lds<KW, KA, NC>();
  const void* fn = reinterpret_cast<const void*>(kernel_of<KW, KA, EPI, NC, BOTH>());
  int cus = 0, per = 0;
  if (hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess ||
      hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
      hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, fn, 64 * kWWaves, lds) != hipSuccess) {
    (void)hipGetLastError();
    return 0;
  }
  const int fit = per > 0 ? cus : 0;  // (one to a compute unit: what a claim counts on)
  if (tracked) known[dev].store(fit + 1, std::memory_order_release);
  return fit;
}

// launch == nullptr: only asks whether the grid fits
template <int KW, int KA, int EPI, int NC, bool BOTH = true>
hipError_t run_one(const SeqWArgs* launch, dim3 grid, hipStream_t s) {
  const int fit = resident_grid<KW, KA, EPI, NC, BOTH>();
  if ((long long)grid.x * grid.y > fit) return hipErrorInvalidValue;
  if (!launch) return hipSuccess;
  hipLaunchKernelGGL((kernel_of<KW, KA, EPI, NC, BOTH>()), grid, dim3(64 * kWWaves), (seqw_lds<KW, KA, NC>()), s, *launch);
  return hipGetLastError();
}

template <int KW, int KA, int EPI>
hipError_t run_cell(const SeqWArgs* l, dim3 grid, int nc, bool both, hipStream_t s) {
  if (nc == 1) return run_one<KW, KA, EPI, 1>(l, grid, s);
  return both ? run_one<KW, KA, EPI, 2>(l, grid, s) : run_one<KW, KA, EPI, 2, false>(l, grid, s);
}

template <int KW, int KA>
hipError_t run_k(const SeqWArgs* l, dim3 grid, int epi, int nc, bool both, hipStream_t s) {
  return epi == kEpiLstm ? run_cell<KW, KA, kEpiLstm>(l, grid, nc, both, s) : run_cell<KW, KA, kEpiGru>(l, grid, nc, both, s);
}

dim3 seqw_grid(long long H, long long batch) {
  return dim3((unsigned)((H + 4 * kWBlocks - 1) / (4 * kWBlocks)), (unsigned)((batch + kTileB - 1) / kTileB));
}

hipError_t run(const SeqWArgs* l, long long I, long long H, long long batch, int k_w, int k_a, int epi, hipStream_t s) {
  const dim3 grid = seqw_grid(H, batch);
  const int nc = (I > H ? I : H) > 1024 ? 2 : 1;
  const bool both = both_gather(k_w, k_a, epi == kEpiGru, I, H);
  switch (k_w * 4 + k_a) {
    case 4 * 1 + 1: return run_k<1, 1>(l, grid, epi, nc, both, s);
    case 4 * 1 + 2: return run_k<1, 2>(l, grid, epi, nc, both, s);
    case 4 * 1 + 3: return run_k<1, 3>(l, grid, epi, nc, both, s);
    case 4 * 2 + 1: return run_k<2, 1>(l, grid, epi, nc, both, s);
    case 4 * 2 + 2: return run_k<2, 2>(l, grid, epi, nc, both, s);
    case 4 * 2 + 3: return run_k<2, 3>(l, grid, epi, nc, both, s);
    case 4 * 3 + 1: return run_k<3, 1>(l, grid, epi, nc, both, s);
    case 4 * 3 + 2: return run_k<3, 2>(l, grid, epi, nc, both, s);
    case 4 * 3 + 3: return run_k<3, 3>(l, grid, epi, nc, both, s);
  }
  return hipErrorInvalidValue;
}

}  // namespace

SeqWScratch seqw_scratch(void* base, long long H, long long B, int k_a) {
  const long long tiles = (B + kTileB - 1) / kTileB, wpr = 4 * ((H + 127) / 128);
  SeqWScratch w;
  size_t off = 256;
  auto take = [&](size_t bytes) {
    char* p = base ? static_cast<char*>(base) + off : nullptr;
    off += (bytes + 255) & ~size_t(255);
    return p;
  };
  w.flag = static_cast<unsigned*>(base);
  const size_t pairs = off;
  w.hbuf = reinterpret_cast<unsigned long long*>(take(sizeof(unsigned long long) * 2 * (size_t)B * H));
  w.cbuf = reinterpret_cast<unsigned long long*>(
      take(sizeof(unsigned long long) * 2 * (size_t)tiles * kTileB * seqw_entry_pairs(k_a, (int)wpr)));
  w.pair_bytes = off - pairs;
  w.save_h = reinterpret_cast<float*>(take(sizeof(float) * (size_t)B * H));
  w.save_c = reinterpret_cast<float*>(take(sizeof(float) * (size_t)B * H));
  w.bytes = off;
  return w;
}

bool seqw_supported(long long I, long long H, long long B, int k_w, int k_a, int epi, long long steps) {
  if (B < 2 || I <= 0 || H <= 0 || I > 2048 || H > 2048 || k_w < 1 || k_w > 3 || k_a < 1 || k_a > 3) return false;
  if (B > 16 * 256) return false;
  return run(nullptr, I, H, B, k_w, k_a, epi, nullptr) == hipSuccess ||
         seqw_tiles_grid(I, H, B, k_w, k_a, epi, steps) > 0;
}

hipError_t launch_seqw(SeqWArgs a, const SeqWScratch& w, int k_w, int k_a, int epi, hipStream_t s) {
  a.flag = w.flag;
  a.hbuf = w.hbuf;
  a.cbuf = w.cbuf;
  a.save_h = w.save_h;
  a.save_c = w.save_c;
  a.limit = sequence_spin_limit();
  const unsigned pairs = (unsigned)(w.pair_bytes / sizeof(unsigned long long));
  const unsigned blocks = (pairs + 2047) / 2048;
  const bool one = run(nullptr, a.x.n, a.H, a.batch, k_w, k_a, epi, nullptr) == hipSuccess;  // a workgroup per tile fits
  const dim3 grid = seqw_grid(a.H, a.batch);
  const ResidentClaim claim =
      resident_claim(one ? (long long)grid.x * grid.y : seqw_tiles_grid(a.x.n, a.H, a.batch, k_w, k_a, epi, kAnySteps), false);
  std::lock_guard<std::mutex> together(resident_launches());
  hipLaunchKernelGGL(seqw_reset_kernel, dim3(blocks < 512 ? blocks : 512), dim3(256), 0, s, w.flag, claim, w.hbuf, pairs);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const hipError_t ran = one ? run(&a, a.x.n, a.H, a.batch, k_w, k_a, epi, s) : launch_seqw_tiles(a, k_w, k_a, epi, s);
  e = launch_recover(a, k_w, k_a, epi, claim, s);
  return ran != hipSuccess ? ran : e;
}

hipError_t launch_seq_recover(const SeqWArgs& a, int k_w, int k_a, int epi, hipStream_t s) {
  return launch_recover(a, k_w, k_a, epi, ResidentClaim{}, s, a.batch == 1);
}

// ---- shares of the chip (amq_resident.h) ---------------------------------------------------------------------
static __device__ unsigned resident_word;

namespace {

__global__ void hold_shares_kernel(unsigned* word, unsigned shares) {
  __hip_atomic_fetch_add(word, shares, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__global__ void read_shares_kernel(unsigned* word, unsigned* room) {
  *room = __hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

struct ResidentDevice {
  std::atomic<unsigned*> word;
  std::atomic<unsigned> shares;
};

// Address of the word on the current device and the shares the device has, looked up once per device.
ResidentClaim resident_device() {
  static ResidentDevice known[64];
  ResidentClaim c{};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return c;
  const bool tracked = dev >= 0 && dev < 64;
  if (tracked && (c.word = known[dev].word.load(std::memory_order_acquire)) != nullptr) {
    c.shares = known[dev].shares.load(std::memory_order_relaxed);
    return c;
  }
  void* p = nullptr;
  int cus = 0;
  if (hipGetSymbolAddress(&p, HIP_SYMBOL(resident_word)) != hipSuccess ||
      hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) {
    (void)hipGetLastError();
    return c;
  }
  c.shares = cus > kShareGrid ? (unsigned)(cus / kShareGrid) : 1u;
  c.word = static_cast<unsigned*>(p);
  if (tracked) {
    known[dev].shares.store(c.shares, std::memory_order_relaxed);
    known[dev].word.store(c.word, std::memory_order_release);
  }
  return c;
}

}  // namespace

ResidentClaim resident_claim(long long grid, bool light) {
  ResidentClaim c = resident_device();
  const long long need = (grid + kShareGrid - 1) / kShareGrid;
  const unsigned shares = need < (long long)c.shares ? (unsigned)need : c.shares;
  c.mine = light ? shares << 8 : shares;
  // as long as a wait of the kernels may take: 2^19 polls are about 0.2 s
  c.ticks = 40ull * sequence_spin_limit();
  return c;
}

std::mutex& resident_launches() {
  static std::mutex m;
  return m;
}

hipError_t launch_hold_shares(int shares, hipStream_t s) {
  const ResidentClaim c = resident_device();
  if (!c.word) return hipErrorInvalidValue;
  hipLaunchKernelGGL(hold_shares_kernel, dim3(1), dim3(1), 0, s, c.word, (unsigned)shares);
  return hipGetLastError();
}

hipError_t launch_read_shares(unsigned* room, hipStream_t s) {
  const ResidentClaim c = resident_device();
  if (!c.word) return hipErrorInvalidValue;
  hipLaunchKernelGGL(read_shares_kernel, dim3(1), dim3(1), 0, s, c.word, room);
  return hipGetLastError();
}

}  // namespace amq
