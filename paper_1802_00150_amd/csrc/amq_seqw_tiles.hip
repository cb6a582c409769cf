// Recurrent sequences of batches with more tiles than the chip has room for in amq_seqw.hip: one launch per piece as there,
// but a workgroup owns its 4 row blocks for several batch tiles (a group of them), which take turns.
//
// What bounds it: with one tile per workgroup a step is a chain of two exchanges and Alg. 2, 4.4 to 8 us, most of which a workgroup
// waits.  Other tiles' work goes into that wait: a turn costs 2.5 us at 1024 units W2/A2, 4 us at W3/A3 (polled gathers, a trip to
// memory each; the image; products; cell), where two launches per step pay for launches, weights and quantizer each time.  1024 units,
// us per step before / here: batch 128 W2/A2 9.3 / 7.5, W3/A3 11.7 / 10.0; batch 192 12.3 / 9.2, 19.3 / 13.1.
//
// A turn ("slot") is step t of tile i of the group, slots go i first.  In slot s a workgroup
//   1. quantizes h_{t-1} of its entries of later slots' tiles (gather, Alg. 2, publish),
//   2. gathers the codes of the tile of slot s, forms the h-side products, the cell, publishes h_t.
// How far ahead: with three tiles and more one slot, so that what both steps wait for is a slot old when they begin (two slots ahead:
// 1024 units batch 192 14.6 us instead of 9.0, since h_{t-1} is then just being published; batch 256 11.8 against 11.5); with two
// tiles both at the start of the step (one slot ahead: batch 128 9.5 instead of 7.5: either tile's chain would pass through both
// slots); a single tile in its own slot.  In every one of these orders a workgroup waits only for what comes earlier in the order
// for all, so nobody waits in vain; and whoever writes the pairs of step t + 2 of a tile has seen data of its step t + 1 that depend
// on every reader of its step t, so two buffers in turn suffice per tile, as with one.
// The entries of all tiles of a group are dealt evenly to its workgroups.  Cell state is kept in LDS, one float per lane and tile.
// (Asking for the next slot's codes a slot early costs more in registers than it gains: 7.5 -> 8.2, 10.0 -> 11.2; the x side next to the
// h side's products instead of next to the gather: 9.5 -> 10.1 at batch 80 W3/A3.)
//
// The arithmetic and its order, the exchange, the claim of room, the bounded waits and the recovery are those of amq_seqw.hip: the
// results are the same bit for bit.
#include <atomic>

#include "amq_seqw_body.h"

namespace amq {

namespace {

constexpr int kMostTiles = 4;  // tiles of a group

template <int KW, int KA, int EPI, int NC>
__global__ __launch_bounds__(64 * kWWaves, 2) __attribute__((amdgpu_num_vgpr(kResidentRegisters / 2))) void
seqw_tiles_kernel(SeqWArgs a) {
  constexpr int NG = (EPI == kEpiGru) ? 3 : 4;
  constexpr int kImage = KA * NC * kSteps * 64;
  constexpr int NJ = 4 * NC;  // slots per lane of the quantizer
  __shared__ double sh[2 * kExchange<kWBlocks>];
  __shared__ int dead;
  __shared__ uint32_t codes[KA * 32 * NC + KA];  // codes of one entry, then its coefficients
  __shared__ float hout[kTileB][4 * kBlocksPad];  // h_t of the workgroup's units
  __shared__ float4 xsum[2][kWBlocks][64];        // x-side sums of two consecutive slots
  extern __shared__ __attribute__((aligned(16))) uint4 lds[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const bool xwave = wv >= kWBlocks;
  const int blk = wv & (kWBlocks - 1);              // row block of the workgroup
  uint4* const image = lds + (xwave ? kImage : 0);  // activations of this wave's side
  float* const keep_state = reinterpret_cast<float*>(lds + 2 * kImage) + (tid & (64 * kWBlocks - 1));  // c (GRU: h), per tile
  static_assert(kWBlocks * kTileB * kWTurn <= 2 * kImage, "the pieces that turn the weights borrow the images");
  const int l16 = lane & 15, l4 = lane >> 4;
  const int H = a.H, batch = a.batch, G = gridDim.x, bx = blockIdx.x;
  const int all_tiles = (batch + kTileB - 1) / kTileB;
  const int tile0 = (int)((long long)all_tiles * blockIdx.y / gridDim.y);
  const int tiles = (int)((long long)all_tiles * (blockIdx.y + 1) / gridDim.y) - tile0;
  const int first = tile0 * kTileB;                                                     // batch entries of the group
  const int entries = (batch < first + tiles * kTileB ? batch : first + tiles * kTileB) - first;
  auto columns = [&](int i) { return entries - i * kTileB < kTileB ? entries - i * kTileB : kTileB; };
  const int slots = a.steps * tiles;
  // vectors of the first so many slots are quantized before the products of slot s
  auto quantized_by = [&](int s) {
    const int q = tiles > 2 ? s + 2 : tiles == 2 ? (s | 1) + 1 : s + 1;
    return q < slots ? q : slots;
  };
  const int rb = bx * kWBlocks + blk;
  const int unit = rb * 4 + l4;
  const bool uok = unit < H;
  const int uc = uok ? unit : 0;
  unsigned* const flag = a.flag;
  const int n = xwave ? a.x.n : H;  // vector length of this wave's side
  const int wq = (n + 127) >> 7;    // 16-byte pieces per row
  const int piece0 = lane & 7;

  // ---- once: this wave's weights in operand layout (rows through a padded piece of LDS, amq_pair_body.h; four waves
  // at a time), coefficients, state
  uint4 w[NC][KW][2];
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
  if (!xwave) {
    for (int i = 0; i < tiles; ++i) {
      const int cols = columns(i), col = l16 < cols ? l16 : cols - 1;
      const size_t state = (size_t)(first + i * kTileB + col) * H + uc;
      const float h = a.h0[state], c = EPI == kEpiLstm ? a.c0[state] : 0.0f;
      keep_state[i * 64 * kWBlocks] = EPI == kEpiLstm ? c : h;
      if (uok && l16 < cols) {
        a.save_h[state] = h;
        if (EPI == kEpiLstm) a.save_c[state] = c;
      }
    }
  }
#pragma unroll
  for (int side = 0; side < 2; ++side) {
    if (xwave == (side == 1)) {
      uint4* const mine = lds + blk * (kTileB * kWTurn);
      const int row = 4 * ((lane >> 3) & 3) + (lane >> 5);
#pragma unroll
      for (int ch = 0; ch < NC; ++ch) {
        const uint32_t keep = 8 * ch + piece0 < wq ? 0xffffffffu : 0u;
#pragma unroll
        for (int i = 0; i < KW; ++i) {
#pragma unroll
          for (int v = 0; v < 2; ++v) {
            const uint4 t = w[ch][i][v];
            mine[(row + 2 * v) * kWTurn + piece0] = make_uint4(t.x & keep, t.y & keep, t.z & keep, t.w & keep);
          }
#pragma unroll
          for (int v = 0; v < 2; ++v) w[ch][i][v] = mine[l16 * kWTurn + l4 + 4 * v];
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
  int asked = 0, asked_t = 0, asked_i = 0;  // the next slot to ask for
  auto request_inputs = [&]() {
    const int cols = columns(asked_i), b0 = first + asked_i * kTileB;
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
      int idx = blk + q * kWBlocks;
      idx = idx < kReq ? idx : kReq - 1;
      const int v = idx & 1, ch = (idx >> 1) % NC, j = (idx >> 1) / NC;
      int cc = 8 * v + (lane >> 3);
      cc = cc < cols ? cc : cols - 1;
      const int p = 8 * ch + piece0;
      const char* src = reinterpret_cast<const char*>(a.x.Xp) + ((size_t)j * a.rows + (size_t)asked_t * batch + b0) * wq * 16;
      xw[q] = *reinterpret_cast<const uint4*>(src + (unsigned)(cc * wq + (p < wq ? p : 0)) * 16u);
    }
    const int col = l16 < cols ? l16 : cols - 1;
    beta_next = a.x.beta[((size_t)asked_t * batch + b0 + col) * KA + (l4 < KA ? l4 : KA - 1)];
    ++asked;
    if (++asked_i == tiles) {
      asked_i = 0;
      ++asked_t;
    }
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
    if constexpr (!kExpandedOnce<KW, KA, NC>) keep_packed(w);
    contract<KW, KA, NC>(w, image, l16, l4, n, acc);
    weigh<KW, KA>(acc, al, bt, y);
  };

  // ---- entries that this workgroup quantizes: the first of tile i that is its own, and the distance to the next
  const int spread = G / entries;  // 0: more entries than workgroups
  const int q_next = spread > 0 ? kTileB : G;
  auto q_first = [&](int i) {
    if (spread > 0) {
      const int e = bx % spread == 0 ? bx / spread - i * kTileB : -1;
      return e < 0 ? kTileB : e;
    }
    const int e = (bx - i * kTileB) % G;
    return e < 0 ? e + G : e;
  };
  const int wprH = 4 * ((H + 127) >> 7);
  const int nslots = wprH >> 1;
  const int nj = (nslots + kWBlocks - 1) / kWBlocks;
  const int base = blk * nj;
  const size_t hhalf = (size_t)batch * H;
  const int centry = seqw_entry_pairs(KA, wprH);
  const size_t chalf = (size_t)all_tiles * kTileB * centry;
  int phase = 0;

  // ---- gathering the codes of a slot (h waves): thread -> word of the row and entry; the same bytes land where
  // expand_inputs puts those of the inputs
  constexpr int kWords = 32 * NC;                   // words of a row, padding included
  constexpr int kColsPer = 64 * kWBlocks / kWords;  // entries per request
  constexpr int kColReq = kTileB / kColsPer;        // requests per plane
  constexpr int kGather = KA * kColReq;
  const int gt = tid & (64 * kWBlocks - 1);
  const int gw = gt & (kWords - 1), gc = gt / kWords;
  const bool gok = gw < wprH;
  const int gdst = ((gw >> 5) * kSteps + 4 * ((gw >> 4) & 1) + (gw & 3)) * 64 + 16 * ((gw >> 2) & 3);
  const int gswz = (((gw >> 2) & 3) << 1) | (((gw >> 4) & 1) << 3);

  // ---- x waves and h waves have a loop of their own each, with the same barriers in both
  if (xwave) {
    float xbeta = 0.0f;
    auto stage_inputs = [&]() {  // of the slot asked for last; then asks for the next
      expand_inputs();
      xbeta = beta_next;
      if (asked < slots) request_inputs();
    };
    request_inputs();
    int qs = 0, qi = 0;  // the next slot to quantize, its tile
    for (int s = -1; s < slots; ++s) {  // (s = -1: the sums of slot 0, and what is quantized that early)
      const bool more = s + 1 < slots;
      if (more) stage_inputs();
      for (const int upto = quantized_by(s); qs < upto; ++qs) {
        const int cols = columns(qi);
        for (int e = q_first(qi); e < cols; e += q_next)
          for (int k = quantize_exchanges<KA>(a.T) + 1; k > 0; --k) lds_barrier();
        if (++qi == tiles) qi = 0;
      }
      lds_barrier();
      if (more) {  // while the codes are under way
        float y[4];
        sums(xbeta, y);
        xsum[(s + 1) & 1][blk][lane] = make_float4(y[0], y[1], y[2], y[3]);
      }
      lds_barrier();
      const int gone = dead;
      lds_barrier();
      if (__builtin_amdgcn_readfirstlane(gone) != 0) return;
    }
    return;
  }

  int t = 0, i = 0;            // of the slot s
  int qs = 0, qt = 0, qi = 0;  // the next slot to quantize, its step and tile
  for (int s = -1; s < slots; ++s) {
    // ---- quantize h_{qt-1} of the entries in this workgroup's charge
    for (const int upto = quantized_by(s); qs < upto; ++qs) {
      const int cols = columns(qi), b0 = first + qi * kTileB;
      for (int e = q_first(qi); e < cols; e += q_next) {
        float v[NJ];
        if (qt == 0) {
          load_slots<NJ>(a.h0 + (size_t)(b0 + e) * H, H, base, nj, v);
        } else {
          const unsigned long long* src = a.hbuf + ((qt - 1) & 1) * hhalf + (size_t)(b0 + e) * H;
          unsigned long long p[NJ];
          unsigned spins = 0;
          for (;;) {
            bool ready = true;
#pragma unroll
            for (int j = 0; j < NJ; ++j) {
              const int idx = (base + j) * 64 + lane;
              p[j] = (unsigned long long)(unsigned)qt << 32;
              if (j < nj && idx < H) p[j] = get_pair(src + idx);
            }
#pragma unroll
            for (int j = 0; j < NJ; ++j) ready = ready && (unsigned)(p[j] >> 32) == (unsigned)qt;
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
        with_slots<NJ, true>(nj, [&](auto count) {
          float w2[count()];
#pragma unroll
          for (int j = 0; j < count(); ++j) w2[j] = v[j];
          quantize_core<KA, count(), kWBlocks, true>(w2, H, base, nj, a.T, beta, mym, sh, phase);
        });
        // through LDS, so that whole cache lines are written at once
        if (lane < nj && base + lane < nslots) {
#pragma unroll
          for (int k = 0; k < KA; ++k) reinterpret_cast<unsigned long long*>(codes + k * wprH)[base + lane] = mym[k];
        }
        if (tid == 0) {
#pragma unroll
          for (int k = 0; k < KA; ++k) codes[KA * wprH + k] = __float_as_uint(beta[k]);
        }
        lds_barrier();
        if (tid < KA * (wprH + 1)) put_pair(a.cbuf + (qt & 1) * chalf + (size_t)(b0 + e) * centry + tid, codes[tid], (unsigned)qt + 1u);
      }
      if (++qi == tiles) {
        qi = 0;
        ++qt;
      }
    }

    lds_barrier();

    // ---- codes of h_{t-1}
    const unsigned tag = (unsigned)t + 1u;
    const int cols = s < 0 ? 1 : columns(i), b0 = first + i * kTileB;
    const int col = l16 < cols ? l16 : cols - 1;
    float beta = 0.0f;
    if (s >= 0) {
      const char* src = reinterpret_cast<const char*>(a.cbuf + (t & 1) * chalf + (size_t)b0 * centry);
      auto at = [](const char* base, unsigned off) { return reinterpret_cast<const unsigned long long*>(base + off); };
      unsigned goff[kColReq];
#pragma unroll
      for (int k = 0; k < kColReq; ++k) {
        const int cc = k * kColsPer + gc;
        goff[k] = (unsigned)((cc < cols ? cc : cols - 1) * centry + (gok ? gw : 0)) * 8u;
      }
      const unsigned gboff = (unsigned)(col * centry + KA * wprH + (l4 < KA ? l4 : KA - 1)) * 8u;
      unsigned long long v[kGather], bv;
      unsigned spins = 0;
      for (;;) {
        bv = get_pair(at(src, gboff));
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
        image[(q / kColReq) * NC * kSteps * 64 + gdst + ((q % kColReq * kColsPer + gc) ^ gswz)] =
            expand4_signed(gok ? (uint32_t)(v[q] & 0xffffffffull) : 0u);
      beta = __uint_as_float((unsigned)(bv & 0xffffffffull));
    }
    lds_barrier();
    const int gone = dead;

    // ---- h side and cell
    if (s >= 0) {
      float y[4];
      sums(beta, y);
      const float4 x4 = xsum[s & 1][blk][lane];
      const float yx[4] = {x4.x, x4.y, x4.z, x4.w};
      float* const mine = keep_state + i * 64 * kWBlocks;
      float h = 0.0f, c = 0.0f;
      if (EPI == kEpiLstm) c = *mine;
      else h = *mine;
      cell<EPI>(yx, y, bs0, bs1, h, c);
      *mine = EPI == kEpiLstm ? c : h;
      if (uok && l16 < cols) {
        const size_t state = (size_t)(b0 + col) * H + uc;
        if (a.hs) a.hs[(size_t)t * hhalf + state] = h;
        if (t + 1 == a.steps) {
          a.h0[state] = h;
          if (EPI == kEpiLstm) a.c0[state] = c;
        }
      }
      hout[l16][4 * blk + l4] = h;
    }
    // published through LDS as well: 16 units are one cache line
    lds_barrier();
    if (s >= 0) {
      const int at_unit = 4 * kWBlocks * bx + (tid & 15), at_col = (tid >> 4) & 15;  // thread -> entry and unit
      if (t + 1 < a.steps && at_unit < H && at_col < cols)
        put_pair(a.hbuf + (t & 1) * hhalf + (size_t)(b0 + at_col) * H + at_unit, __float_as_uint(hout[at_col][tid & 15]), tag);
      if (++i == tiles) {
        i = 0;
        ++t;
      }
    }
    if (__builtin_amdgcn_readfirstlane(gone) != 0) return;
  }
}

// Compute units that hold a workgroup of an instantiation on the current device (asked for once per device).
template <int KW, int KA, int EPI, int NC>
int units_that_fit() {
  static std::atomic<int> known[64];
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return 0;
  const bool tracked = dev >= 0 && dev < 64;
  if (tracked) {
    const int k = known[dev].load(std::memory_order_acquire);
    if (k > 0) return k - 1;
  }
  constexpr size_t lds = seqw_lds<KW, KA, NC>() + sizeof(float) * kMostTiles * 64 * kWBlocks;
  const void* fn = reinterpret_cast<const void*>(&seqw_tiles_kernel<KW, KA, EPI, NC>);
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

// Steps from which on the tiles of a batch take turns rather than launches each step: the launch costs about 20 us before its first
// step (claim, cleared pairs, weights, what follows it) that the per-step form has not, and saves 1.5 to 6 us per step.  us, per-step
// form / here, W2/A2: 1024 units batch 80 4 steps 38.2 / 41.8, 6 steps 54.3 / 54.7, 8 steps 71.2 / 67.5; 1500 units batch 64 48.1 / 51.2,
// 68.5 / 69.1, 88.6 / 86.3; 512 units batch 200 36.3 / 38.5, 53.6 / 49.6, 70.1 / 60.9; 1024 batch 80 W3/A3 46.6 / 52.1, 67.4 / 69.7,
// 88.2 / 88.9 and 12 steps 130 / 124.
constexpr long long kTiledSteps = 8;

// Where this is ahead of what else such a batch takes (two launches per step, amq_step.hip, amq_mfma32_cell.hip).  us per step, that
// form / here, W2/A2 and W3/A3 (LSTM, 35 steps):
//   2 tiles each: 512 units batch 256 9.3 / 7.0 and 11.3 / 9.2; 650 batch 192 10.2 / 7.4 and 12.8 / 9.9; 1024 batch 128 9.3 / 7.5 and
//   11.7 / 10.0; 1500 batch 64 10.7 / 9.1; 2048 batch 64 11.3 / 10.0
//   3 tiles each: 650 batch 256 12.9 / 11.3 and 21.1 / 15.8; 1024 batch 192 12.3 / 9.2 and 19.3 / 13.1; 1500 batch 96 16.3 / 11.7; 2048
//   batch 96 18.9 / 13.2
//   4 tiles each: 1024 batch 256 12.4 / 11.7 and 19.9 / 16.9; 1500 batch 128 16.6 / 15.2; 2048 batch 128 19.6 / 17.0
// Not: more tiles than that (1500 units batch 192 20.9 / 24.4).  Where workgroups quantize two entries of a step, the price of the second
// is Alg. 2 again: at 4 tiles each that is too much (800 units batch 256 12.9 / 13.7), below 512 units at 3-bit activations also
// (450 units batch 160 W2/A3 9.6 / 10.0), and three entries always.  On two stretches with 3 bits registers run out (spilled: 40 to 97):
// W3/A3 at 1500 units batch 64 14.2 / 16.5, W2/A3 11.9 / 13.2, while W3/A2 (47 to 51 spilled, 148 to 156 bytes per lane) is ahead with 3
// tiles (batch 96 19.7 / 15.7) but not with 2 (2048 units batch 48 LSTM 13.1 / 13.7, GRU 12.7 / 14.1; 12 steps 13.3 / 14.8 and 12.8 / 15.0).
// On one stretch W3/A2 spills 15 registers (64 bytes) and is ahead all the same (1024 units batch 80 9.6 / 8.2, 192 17.2 / 11.1).  Two tiles
// on two stretches are the only ones for which the launch's own cost shows beyond 8 steps (2048 units batch 48, inputs of 300, 8 steps 4 to
// 6 % behind): from 12 on.  And as long as the per-step launch has one round of workgroups for all tiles, two per compute unit and a
// few, three tiles are not ahead either (1500 units batch 80 11.0 / 11.8, 700 batch 176 W3/A3 12.5 / 14.7, 600 batch 208 W2/A3 11.4 /
// 13.4, 740 batch 176 W3/A3, 517 workgroups, 12.4 / 13.8; 606 batch 224, 532, 19.4 / 14.0), save for W2/A2 with one entry of a step per
// workgroup (872 batch 144 8 % ahead).
bool worth_it(int k_w, int k_a, int nc, long long width, long long tiles, long long each, long long steps) {
  const long long entries = each * kTileB;
  if (each > kMostTiles || entries > 2 * width || (each == 4 && entries > width)) return false;
  if (each > 2 && tiles * width <= 520) return nc == 1 && k_w * k_a == 4 && entries <= width;
  if (nc == 1) return k_a == 2 || width >= 32;
  return each == 2 ? k_w == 2 && steps >= 12 : each == 3 || k_w == 2;
}

// launch == nullptr: only asks for the grid (0: not taken)
template <int KW, int KA, int EPI, int NC>
dim3 run_one(const SeqWArgs* launch, long long H, long long batch, long long steps, hipStream_t s) {
  const long long width = (H + 4 * kWBlocks - 1) / (4 * kWBlocks), tiles = (batch + kTileB - 1) / kTileB;
  const long long room = units_that_fit<KW, KA, EPI, NC>() / width;
  if (room == 0) return dim3(0);
  const long long each = (tiles + room - 1) / room;
  if (!worth_it(KW, KA, NC, width, tiles, each, steps)) return dim3(0);
  const dim3 grid((unsigned)width, (unsigned)((tiles + each - 1) / each));
  if (launch)
    hipLaunchKernelGGL((seqw_tiles_kernel<KW, KA, EPI, NC>), grid, dim3(64 * kWWaves),
                       (seqw_lds<KW, KA, NC>() + sizeof(float) * (size_t)each * 64 * kWBlocks), s, *launch);
  return grid;
}

template <int KW, int KA, int EPI>
dim3 run_k(const SeqWArgs* l, long long H, long long batch, long long steps, int nc, hipStream_t s) {
  if (nc == 1) return run_one<KW, KA, EPI, 1>(l, H, batch, steps, s);
  if constexpr (KA == 2) return run_one<KW, KA, EPI, 2>(l, H, batch, steps, s);
  return dim3(0);
}

template <int KW, int KA>
dim3 run_epi(const SeqWArgs* l, long long H, long long batch, long long steps, int epi, int nc, hipStream_t s) {
  return epi == kEpiLstm ? run_k<KW, KA, kEpiLstm>(l, H, batch, steps, nc, s) : run_k<KW, KA, kEpiGru>(l, H, batch, steps, nc, s);
}

dim3 run(const SeqWArgs* l, long long I, long long H, long long batch, int k_w, int k_a, int epi, long long steps, hipStream_t s) {
  const int nc = (I > H ? I : H) > 1024 ? 2 : 1;
  switch (k_w * 4 + k_a) {
    case 4 * 2 + 2: return run_epi<2, 2>(l, H, batch, steps, epi, nc, s);
    case 4 * 2 + 3: return run_epi<2, 3>(l, H, batch, steps, epi, nc, s);
    case 4 * 3 + 2: return run_epi<3, 2>(l, H, batch, steps, epi, nc, s);
    case 4 * 3 + 3: return run_epi<3, 3>(l, H, batch, steps, epi, nc, s);
  }
  return dim3(0);
}

}  // namespace

long long seqw_tiles_grid(long long I, long long H, long long B, int k_w, int k_a, int epi, long long steps) {
  if (steps < kTiledSteps) return 0;
  const dim3 grid = run(nullptr, I, H, B, k_w, k_a, epi, steps, nullptr);
  return (long long)grid.x * grid.y;
}

hipError_t launch_seqw_tiles(const SeqWArgs& a, int k_w, int k_a, int epi, hipStream_t s) {
  if (run(&a, a.x.n, a.H, a.batch, k_w, k_a, epi, kAnySteps, s).x == 0) return hipErrorInvalidValue;
  return hipGetLastError();
}

}  // namespace amq
