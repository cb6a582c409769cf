// Large plain binary matrix products on the fp4 matrix cores of gfx950 (Fig. 3 right):
//   Y[b][r] = bias[r] + sum_i alpha[r][i] sum_j beta[b][j] d_ij,   d_ij = inner product of {-1, +1} codes,
// on v_mfma_f32_32x32x64_f8f6f4 with E2M1 codes (exact: every partial sum is a small integer).
//
// Against the 16 x 16 x 128 form this instruction does twice the work on the same operand bytes: half the LDS reads,
// half the weight expansion and half the issue slots per product.  Measured on this chip it occupies the issue port
// for 8 of its 32 cycles on the matrix cores, so about five vector instructions hide behind each; the 16 x 16 form
// leaves room for two, and its kernels were bound by vector instructions and LDS reads.
//
// Work split: a workgroup of 8 waves stages NT * 32 batch columns (all planes, the whole of K) in LDS as operand
// images [tile][plane][k-step][64 lanes x 16 B], once; its waves walk over blocks of 32 rows.  A k-step of 64
// positions is one packed word of each of the two k-blocks of the instruction: lane (row l % 32, k-block l / 32) takes
// the pieces (of 4 words) kb * NP .. kb * NP + NP - 1 of its row, NP = half the pieces of a row, so any vector length
// costs at most one padded piece.  Weight pieces go from memory to registers two pieces ahead of their use and across
// row blocks, and are expanded there, one word per k-step.  Positions past the end of a vector are 0.0 in the staged
// operand, so the weight side needs no masks.
//
// Row coefficients and biases of a row block pass through a private piece of LDS per wave, from which the epilogue
// takes them four rows at a time (C layout: lane = column l % 32, register r = row 8 (r / 4) + 4 (l / 32) + r % 4).
// The linear workgroup index is dealt out so that the workgroups of one XCD work on neighbouring row ranges: each
// XCD's L2 then holds its share of the weights.
//
// Bound: power.  A wave alone in its contraction keeps the matrix cores busy at the 1.5 to 1.8 GHz that the chip then holds; a
// better balance between the two waves of a SIMD (row blocks drawn by ticket: last end 28.8 -> 28.1 us) and fewer vector
// instructions per output (a log-sum-exp without its maximum) change the time by less than 1 %, while the contraction's precedence
// does (below).  Measured (us), int8 or 16 x 16 kernel -> here: 10000 x 1500 W2/A2 at batch 256
// 35.9 -> 13.4, 6144 x 2048 W2/A2 batch 256 29.1 -> 15.6, 20000 x 2048 W3/A3 batch 40 33.9 -> 16.8, 2000 x 512 W2/A2
// batch 1024 11.8 -> 7.3, 10000 x 650 W2/A3 batch 700 22.6 -> 19.1, 10000 x 1024 W2/A3 batch 1024 34.5 -> 32.5.
#pragma once
#include <type_traits>

#include "amq_device.h"
#include "amq_launch.h"

namespace amq {

namespace mfma32 {

constexpr int kWaves = 8;
constexpr int kTileN = 32;             // columns per tile, rows per row block
constexpr int kXcds = 8;
constexpr int kMaxLds = 160 * 1024;

typedef float v16f __attribute__((ext_vector_type(16)));
// Four adjacent outputs of a column, in one request at any multiple of four bytes: the columns of Y begin anywhere when the rows
// are not a multiple of four.  (Requests of 4 bytes instead: 9999 x 1024 W3/A3 batch 700 42.4 against 30.8 us, 42001 x 1024 W2/A3
// batch 128 29.4 against 19.3.)
typedef float Rows4 __attribute__((ext_vector_type(4), aligned(4)));

__device__ __forceinline__ v16f mfma32_fp4(uint4 a, uint4 b, v16f c) {
  return __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(as_operand(a), as_operand(b), c, 4, 4, 0, 0, 0, 0);
}

// Pieces per k-block of a row.  Up to 4 (vectors of at most 1024 entries) the contraction is unrolled over exactly that
// many, 2 at least; longer rows take an even number in a loop over pairs.
constexpr int kStaticPieces = 4;
__host__ __device__ constexpr int half_pieces(int n) {
  const int np = (((n + 127) >> 7) + 1) >> 1;
  return np <= 2 ? 2 : np <= kStaticPieces ? np : (np + 1) / 2 * 2;
}

// LDS: operand images, then per wave 32 x (KW coefficients + bias)
__host__ __device__ constexpr size_t image_bytes(int ka, int nt, int n) { return (size_t)nt * ka * half_pieces(n) * 4 * 1024; }
__host__ __device__ constexpr size_t lds_bytes(int kw, int ka, int nt, int n) {
  return image_bytes(ka, nt, n) + (size_t)kWaves * kTileN * (kw + 1) * sizeof(float);
}

// What a launch leaves: the outputs; the outputs and their partial log-sum-exp; the partial log-sum-exp and one chosen
// output per column.
enum { kOutY = 0, kOutYLse = 1, kOutScore = 2 };

// Where the columns of a (k-block, piece) of the image begin: no two pieces of a row of up to 8 meet in a bank.
template <int NP>
__device__ __forceinline__ int swizzle(int half, int p) {
  return NP > 0 ? 8 * half | (NP == 2 ? 4 : 2) * p : 0;
}

template <int N, int I = 0, typename F>
__device__ __forceinline__ void static_for(F f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    static_for<N, I + 1>(f);
  }
}

// AHEAD: a wave in its contraction has precedence (contraction_first).
template <int KW, int KA, int NT, int NP, int OUT, bool AHEAD>
__global__ __launch_bounds__(64 * kWaves) void mfma32_kernel(BmvArgs a, int rb_per_wg, int rowblocks, int groups,
                                                              int per_xcd) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  asm volatile("" ::AMQ_ARG(a.blk[0].Wp), AMQ_ARG(a.blk[0].alpha), AMQ_ARG(a.blk[0].Xp), AMQ_ARG(a.blk[0].beta),
               AMQ_ARG(a.blk[0].n), AMQ_ARG(a.m), AMQ_ARG(a.batch), AMQ_ARG(a.bias0), AMQ_ARG(a.Y), AMQ_ARG(a.accumulate),
               AMQ_ARG(a.lse_part), AMQ_ARG(rb_per_wg), AMQ_ARG(rowblocks), AMQ_ARG(groups), AMQ_ARG(per_xcd));
  // weight pieces in registers or under way: a whole row block's, or two where those take too many registers
  constexpr int kRing = NP == 0 || (NP == 4 && KW > 2) ? 2 : NP;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, kb = lane >> 5;
  const int task = (blockIdx.x % kXcds) * per_xcd + blockIdx.x / kXcds;
  const int rb_first = (task / groups) * rb_per_wg;
  if (rb_first >= rowblocks) return;  // (the whole workgroup)
  const int bg0 = (task % groups) * (NT * kTileN);
  const int rb_end = min(rb_first + rb_per_wg, rowblocks);
  const int batch = a.batch, m = (int)a.m, n = a.blk[0].n;
  const int wq = (n + 127) >> 7, np = NP > 0 ? NP : half_pieces(n), steps = 4 * np;

  // weight pieces: piece p of row block rb into registers (rows and pieces past the end are clamped: their results
  // are never stored, or meet zeros of the staged operand)
  const uint4* const Wp4 = reinterpret_cast<const uint4*>(a.blk[0].Wp);
  const size_t plane = (size_t)m * wq;
  auto request = [&](int rb, int p, uint4 (&w)[KW]) {
    const int row = (rb < rowblocks ? rb : rowblocks - 1) * kTileN + l32;
    const int g = kb * np + p;
    const uint4* at = Wp4 + (unsigned)((row < m ? row : m - 1) * wq + (g < wq ? g : 0));
#pragma unroll
    for (int i = 0; i < KW; ++i) w[i] = at[i * plane];
  };

  // ---- stage the activation operands.  Rows of up to 8 pieces: item -> (tile, plane, column, piece), pieces adjacent, so that a
  // request takes whole rows, and the weights after the first piece are asked for when every wave has asked for its share of the
  // image.  (Columns adjacent, 16 bytes of 64 rows per request, and all weights behind them: the image is complete 3.3 us after
  // the start, not 2.2; 10000 x 1024 W2/A3 batch 256 13.4 us, not 12.5.)  Column c of (k-block, piece) lies at c ^ swizzle: the
  // writes of 16 lanes then meet all banks, and so do the reads.  Rows of 5 and 6 pieces, which no number of lanes divides into, columns
  // adjacent (10000 x 650 W2/A2 batch 100 5.7 / 6.0, 36000 x 650 W2/A3 batch 40 7.3 / 7.6).
  // Longer rows: columns adjacent, four requests of a thread at a time, the first weight pieces behind them (pieces adjacent:
  // 0 to 8 % slower, 8475 x 2068 W3/A3 batch 99 24.0 / 24.9).
  constexpr bool kWholeRows = NP == 2 || NP == 4;
  uint4 w[kRing][KW];
  {
    const uint4* Xp4 = reinterpret_cast<const uint4*>(a.blk[0].Xp);
    uint4* dst = reinterpret_cast<uint4*>(smem);
    const int items = NT * KA * np * 64;
    constexpr int kBatch = NP > 0 ? (NT * KA * NP * 64 + 64 * kWaves - 1) / (64 * kWaves) : 4;  // (NP > 0: all of them)
    struct Item {
      unsigned tj, col, half, p;
    };
    auto item = [&](unsigned e) {
      Item x;
      if constexpr (kWholeRows) {
        const unsigned q = e / (2u * NP), g = e % (2u * NP);
        x = Item{q / kTileN, q % kTileN, g / NP, g % NP};
      } else {
        const unsigned q = e >> 6;
        x = Item{q / (unsigned)np, e & 31, (e >> 5) & 1, q % (unsigned)np};
      }
      return x;
    };
    for (int e0 = 0; e0 < items; e0 += kBatch * 64 * kWaves) {  // (uniform)
      uint4 xw[kBatch];
#pragma unroll
      for (int v = 0; v < kBatch; ++v) {
        const Item x = item(min(e0 + tid + v * 64 * kWaves, items - 1));
        const int col = bg0 + (int)(x.tj / KA) * kTileN + (int)x.col, g = (int)x.half * np + (int)x.p;
        xw[v] = Xp4[((size_t)(x.tj % KA) * batch + (col < batch ? col : batch - 1)) * wq + (g < wq ? g : 0)];
      }
      if (e0 == 0) {
#pragma unroll
        for (int p = 0; p < (NP > 0 ? 1 : kRing); ++p) request(rb_first + wv, p, w[p]);
      }
#pragma unroll
      for (int v = 0; v < kBatch; ++v) {
        const unsigned e = e0 + tid + v * 64 * kWaves;
        if (e < (unsigned)items) {
          const Item x = item(e);
          const int g = (int)x.half * np + (int)x.p;
          const uint32_t ws[4] = {xw[v].x, xw[v].y, xw[v].z, xw[v].w};
          uint4* d = dst + (x.tj * steps + 4 * x.p) * 64 + 32 * x.half + (x.col ^ swizzle<NP>(x.half, x.p));
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
    }
    if constexpr (NP > 0) {
#pragma unroll
      for (int p = 1; p < kRing; ++p) request(rb_first + wv, p, w[p]);
    }
  }

  int bcol[NT];
  bool bok[NT];
  float btv[NT][KA];
  int tg[NT];
  float* yp[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    bcol[t] = bg0 + t * kTileN + l32;
    bok[t] = bcol[t] < batch;
    const int bc = bok[t] ? bcol[t] : batch - 1;
#pragma unroll
    for (int j = 0; j < KA; ++j) btv[t][j] = a.blk[0].beta[bc * KA + j];
    tg[t] = -1;
    if constexpr (OUT == kOutScore) {
      const long long d = a.tgt[bc];
      if (bok[t] && d >= 0 && d < m) tg[t] = (int)d;
    }
    yp[t] = a.Y + (size_t)bc * m + 4 * kb;
  }
  float lse_m[NT], lse_s[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    lse_m[t] = kLseLow;
    lse_s[t] = 0.0f;
  }
  const uint4* const img = reinterpret_cast<const uint4*>(smem) + 32 * kb;
  float* const mine = reinterpret_cast<float*>(smem + image_bytes(KA, NT, n)) + wv * kTileN * (KW + 1);
  if constexpr (NP > 0) lds_barrier();  // (the weights under way are not waited for)
  else __syncthreads();

  uint4 bop[NT][KA], bnx[NT][KA], aop[KW], anx[KW];
  // column: this lane's place in the piece of the step
  auto fetch = [&](int step, int column, uint4 (&b)[NT][KA]) {
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int j = 0; j < KA; ++j) b[t][j] = img[((t * KA + j) * steps + step) * 64 + column];
  };
  auto expand = [&](const uint4 (&from)[KW], int word, uint4 (&to)[KW]) {
#pragma unroll
    for (int i = 0; i < KW; ++i)
      to[i] = expand4_signed(word == 0 ? from[i].x : word == 1 ? from[i].y : word == 2 ? from[i].z : from[i].w);
  };
  fetch(0, l32 ^ swizzle<NP>(kb, 0), bop);
  expand(w[0], 0, aop);

  for (int rb = rb_first + wv; rb < rb_end; rb += kWaves) {
    // row coefficients and biases of this row block
    float coef_req[(KW + 1) / 2], bias_req;
    {
      const int c0 = rb * kTileN * KW;
#pragma unroll
      for (int v = 0; v < (KW + 1) / 2; ++v) {
        const int ci = c0 + v * 64 + lane;
        coef_req[v] = a.blk[0].alpha[ci < m * KW ? ci : m * KW - 1];
      }
      const int bi = rb * kTileN + l32;
      bias_req = a.bias0 ? a.bias0[bi < m ? bi : m - 1] : 0.0f;
    }

    if constexpr (AHEAD) __builtin_amdgcn_s_setprio(2);
    v16f acc[NT][KW][KA];
    // k-step s of the piece in `cur` (the piece after it in `nxt`): the operands of the following step are fetched (from
    // `column` of its piece) and expanded under the matrix instructions
    auto step = [&](int index, int column, auto s_c, const uint4 (&cur)[KW], const uint4 (&nxt)[KW], auto first_c) {
      constexpr int s = decltype(s_c)::value;
      constexpr bool FIRST = decltype(first_c)::value;
      fetch(index + 1 == steps ? 0 : index + 1, column, bnx);
      if constexpr (s < 3) expand(cur, s + 1, anx); else expand(nxt, 0, anx);
#pragma unroll
      for (int i = 0; i < KW; ++i)
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
          for (int j = 0; j < KA; ++j)
            acc[t][i][j] = mfma32_fp4(aop[i], bop[t][j], FIRST ? v16f{} : acc[t][i][j]);
      constexpr int kValu = (7 * KW + NT * KW * KA - 1) / (NT * KW * KA);
      __builtin_amdgcn_sched_group_barrier(0x100, NT * KA, 0);
#pragma unroll
      for (int g = 0; g < NT * KW * KA; ++g) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x002, kValu, 0);
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int j = 0; j < KA; ++j) bop[t][j] = bnx[t][j];
#pragma unroll
      for (int i = 0; i < KW; ++i) aop[i] = anx[i];
    };
    auto piece = [&](int p, const uint4 (&cur)[KW], const uint4 (&nxt)[KW], auto first_c) {
      const int here = l32 ^ swizzle<NP>(kb, p), there = l32 ^ swizzle<NP>(kb, p + 1 == np ? 0 : p + 1);
      step(4 * p, here, std::integral_constant<int, 0>{}, cur, nxt, first_c);
      step(4 * p + 1, here, std::integral_constant<int, 1>{}, cur, nxt, std::false_type{});
      step(4 * p + 2, here, std::integral_constant<int, 2>{}, cur, nxt, std::false_type{});
      step(4 * p + 3, there, std::integral_constant<int, 3>{}, cur, nxt, std::false_type{});
    };
    // a ring slot is asked for its next piece as soon as it has been used up
    if constexpr (NP > 0) {
      static_for<NP>([&](auto p_c) {
        constexpr int p = decltype(p_c)::value;
        if constexpr (p == 0) piece(0, w[0], w[1], std::true_type{});
        else piece(p, w[p % kRing], w[(p + 1) % kRing], std::false_type{});
        request(p + kRing < NP ? rb : rb + kWaves, p + kRing < NP ? p + kRing : p + kRing - NP, w[p % kRing]);
      });
    } else {
#pragma unroll
      for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int i = 0; i < KW; ++i)
#pragma unroll
          for (int j = 0; j < KA; ++j) acc[t][i][j] = v16f{};
      for (int p = 0; p < np; p += 2) {
        const bool more = p + 2 < np;
        piece(p, w[0], w[1], std::false_type{});
        request(more ? rb : rb + kWaves, more ? p + 2 : 0, w[0]);
        piece(p + 1, w[1], w[0], std::false_type{});
        request(more ? rb : rb + kWaves, more ? p + 3 : 1, w[1]);
      }
    }
    // (pinned in uniform control flow: the compiler takes a matrix instruction for lane-local and would sink it under
    // the store predicates)
    settle_accumulators<32>();
    if constexpr (AHEAD) __builtin_amdgcn_s_setprio(0);
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int i = 0; i < KW; ++i)
#pragma unroll
        for (int j = 0; j < KA; ++j) asm volatile("" : "+v"(acc[t][i][j]));

    // ---- epilogue: coefficients to the wave's piece of LDS as [plane][row], then four rows at a time
#pragma unroll
    for (int v = 0; v < (KW + 1) / 2; ++v) {
      const int e = v * 64 + lane;
      if (KW % 2 == 0 || e < kTileN * KW) mine[(e % KW) * kTileN + e / KW] = coef_req[v];
    }
    if (lane < kTileN) mine[KW * kTileN + lane] = bias_req;
    const bool whole = (rb + 1) * kTileN <= m;  // (uniform)
    const int row0 = rb * kTileN + 4 * kb;      // this lane's rows: row0 + 8 q + 0..3
    float yv[NT][16];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      float4 al[KW];
#pragma unroll
      for (int i = 0; i < KW; ++i) al[i] = *reinterpret_cast<const float4*>(&mine[i * kTileN + 8 * q + 4 * kb]);
      const float4 bs = *reinterpret_cast<const float4*>(&mine[KW * kTileN + 8 * q + 4 * kb]);
#pragma unroll
      for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          float y = 0.0f;
#pragma unroll
          for (int i = 0; i < KW; ++i) {
            float inner = 0.0f;
#pragma unroll
            for (int j = 0; j < KA; ++j) inner = j == 0 ? btv[t][j] * acc[t][i][j][4 * q + r] : fmaf(btv[t][j], acc[t][i][j][4 * q + r], inner);
            const float al_r = r == 0 ? al[i].x : r == 1 ? al[i].y : r == 2 ? al[i].z : al[i].w;
            y = i == 0 ? al_r * inner : fmaf(al_r, inner, y);
          }
          yv[t][4 * q + r] = y + (r == 0 ? bs.x : r == 1 ? bs.y : r == 2 ? bs.z : bs.w);
        }
    }
    if constexpr (OUT == kOutScore) {
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        const int d = tg[t] - row0;
        if (d >= 0 && d < 32 && (d & 4) == 0) {
          float yt = 0.0f;
#pragma unroll
          for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int r = 0; r < 4; ++r) yt = (d == 8 * q + r) ? yv[t][4 * q + r] : yt;
          a.tgt_out[bcol[t]] = yt;
        }
      }
    } else {
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        float* y = yp[t] + (size_t)rb * kTileN;
        if (whole && !a.accumulate) {
          if (bok[t]) {
#pragma unroll
            for (int q = 0; q < 4; ++q)
              *reinterpret_cast<Rows4*>(y + 8 * q) = Rows4{yv[t][4 * q], yv[t][4 * q + 1], yv[t][4 * q + 2], yv[t][4 * q + 3]};
          }
        } else if (bok[t]) {
#pragma unroll
          for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int r = 0; r < 4; ++r)
              if (row0 + 8 * q + r < m) {
                if (a.accumulate) yv[t][4 * q + r] += y[8 * q + r];
                y[8 * q + r] = yv[t][4 * q + r];
              }
        }
      }
    }
    if constexpr (OUT != kOutY) {  // fold this row block's outputs into the running (max, sum)
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        if (!whole) {
#pragma unroll
          for (int e = 0; e < 16; ++e)
            if (row0 + 8 * (e >> 2) + (e & 3) >= m) yv[t][e] = kLseLow;
        }
        float mx = lse_m[t];
#pragma unroll
        for (int e = 0; e < 16; ++e) mx = fmaxf(mx, yv[t][e]);
        float sm = lse_s[t] * __expf(lse_m[t] - mx);
#pragma unroll
        for (int e = 0; e < 16; ++e) sm += __expf(yv[t][e] - mx);
        lse_m[t] = mx;
        lse_s[t] = sm;
      }
    }
  }

  if constexpr (OUT != kOutY) {
    // one slot per workgroup and batch column: the two k-block halves of a wave, then the eight waves through LDS
    float2* xch = reinterpret_cast<float2*>(smem);  // [wave][tile][column]
    __syncthreads();
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      const float m2 = __shfl_xor(lse_m[t], 32, kWave), s2 = __shfl_xor(lse_s[t], 32, kWave);
      lse_merge(lse_m[t], lse_s[t], m2, s2);
      if (kb == 0) xch[(wv * NT + t) * kTileN + l32] = make_float2(lse_m[t], lse_s[t]);
    }
    __syncthreads();
    if (tid < NT * kTileN) {
      const int b = bg0 + tid;
      float mm = kLseLow, ss = 0.0f;
#pragma unroll
      for (int v = 0; v < kWaves; ++v) {
        const float2 p = xch[v * NT * kTileN + tid];
        lse_merge(mm, ss, p.x, p.y);
      }
      if (b < batch) {
        float* dst = a.lse_part + ((long long)b * a.lse_slots + task / groups) * 2;
        dst[0] = mm;
        dst[1] = ss;
      }
    }
  }
}

// Tiles of 32 columns per wave: two where the accumulators (16 registers per plane pair and tile) stay within 128
// and the columns fill them.
constexpr int max_tiles(int kw, int ka) { return kw * ka <= 4 ? 2 : 1; }

// Row blocks of a workgroup: about one workgroup per compute unit.
inline int blocks_each(int rowblocks, int groups) {
  const int splits = groups < 256 ? 256 / groups : 1;
  return (rowblocks + splits - 1) / splits;
}

// Whether, of the two waves of a SIMD, the one in its contraction goes first.  By age, a wave in its epilogue keeps the matrix cores
// from the younger one: 42000 x 1024 W2/A2 batch 2240 scored 146 -> 136 us, 25433 x 445 W3/A3 batch 959 54.7 -> 51.8, 36000 x 589 W2/A3
// batch 70 10.5 -> 9.8 (rows of more than 1024 entries +-2 %, left alone).  Not where a SIMD has three row blocks, two of them the older
// wave's, which age serves better (10000 x 300 W3/A2 batch 256 7.44 / 7.68; from 769 entries on no difference), nor with short rows and
// one tile per wave where half of the SIMDs have five (20000 x 250 W2/A2 batch 200 8.41 / 8.75, but two tiles, batch 256, 13.3 / 12.8).
inline bool contraction_first(int np, int nt, int per) {
  const int of_simd = (per + 3) / 4;
  return np > 0 && !(np < 4 && of_simd == 3) && !(np == 2 && nt == 1 && of_simd == 5 && per <= 18);
}

template <int KW, int KA, int NT, int NP, int OUT>
hipError_t launch_form(BmvArgs a, hipStream_t s, int* lse_slots) {
  const int rowblocks = (int)((a.m + kTileN - 1) / kTileN);
  const int groups = (a.batch + NT * kTileN - 1) / (NT * kTileN);
  // The row blocks are dealt out evenly: a SIMD's two waves take blocks s, s + 4, s + 8 ..
  // of the workgroup, so what counts is the quarter of `per` rounded up, and that is least for the smallest `per` that fits.
  // (Multiples of the 8 waves instead left compute units idle: 10000 x 1024 W2/A3 batch 256 13.3 against 10.8 us, 42000 x
  // 1024 W3/A3 batch 64 15.5 / 13.0, 10000 x 1500 W2/A3 batch 256 16.1 / 13.9, 10000 x 650 W3/A3 batch 256 12.9 / 10.6;
  // no difference from about 16 blocks per wave on.  Among counts of the same quarter the smallest is ahead by 1 to 4 % below 16
  // blocks, fewer workgroups to stage the image by 0 to 2 % above, at nine plane products, and neither by more than the power
  // that the neighbours leave: 619 sizes of nine products with multiples of 4 from 16 blocks on 0.999 of their time.)
  const int per = blocks_each(rowblocks, groups);
  const int splits = (rowblocks + per - 1) / per;
  const int per_xcd = (splits * groups + kXcds - 1) / kXcds;
  const size_t lds = lds_bytes(KW, KA, NT, a.blk[0].n);
  const bool first = contraction_first(NP, NT, per);
  auto* kernel = &mfma32_kernel<KW, KA, NT, NP, OUT, false>;
  if constexpr (NP > 0) {
    if (first) kernel = &mfma32_kernel<KW, KA, NT, NP, OUT, true>;
  }
  static std::atomic<unsigned long long> configured[2] = {{0}, {0}};
  hipError_t e = ensure_dynamic_lds(reinterpret_cast<const void*>(kernel), kMaxLds, configured[first]);
  if (e != hipSuccess) return e;
  if (OUT != kOutY) {
    a.lse_slots = splits;
    if (lse_slots) *lse_slots = splits;
  }
  hipLaunchKernelGGL(kernel, dim3((unsigned)(per_xcd * kXcds)), dim3(64 * kWaves), lds, s, a, per, rowblocks, groups, per_xcd);
  return hipGetLastError();
}

template <int KW, int KA, int NT, int NP>
hipError_t launch_out(const BmvArgs& a, hipStream_t s, int* lse_slots) {
  // (at most 256 row ranges per column, so the caller's room for the partial log-sum-exp is never short of them)
  if (!a.lse_part || a.lse_cap < 256) return launch_form<KW, KA, NT, NP, kOutY>(a, s, lse_slots);
  if (a.Y) return launch_form<KW, KA, NT, NP, kOutYLse>(a, s, lse_slots);
  return launch_form<KW, KA, NT, NP, kOutScore>(a, s, lse_slots);
}

template <int KW, int KA, int NT>
hipError_t launch_one(const BmvArgs& a, hipStream_t s, int* lse_slots) {
  if constexpr (NT > max_tiles(KW, KA)) {
    return hipErrorInvalidValue;
  } else {
    switch (half_pieces(a.blk[0].n)) {
      case 2: return launch_out<KW, KA, NT, 2>(a, s, lse_slots);
      case 3: return launch_out<KW, KA, NT, 3>(a, s, lse_slots);
      case 4: return launch_out<KW, KA, NT, 4>(a, s, lse_slots);
    }
    return launch_out<KW, KA, NT, 0>(a, s, lse_slots);
  }
}

inline int tiles_for(const BmvArgs& a, int k_w, int k_a) {
  if (max_tiles(k_w, k_a) < 2 || a.batch <= kTileN || lds_bytes(k_w, k_a, 2, a.blk[0].n) > kMaxLds) return 1;
  return ((a.batch + kTileN - 1) / kTileN) % 2 == 0 || a.batch > 8 * kTileN ? 2 : 1;
}

template <int KW, int KA>
hipError_t launch_tiles(const BmvArgs& a, hipStream_t s, int* lse_slots) {
  return tiles_for(a, KW, KA) == 2 ? launch_one<KW, KA, 2>(a, s, lse_slots) : launch_one<KW, KA, 1>(a, s, lse_slots);
}


}  // namespace mfma32

}  // namespace amq
