// Whole recurrent sequences of one batch entry in one launch, spread over the chip (Eq. 6 over a sequence): LSTM and GRU,
// vectors of up to 2048 entries.
//
// A step at batch 1 is a chain of latencies: h_{t-1} becomes visible to whoever needs it, is quantized (Alg. 2: three or
// four dependent sums over the whole vector), multiplied, and passed through the cell.  The weights stay in registers for
// the whole sequence and every reader quantizes h_{t-1} itself, so that one exchange per step is all there is:
//   - a hidden unit's rows are spread over adjacent lanes (amq_unit_lanes.h), their weights in registers;
//   - h_t is published as 8-byte {value, step tag} pairs, each written with one 64-bit device-scope store; readers poll the
//     pairs they need until all carry the tag of the step, so the data is its own arrival signal.  Two buffers in turn
//     suffice: a buffer is written again by waves that have seen every pair of the step between;
//   - the codes of all inputs are formed (or looked up) before this launch, and the x-side sums of step t + 1 are formed
//     after h_t has been published, while it is under way.
// QW = 1: every wave is on its own -- it polls and quantizes the whole vector (up to 8 slots of 64 entries per lane) and
// multiplies its own rows, with no barrier anywhere in a step.  QW = 4: the four waves of a workgroup quantize together.
// One wave takes longer over the entries and needs no exchange between waves (about 250 cycles less per sum).
//
// Bound: latency -- at 300 units about 0.9 us until h_t is seen, 0.8 for Alg. 2, the rest products, cell and LDS.  Measured, us
// per step in sequences of 35, forms before this kernel -> now, W2/A2: LSTM 300 units 3.50 -> 2.47, 650 4.31 -> 2.93, 1024 5.04 -> 3.08
// (lstm_seqg_kernel), 2048 8.69 -> 3.71; GRU 300 8.06 -> 2.51, 1024 8.09 -> 3.12, 2048 8.50 -> 3.85 (two launches per step);
// W3/A3: LSTM 300 4.22 -> 3.25, 1024 5.79 -> 3.90, 2048 11.0 -> 5.03, GRU 9.23 -> 3.27, 9.61 -> 3.92, 10.3 -> 5.18.
//
// The order of additions is that of the per-step kernels (amq_bmv_body.h); JOINT false: that of lstm_seqg_kernel, which
// sums the two operand blocks of a row apart.
//
// The workgroups are spread over the dies.  All of them on one (up to 28, every eighth of eight times as many), whose own L2 answers
// sooner, was faster alone, 300 units W2/A2 145 -> 125 us per 60 steps, but most compute units of that die are then busy for
// whatever else runs, and everybody waits for the last die: a copy of 256 MiB on another stream 117 -> 143 us (448 units 126 -> 155),
// a 4096 x 4096 bf16 product 163 -> 193, with the sequence beside it 184 -> 212.
//
// Every wait is bounded.  If one gives up a flag is raised and everybody leaves; the caller of this launch follows it with
// one that either computes the piece again from the saved state or takes it back and marks what was derived from it
// (launch_seqg_undo).
#pragma once
#include "amq_launch.h"
#include "amq_quantize_body.h"
#include "amq_unit_lanes.h"

namespace amq {

namespace seq1 {

constexpr int k1Waves = 4;

// How long a wave waits, after the x side of the next step, before it asks for h_t for the first time, in units of 64 cycles: h_t is
// seen elsewhere about 1400 cycles after it was stored, and a poll that finds a part of it costs another trip (about 900).  The x side
// itself takes the longer the more gates and plane products a lane has, so the wait is the rest: 8 or 7, 5, 3 for the four, six and nine
// products of a GRU, 5, 4 or 2, 0 for an LSTM, 0 with two units per lane.  Swept over 0 to 14 units for each form; two more or fewer cost 1 %.
// us per 35 steps, at once / here: LSTM W2/A2 300 units 90.9 / 86.4, 448 97.8 / 90.7, 650 109.3 / 103.0, 1024 112.9 / 107.1, W2/A3 350
// 121.0 / 116.7, W3/A2 350 97.0 / 90.9, GRU W2/A2 300 92.4 / 88.5, 650 109.8 / 105.2, W2/A3 200 110.5 / 106.3, W3/A3 256 113.4 / 109.0.  Four
// waves gain nothing with 3-bit weights in a GRU or 3-bit activations in an LSTM of up to 768 units: at once / with the 5 or 2 units of the
// others W3/A2 650 108.9 / 109.6, 1024 112.3 / 114, W2/A3 650 129.9 / 130.4, 768 129.2 / 130.0; nor do two units per lane: 1500 units W2/A2
// 123.8 / 125.3.  LSTMs of six products and up to 256 units ask at once: with the wait 1 to 2 % faster from 200 units on, but 4 % slower
// below even where it is passed over (W3/A2 112 units 76.5 / 79.4), as the x side then is not formed under the first poll.
constexpr int first_poll(int kw, int ka, bool gru, int qw, int nj, int u) {
  const int planes = kw * ka;
  if (u == 2) return 0;
  if (gru) return planes == 4 ? (qw == 1 ? 8 : 7) : planes == 9 ? 3 : qw == 4 && kw == 3 ? 0 : 5;
  if (planes == 6 && qw == 1 && nj == 4) return 0;
  return planes == 4 ? 5 : planes == 9 ? 0 : ka == 2 ? 4 : qw == 4 && nj == 3 ? 0 : 2;
}

// States longer than this wait.  Shorter ones are a few workgroups that finish close together, and their first poll succeeds: us per 35
// steps, at once / wait / here, LSTM W2/A2 16 units 75.8 / 81.2 / 77.6, 64 80.9 / 84.3 / 80.9, 144 80.5 / 84.1 / 81.1, GRU W2/A2 64 75.5 /
// 79.8 / 73.1, W3/A3 128 105.9 / 105.8 / 102.8; above, at once / here, LSTM 200 units 86.0 / 84.1, GRU 160 91.7 / 87.5.
constexpr int first_poll_from(bool gru) { return gru ? 128 : 192; }

template <int KW, int KA, int EPI, int QW, int NJ, int U, bool JOINT>
__global__ __launch_bounds__(64 * k1Waves, 2) void seq1_kernel(Seq1Args a) {
  constexpr int NG = EPI == kEpiGru ? 3 : 4;
  constexpr int kChunks = 16;
  constexpr int kFirstPoll = first_poll(KW, KA, EPI == kEpiGru, QW, NJ, U);
  __shared__ double sh[2 * kExchange<QW>];
  __shared__ __attribute__((aligned(16))) uint4 hq[QW == 1 ? k1Waves : 2][KA][kChunks];  // codes of h_{t-1}
  __shared__ float hb[2][KA];                                                           // and coefficients (QW = 4)
  __shared__ int dead;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int I = a.I, H = a.H;
  const int cprI = (I + 127) >> 7, cprH = (H + 127) >> 7;
  const UnitLanes l(a.lg, lane);
  const int c = l.c, per = l.per;
  const int unit0 = (blockIdx.x * k1Waves + wv) * U * per + l.uo;
  if (tid == 0) dead = 0;

  // an earlier launch of the same call gave up
  __shared__ unsigned gave_up;
  if (tid == 0) gave_up = __hip_atomic_load(a.sync, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  __syncthreads();
  if (gave_up != 0u) {
    if (tid == 0) seqg_leave(a.sync, a.claim);
    return;
  }

  UnitWeights<KW, U> q;
  load_unit_weights<KW, U, NG>(q, l, unit0, a.Wxp, a.ax, I, a.Whp, a.ah, H);
  const int unit = unit0 + unit_slot<U>(l) * per;
  const bool cell = c == 0 && l.gate < U && unit < H;
  float b0[NG], b1[NG], cst = 0.0f, hlast = 0.0f;
#pragma unroll
  for (int r = 0; r < NG; ++r) {
    b0[r] = (cell && a.bias0) ? a.bias0[r * H + unit] : 0.0f;
    b1[r] = (EPI == kEpiGru && cell && a.bias1) ? a.bias1[r * H + unit] : 0.0f;
  }
  if (cell) {
    hlast = a.h[unit];
    if (EPI == kEpiLstm) cst = a.c[unit];
  }

  const int nslots = (H + 63) >> 6;
  const int nj = (nslots + QW - 1) / QW, base = QW == 1 ? 0 : wv * nj;
  int phase = 0;
  const unsigned limit = a.limit;

  // codes of x_t: this lane's chunk and the coefficients, requested a step ahead
  uint4 xv[KA];
  float xb[KA];
  auto request_x = [&](int t) {
    const uint4* Xp4 = reinterpret_cast<const uint4*>(a.xq);
    const int cc = c < cprI ? c : 0;
#pragma unroll
    for (int j = 0; j < KA; ++j) {
      xv[j] = Xp4[((long long)j * a.steps + t) * cprI + cc];
      xb[j] = a.xbeta[t * KA + j];
    }
  };
  float px[U];  // x-side sums of the step to come: per lane, or (JOINT false) already over the row
  auto x_side = [&]() {
    if (c >= cprI) {
#pragma unroll
      for (int j = 0; j < KA; ++j) xv[j] = make_uint4(0, 0, 0, 0);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      px[u] = unit_dot(q, 0, u, xv, xb);
      if constexpr (!JOINT) px[u] = group_sum(px[u], l.lg);
    }
  };
  request_x(0);
  x_side();
  if (a.steps > 1) request_x(1);

  // (a wave on its own that owns no unit publishes nothing, so nobody would wait for it to have read a buffer)
  const int steps = QW == 1 && (int)(blockIdx.x * k1Waves + wv) * U * per >= H ? 0 : a.steps;
  bool alive = true;
  // (a loop over single units, of a count that the compiler does not see: with one s_sleep of the whole count forms of more than 256 units
  // are up to 2.6 % slower, in the mean 0.2 %)
  const int first_wait = kFirstPoll > 0 && (QW > 1 || NJ > 4 || H > first_poll_from(EPI == kEpiGru)) ? opaque_s(kFirstPoll) : 0;
  for (int t = 0; t < steps; ++t) {
    if (kFirstPoll > 0 && t > 0)
      for (int i = 0; i < first_wait; ++i) __builtin_amdgcn_s_sleep(1);
    // ---- h_{t-1}, published with tag t (the initial state with tag 0, by the launch before)
    float alpha[KA];
    unsigned long long mym[KA];
    float w[NJ];
    {
      const unsigned long long* src = a.hbuf + ((t + 1) & 1) * H;
      unsigned long long p[NJ];
      unsigned spins = 0;
      for (;;) {
        bool ready = true;
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
          const int e = (base + j) * 64 + lane;
          p[j] = __hip_atomic_load(src + (e < H ? e : H - 1), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
#pragma unroll
        for (int j = 0; j < NJ; ++j) ready = ready && (unsigned)(p[j] >> 32) == (unsigned)t;
        if (__all(ready)) break;
        ++spins;
        if (spins >= limit) {
          __hip_atomic_store(a.sync, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          alive = false;
          break;
        }
        if ((spins & 63u) == 0 && __hip_atomic_load(a.sync, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) {
          alive = false;
          break;
        }
      }
#pragma unroll
      for (int j = 0; j < NJ; ++j)
        w[j] = j < nj && (base + j) * 64 + lane < H ? __uint_as_float((unsigned)(p[j] & 0xffffffffull)) : 0.0f;
    }
    if (QW == 1 && !alive) break;
    quantize_core<KA, NJ, QW, true>(w, H, base, nj, a.T, alpha, mym, sh, phase);

    // ---- codes and coefficients to the lanes that multiply
    uint4* const codes = hq[QW == 1 ? wv : t & 1][0];
    if (lane < (base + nj >= nslots ? 2 * cprH - base : nj)) {
#pragma unroll
      for (int j = 0; j < KA; ++j)
        reinterpret_cast<unsigned long long*>(codes + j * kChunks)[base + lane] = mym[j];
    }
    float bt[KA];
    if constexpr (QW == 1) {
      // (LDS serves the accesses of a wave in order)
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
#pragma unroll
      for (int j = 0; j < KA; ++j) bt[j] = alpha[j];
    } else {
      if (tid == 0) {
#pragma unroll
        for (int j = 0; j < KA; ++j) hb[t & 1][j] = alpha[j];
      }
      if (!alive) dead = 1;
      lds_barrier();
      if (__builtin_amdgcn_readfirstlane(dead) != 0) {
        alive = false;
        break;
      }
#pragma unroll
      for (int j = 0; j < KA; ++j) bt[j] = hb[t & 1][j];
    }
    uint4 hv[KA];
#pragma unroll
    for (int j = 0; j < KA; ++j) {
      const uint4 v = codes[j * kChunks + (c < cprH ? c : 0)];
      hv[j] = c < cprH ? v : make_uint4(0, 0, 0, 0);
    }

    float ph[U];
#pragma unroll
    for (int u = 0; u < U; ++u) ph[u] = unit_dot(q, 1, u, hv, bt);
    unit_cell<EPI, U, JOINT, NG>(l, px, ph, b0, b1, hlast, cst);
    if constexpr (kFirstPoll > 0) {
      // the inputs of the next step, asked for a step ago: waited for here and not behind the store, with which loads are counted
#pragma unroll
      for (int j = 0; j < KA; ++j) asm volatile("" : "+v"(xv[j].x), "+v"(xv[j].y), "+v"(xv[j].z), "+v"(xv[j].w), "+v"(xb[j]));
    }
    if (cell) {
      if (t + 1 < a.steps)
        __hip_atomic_store(a.hbuf + (t & 1) * H + unit,
                           ((unsigned long long)(unsigned)(t + 1) << 32) | __float_as_uint(hlast), __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
      if (a.hs) a.hs[(long long)t * H + unit] = hlast;
    }
    // ---- while h_t is under way
    if (t + 1 < a.steps) {
      x_side();
      if constexpr (kFirstPoll > 0) {
#pragma unroll
        for (int u = 0; u < U; ++u) asm volatile("" : "+v"(px[u]));
      }
      if (t + 2 < a.steps) request_x(t + 2);
    }
  }

  if (alive && cell) {
    a.h[unit] = hlast;
    if (EPI == kEpiLstm) a.c[unit] = cst;
  }
  __syncthreads();
  if (tid == 0) seqg_leave(a.sync, a.claim);
}

template <int KW, int KA, int EPI, int QW, int NJ, int U, bool JOINT>
hipError_t run_form(const Seq1Args& a, hipStream_t s) {
  const int units = k1Waves * U * (16 >> a.lg);
  const int grid = (a.H + units - 1) / units;
  if (grid > kSeqGMaxGrid) return hipErrorInvalidValue;
  Seq1Args q = a;
  // Light for the forms of 513 to 1024 units (at most 160 registers), which are the large grids of vectors up to 1024 entries.
  // Measured, 35 steps on 3 / 4 streams, us until all have finished, full / light: 650 units W2/A2 249 / 272 -> 152 / 233, 1024
  // units 264 / 288 -> 232 / 248, W3/A3 251 / 339 -> 212 / 294.  Grids of up to 512 units are one or two shares of eight as they are.
  q.claim = resident_claim(grid, QW == 4 && U == 1);
  std::lock_guard<std::mutex> together(resident_launches());
  hipError_t e = launch_seqg_reset(q.sync, q.hbuf, q.h, q.c, q.save_h, q.save_c, q.H, q.clear_flag, q.claim, s);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((seq1_kernel<KW, KA, EPI, QW, NJ, U, JOINT>), dim3((unsigned)grid), dim3(64 * k1Waves), 0, s, q);
  e = hipGetLastError();
  if (e != hipSuccess) launch_seqg_abandon(q.sync, q.claim, s);
  return e;
}

// How many slots of 64 entries a lane of the quantizing waves holds: as many as H needs, so that no slot is computed for
// nothing.  What the forms between were worth when they were added (no form waited before its first poll then), us per step W2/A2 /
// W3/A3 with the next larger of 4, 6, 8 (one wave), 4 (four waves) or 8 (two units per lane) instead: 300 units LSTM 2.58 -> 2.60 / 3.19 ->
// 3.35, GRU 2.54 -> 2.65 / 3.26 -> 3.47, 448 units 2.71 -> 2.80 / 3.44 -> 3.55, 768 3.12 -> 3.17 / 3.73 -> 3.89, 1200 3.40 -> 3.71 / 4.54 -> 5.08,
// 1500 3.47 -> 3.70 / 4.71 -> 5.11, 1700 3.61 -> 3.73 / 4.85 -> 5.12; 500 units with inputs of 1500 3.07 -> 3.29 / 4.09 -> 4.47.  Up to 512
// units a wave is on its own, beyond four share the work: at 512 units one wave took 2.88 (W2/A2) and
// 3.68 us (W3/A3) per step against 2.97 and 4.24 for four, and at 640 its chain is the longer one.  Vectors above 1024
// entries take 16 lanes per row and gate and two units per lane, so that 2048 units are 256 workgroups; there four waves
// always share the work (fewer forms; 300 units with inputs of 1500: 2.97 against 2.81 us).
template <int KW, int KA, int EPI>
hipError_t run_cell(const Seq1Args& a, hipStream_t s) {
  constexpr bool kApart = EPI == kEpiLstm;  // (short vectors: the order of lstm_seqg_kernel)
  if (a.lg == 4) {
    switch ((a.H + 255) / 256) {
      case 1: case 2: return run_form<KW, KA, EPI, 4, 2, 2, true>(a, s);
      case 3: case 4: return run_form<KW, KA, EPI, 4, 4, 2, true>(a, s);
      case 5: return run_form<KW, KA, EPI, 4, 5, 2, true>(a, s);
      case 6: return run_form<KW, KA, EPI, 4, 6, 2, true>(a, s);
      case 7: return run_form<KW, KA, EPI, 4, 7, 2, true>(a, s);
    }
    return run_form<KW, KA, EPI, 4, 8, 2, true>(a, s);
  }
  switch ((a.H + 63) / 64) {
    case 1: case 2: case 3: case 4: return run_form<KW, KA, EPI, 1, 4, 1, !kApart>(a, s);
    case 5: return run_form<KW, KA, EPI, 1, 5, 1, !kApart>(a, s);
    case 6: return run_form<KW, KA, EPI, 1, 6, 1, !kApart>(a, s);
    case 7: return run_form<KW, KA, EPI, 1, 7, 1, !kApart>(a, s);
    case 8: return run_form<KW, KA, EPI, 1, 8, 1, !kApart>(a, s);
  }
  return a.H <= 768 ? run_form<KW, KA, EPI, 4, 3, 1, !kApart>(a, s) : run_form<KW, KA, EPI, 4, 4, 1, !kApart>(a, s);
}

template <int KW>
hipError_t run_weights(const Seq1Args& a, int k_a, int epi, hipStream_t s) {
  if (k_a == 2) return epi == kEpiGru ? run_cell<KW, 2, kEpiGru>(a, s) : run_cell<KW, 2, kEpiLstm>(a, s);
  return epi == kEpiGru ? run_cell<KW, 3, kEpiGru>(a, s) : run_cell<KW, 3, kEpiLstm>(a, s);
}

}  // namespace seq1

}  // namespace amq
