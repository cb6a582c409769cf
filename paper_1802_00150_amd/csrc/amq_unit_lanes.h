// One batch entry's products and cell with a hidden unit's rows spread over adjacent lanes, shared by the one-launch recurrence
// (amq_seq1_body.h) and the single step (amq_cell1.hip).
//
// lane = (hidden unit, gate, 16-byte chunk of the row): Gl = 2^lg lanes per row (at least its chunks), 4 * Gl per unit,
// 16 / Gl units of a wave side by side; a lane holds the KW plane chunks of both operand blocks of U units, `per` apart.
// Against a lane per chunk that holds all gates (amq_bmv_body.h) a unit's weights come through four times as many lanes, so
// that they are spread over four times as many compute units.
#pragma once
#include "amq_device.h"
#include "amq_launch.h"

namespace amq {

struct UnitLanes {
  int lg, c, gate, first, per, uo;
  __device__ __forceinline__ UnitLanes(int log_lanes, int lane)
      : lg(log_lanes), c(lane & ((1 << log_lanes) - 1)), gate((lane >> log_lanes) & 3), first(lane & ~((4 << log_lanes) - 1)),
        per(16 >> log_lanes), uo(lane >> (log_lanes + 2)) {}
};

// This lane's plane chunks and coefficients of both blocks, and how many entries its chunk has (0: none of its business).
template <int KW, int U>
struct UnitWeights {
  uint4 w[2][U][KW];
  float al[2][U][KW];
  float bits[2][U];
};
template <int KW, int U, int NG>
__device__ __forceinline__ void load_unit_weights(UnitWeights<KW, U>& q, const UnitLanes& l, int unit0, const uint32_t* Wxp,
                                                  const float* ax, int I, const uint32_t* Whp, const float* ah, int H) {
  const int g = l.gate < NG ? l.gate : NG - 1;
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    const uint4* Wp4 = reinterpret_cast<const uint4*>(k ? Whp : Wxp);
    const float* alpha = k ? ah : ax;
    const int n = k ? H : I, cpr = (n + 127) >> 7, left = n - 128 * l.c;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int unit = unit0 + u * l.per;
      const bool ok = unit < H && l.c < cpr && l.gate < NG;
      const int row = g * H + (unit < H ? unit : 0);
#pragma unroll
      for (int i = 0; i < KW; ++i) {
        const uint4 t = Wp4[((long long)i * NG * H + row) * cpr + (l.c < cpr ? l.c : 0)];
        q.w[k][u][i] = ok ? t : make_uint4(0, 0, 0, 0);
        q.al[k][u][i] = alpha[row * KW + i];
      }
      q.bits[k][u] = ok ? (float)(left > 128 ? 128 : left) : 0.0f;
    }
  }
}

// sum_i alpha_i sum_j beta_j (inner product of the chunk's codes)
template <int KW, int KA, int U>
__device__ __forceinline__ float unit_dot(const UnitWeights<KW, U>& q, int k, int u, const uint4 (&v)[KA], const float (&bt)[KA]) {
  float acc = 0.0f;
#pragma unroll
  for (int i = 0; i < KW; ++i) {
    float inner = 0.0f;
#pragma unroll
    for (int j = 0; j < KA; ++j) inner = fmaf(bt[j], q.bits[k][u] - 2.0f * (float)popc4(q.w[k][u][i], v[j]), inner);
    acc = fmaf(q.al[k][u][i], inner, acc);
  }
  return acc;
}

// The slot whose cell this lane applies (its chunk 0 lanes: gate u takes slot u).
template <int U>
__device__ __forceinline__ int unit_slot(const UnitLanes& l) { return U == 1 ? 0 : l.gate & (U - 1); }

// From the lanes' shares px (x side; with JOINT false already the sum over the row) and ph to the new state of the unit this
// lane applies the cell of: sums over the chunks of a row, the four gates handed together, Eq. 6 or the GRU cell.  The order
// of additions is that of amq_bmv_body.h; JOINT false: that of lstm_seqg_kernel, which sums the operand blocks apart.
template <int EPI, int U, bool JOINT, int NG>
__device__ __forceinline__ void unit_cell(const UnitLanes& l, const float (&px)[U], const float (&ph)[U], const float (&b0)[NG],
                                          const float (&b1)[NG], float& h, float& c) {
  float y[U], yh[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    if constexpr (EPI == kEpiGru) {  // (candidate: its h side in yh, its x side in y)
      y[u] = group_sum(l.gate == 2 ? px[u] : px[u] + ph[u], l.lg);
      yh[u] = group_sum(ph[u], l.lg);
    } else if constexpr (JOINT) {
      y[u] = group_sum(px[u] + ph[u], l.lg);
    } else {
      y[u] = px[u] + group_sum(ph[u], l.lg);
    }
  }
  const int mine = unit_slot<U>(l);
  auto of_gate = [&](const float (&v)[U], int r) {
    float s = __shfl(v[0], l.first + (r << l.lg), kWave);
#pragma unroll
    for (int u = 1; u < U; ++u) {
      const float o = __shfl(v[u], l.first + (r << l.lg), kWave);
      s = mine == u ? o : s;
    }
    return s;
  };
  if constexpr (EPI == kEpiLstm) {
    const float gi = sigmoidf_dev(of_gate(y, 0) + b0[0]);
    const float gf = sigmoidf_dev(of_gate(y, 1) + b0[1]);
    const float go = sigmoidf_dev(of_gate(y, 2) + b0[2]);
    const float gg = tanhf_dev(of_gate(y, 3) + b0[3]);
    c = fmaf(gf, c, gi * gg);
    h = go * tanhf_dev(c);
  } else {
    const float r = sigmoidf_dev(of_gate(y, 0) + b0[0] + b1[0]);
    const float z = sigmoidf_dev(of_gate(y, 1) + b0[1] + b1[1]);
    const float nn = tanhf_dev(fmaf(r, of_gate(yh, 2) + b1[2], of_gate(y, 2) + b0[2]));
    h = fmaf(z, h - nn, nn);
  }
}

}  // namespace amq
