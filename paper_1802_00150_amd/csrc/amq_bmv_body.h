// Small-batch binary matrix-vector products with the weight planes held in registers and the
// epilogue fused: plain output (streaming GEMV), LSTM cell (Eq. 6) or GRU cell.
//
// Mapping (gfx950, wave64): a weight row of one plane is cpr = wpr/4 16-byte chunks.  A wave
// is split into groups of G = 2^lg lanes (G >= cpr, at most 64); a group owns R = 64/G
// consecutive rows (or hidden units), a lane one chunk.  One wave-wide dwordx4 load therefore
// reads up to 1 KiB of contiguous plane memory.  A wave loads, up front, NSEG row segments
// (gate blocks, or consecutive row groups when streaming) x NBLK operand blocks (x and h) x
// KW planes -- all loads in flight before the first use -- and then loops over the batch with
// the activation planes staged in LDS.  Per batch entry a lane forms the float partial
//   sum_i alpha_i * sum_j beta_j * (bits_in_chunk - 2 * popcount(w_i xor x_j))
// and the G lanes of a group are summed with DPP butterflies (one value per segment instead of
// KW*KA integers).  Lane 0 of the group applies bias / cell nonlinearity and stores.
#pragma once
#include <type_traits>

#include "amq_launch.h"
#include "amq_quantize_body.h"

namespace amq {

// LSE (store mode only): also leave, per batch entry and wave, the (max, sum of exponentials) of
// the outputs the wave produced, for a log-softmax over the rows that follows.
// ONLINE (plain product, one batch entry, one group): the operand is given as a vector (a.raw[0]) that every workgroup
// quantizes for itself while its weights are on the way.  Against a quantizer launch of its own that is about a microsecond
// of arithmetic in every workgroup instead of a launch (2.5 us on the host, 1.6 to 3.4 us between dependent kernels).
template <int KW, int KA, int NSEG, int NBLK, int EPI, bool LSE, bool ONLINE>
__device__ __forceinline__ void bmv_body(const BmvArgs& a, uint4* xs, double* sh, float* bts) {
  static_assert(!ONLINE || (EPI == kEpiStore && NBLK == 1), "steps of one entry: amq_cell1.hip");
  const int lane = lane_id(), wv = wave_id();
  const int lg = a.lg;
  const int G = 1 << lg, R = 64 >> lg;
  const int sub = lane & (G - 1), rloc = lane >> lg;
  const long long wave_global = (long long)blockIdx.x * 4 + wv;
  const long long grp = blockIdx.y;
  const int batch = a.batch;

  int cpr[NBLK], xoff[NBLK], bits[NBLK];
  {
    int off = 0;
#pragma unroll
    for (int k = 0; k < NBLK; ++k) {
      const int n = a.blk[k].n;
      cpr[k] = (n + 127) >> 7;
      xoff[k] = off;
      off += KA * batch * cpr[k];
      const int left = n - 128 * sub;
      bits[k] = left < 0 ? 0 : (left > 128 ? 128 : left);
    }
  }

  // (the vectors to quantize are requested before anything else: the loads return in order)
  constexpr int kRawSlots = ONLINE ? 8 : 1;
  float raw[kRawSlots];
  if constexpr (ONLINE) {
    const int nj = (2 * cpr[0] + 3) >> 2;
    load_slots<kRawSlots>(a.raw[0], a.blk[0].n, __builtin_amdgcn_readfirstlane(wv) * nj, nj, raw);
  }

  // rows of this lane: segment s covers rows seg_base(s) + [0, R)
  const long long nrow = (EPI == kEpiStore) ? a.m : a.H;  // rows per segment space
  long long row[NSEG];
  bool ok[NSEG];
#pragma unroll
  for (int s = 0; s < NSEG; ++s) {
    long long r;
    if (EPI == kEpiStore) {
      r = (wave_global * NSEG + s) * R + rloc;
      ok[s] = r < a.m;
    } else {
      const long long u = wave_global * R + rloc;
      ok[s] = u < a.H;
      r = (long long)s * a.H + u;
    }
    row[s] = ok[s] ? r : 0;
  }

  // weight planes and coefficients first: the longest loads go out before anything waits.  Planes that
  // are read once (more of them than the caches hold) are loaded non-temporal: measured on 512 MiB of
  // planes, 6.3 against 5.95 TB/s for the plain product and 4.95 against 4.63 TB/s for the LSTM step.
  uint4 wq[NBLK][NSEG][KW];
  float al[NBLK][NSEG][KW];
  auto request_weights = [&](auto streaming) {
#pragma unroll
    for (int k = 0; k < NBLK; ++k) {
      const int wpr = cpr[k] * 4;
      const uint32_t* Wp = a.blk[k].Wp + grp * (k ? a.g_Wp1 : a.g_Wp);
      const float* alpha = a.blk[k].alpha + grp * (k ? a.g_alpha1 : a.g_alpha);
#pragma unroll
      for (int s = 0; s < NSEG; ++s)
#pragma unroll
        for (int i = 0; i < KW; ++i) {
          const uint4* src = reinterpret_cast<const uint4*>(Wp + ((long long)i * a.m + row[s]) * wpr) + sub;
          if (sub < cpr[k]) wq[k][s][i] = decltype(streaming)::value ? load_streaming(src) : *src;
          else wq[k][s][i] = make_uint4(0, 0, 0, 0);
          al[k][s][i] = alpha[row[s] * KW + i];
        }
    }
  };
  if (a.streaming) request_weights(std::true_type{});
  else request_weights(std::false_type{});
  // biases of this lane's rows (loop-invariant over the batch)
  float bs0[NSEG], bs1[NSEG];
#pragma unroll
  for (int s = 0; s < NSEG; ++s) {
    bs0[s] = a.bias0 ? a.bias0[row[s]] : 0.0f;
    bs1[s] = (EPI == kEpiGru && a.bias1) ? a.bias1[row[s]] : 0.0f;
  }

  // activation planes of every batch entry into LDS
#pragma unroll
  for (int k = 0; k < NBLK; ++k) {
    if constexpr (ONLINE) {
      int phase = 0;
      const int n = a.blk[0].n, nj = (2 * cpr[0] + 3) >> 2, base = __builtin_amdgcn_readfirstlane(wv) * nj;
      float alpha[KA];
      unsigned long long mym[KA];
      with_slots<kRawSlots, true>(nj, [&](auto slots) {
        float v[slots()];
#pragma unroll
        for (int j = 0; j < slots(); ++j) v[j] = raw[j];
        quantize_core<KA, slots(), 4, true>(v, n, base, nj, a.T, alpha, mym, sh, phase);
      });
#pragma unroll
      for (int i = 0; i < KA; ++i) {
        if (lane < nj && base + lane < 2 * cpr[0])
          reinterpret_cast<unsigned long long*>(xs + i * cpr[0])[base + lane] = mym[i];
        if (threadIdx.x == 0) bts[i] = alpha[i];
      }
      if (a.copy_to && blockIdx.x == 0)
        for (int t = threadIdx.x; t < n; t += 256) a.copy_to[t] = a.raw[0][t];
      continue;
    }
    const int total = KA * batch * cpr[k];
    const uint4* src = reinterpret_cast<const uint4*>(a.blk[k].Xp + grp * (k ? a.g_Xp1 : a.g_Xp));
    for (int t = threadIdx.x; t < total; t += 256) xs[xoff[k] + t] = src[t];
  }
  __syncthreads();
  {
    const long long first = (EPI == kEpiStore) ? wave_global * NSEG * R : wave_global * R;
    if (first >= nrow) return;  // whole wave past the end (after the barrier)
  }

  float* const lse_part = LSE ? a.lse_part : nullptr;  // read once, not per batch entry
  const int lse_slots = a.lse_slots;
  for (int b = 0; b < batch; ++b) {
    // previous state / old output of this batch entry, requested before the popcount work
    float prev[NSEG];
#pragma unroll
    for (int s = 0; s < NSEG; ++s) prev[s] = 0.0f;
    if (sub == 0) {
      if constexpr (EPI == kEpiStore) {
        if (a.accumulate) {
#pragma unroll
          for (int s = 0; s < NSEG; ++s)
            if (ok[s]) prev[s] = a.Y[grp * a.g_Y + (long long)b * a.m + row[s]];
        }
      } else if (ok[0]) {
        prev[0] = (EPI == kEpiLstm) ? a.c_prev[grp * a.g_state + (long long)b * a.H + row[0]]
                                    : a.h_prev[(long long)b * a.H + row[0]];
      }
    }
    float part[NBLK][NSEG];
#pragma unroll
    for (int k = 0; k < NBLK; ++k) {
      uint4 xq[KA];
      float bt[KA];
      const float* beta = a.blk[k].beta + grp * (k ? a.g_beta1 : a.g_beta);
#pragma unroll
      for (int j = 0; j < KA; ++j) {
        xq[j] = (sub < cpr[k]) ? xs[xoff[k] + (j * batch + b) * cpr[k] + sub] : make_uint4(0, 0, 0, 0);
        bt[j] = ONLINE ? bts[j] : beta[b * KA + j];
      }
#pragma unroll
      for (int s = 0; s < NSEG; ++s) {
        float acc = 0.0f;
#pragma unroll
        for (int i = 0; i < KW; ++i) {
          float inner = 0.0f;
#pragma unroll
          for (int j = 0; j < KA; ++j)
            inner = fmaf(bt[j], (float)(bits[k] - 2 * popc4(wq[k][s][i], xq[j])), inner);
          acc = fmaf(al[k][s][i], inner, acc);
        }
        part[k][s] = acc;
      }
    }

    if constexpr (EPI == kEpiStore) {
      float yv[NSEG];
#pragma unroll
      for (int s = 0; s < NSEG; ++s) {
        yv[s] = group_sum(part[0][s], lg) + bs0[s] + prev[s];
        if (sub == 0 && ok[s]) a.Y[grp * a.g_Y + (long long)b * a.m + row[s]] = yv[s];
      }
      if constexpr (LSE) {  // (max, sum of exponentials) over this wave's outputs
        float pm = kLseLow, ps = 0.0f;
#pragma unroll
        for (int s = 0; s < NSEG; ++s)
          if (sub == 0 && ok[s]) pm = fmaxf(pm, yv[s]);
#pragma unroll
        for (int s = 0; s < NSEG; ++s)
          if (sub == 0 && ok[s]) ps += __expf(yv[s] - pm);
        lse_wave_merge(pm, ps);
        if (lane == 0) {
          float* dst = lse_part + ((long long)b * lse_slots + wave_global) * 2;
          dst[0] = pm;
          dst[1] = ps;
        }
      }
    } else if constexpr (EPI == kEpiLstm) {
      float pre[4];
#pragma unroll
      for (int s = 0; s < 4; ++s) pre[s] = group_sum(part[0][s] + part[1][s], lg);
      if (sub == 0 && ok[0]) {
        const long long u = row[0];
#pragma unroll
        for (int s = 0; s < 4; ++s) pre[s] += bs0[s];
        const long long t = grp * a.g_state + (long long)b * a.H + u;
        const float gi = sigmoidf_dev(pre[0]);
        const float gf = sigmoidf_dev(pre[1]);
        const float go = sigmoidf_dev(pre[2]);
        const float gg = tanhf_dev(pre[3]);
        const float c = fmaf(gf, prev[0], gi * gg);
        const float h = go * tanhf_dev(c);
        a.c_out[t] = c;
        a.h_out[t] = h;
        if (a.hs_out) a.hs_out[t] = h;
      }
    } else {  // GRU: segments r, z, n; the candidate keeps its x-side and h-side sums apart
      const float sr = group_sum(part[0][0] + part[1][0], lg);
      const float sz = group_sum(part[0][1] + part[1][1], lg);
      const float nx = group_sum(part[0][2], lg);
      const float nh = group_sum(part[1][2], lg);
      if (sub == 0 && ok[0]) {
        const long long t = (long long)b * a.H + row[0];
        const float r = sigmoidf_dev(sr + bs0[0] + bs1[0]);
        const float z = sigmoidf_dev(sz + bs0[1] + bs1[1]);
        const float nn = tanhf_dev(fmaf(r, nh + bs1[2], nx + bs0[2]));
        a.h_out[t] = fmaf(z, prev[0] - nn, nn);
      }
    }
  }
}

}  // namespace amq
