// Device-side core of the alternating multi-bit quantizer (Alg. 2), shared by the stand-alone quantizer
// kernels, the front kernel of the split recurrent step and the persistent recurrent kernel.  gfx950,
// 64-wide wavefronts.
//
// Element layout in a wave: "slot" j of a lane holds entry (slot_base + j) * 64 + lane, so a wave-wide
// comparison is, as a 64-bit mask, exactly two packed code words of the exchange format.
//
// Precision: stored quantities are binary32; the reductions (sum |r|, B^T w) are accumulated in binary64
// and the k x k system is solved in binary64 with exact integer cofactors, then rounded once.  The
// comparison that decides a code is binary32.
#pragma once
#include <type_traits>

#include "amq_device.h"

namespace amq {

template <int N>
__device__ __forceinline__ long long idet(const long long* m) {
  if constexpr (N == 1) {
    return m[0];
  } else if constexpr (N == 2) {
    return m[0] * m[3] - m[1] * m[2];
  } else {
    long long d = 0;
#pragma unroll
    for (int c = 0; c < N; ++c) {
      long long sub[(N - 1) * (N - 1)];
#pragma unroll
      for (int i = 1; i < N; ++i) {
        int cc = 0;
#pragma unroll
        for (int j = 0; j < N; ++j) {
          if (j == c) continue;
          sub[(i - 1) * (N - 1) + cc] = m[i * N + j];
          ++cc;
        }
      }
      long long t = m[c] * idet<N - 1>(sub);
      d += (c & 1) ? -t : t;
    }
    return d;
  }
}

// Eq. 5 for one vector: alpha = G^{-1} q with G the integer Gram matrix of the codes.
// G^{-1} = adj(G) / det(G) with exact integer cofactors (|entries| <= n <= 16384, K <= 4 fits
// 64-bit).  A singular G leaves alpha unchanged.
template <int K>
__device__ __forceinline__ void ls_solve(const int (&G)[K][K], const double (&q)[K], float (&alpha)[K]) {
  if constexpr (K == 1) {
    alpha[0] = (float)(q[0] / (double)G[0][0]);
  } else {
    long long m[K * K];
#pragma unroll
    for (int i = 0; i < K; ++i)
#pragma unroll
      for (int j = 0; j < K; ++j) m[i * K + j] = G[i][j];
    // cofactors of the first column give the determinant; all cofactors give the adjugate
    long long cof[K][K];
#pragma unroll
    for (int i = 0; i < K; ++i)
#pragma unroll
      for (int j = 0; j < K; ++j) {
        long long sub[(K - 1) * (K - 1)];
        int rr = 0;
#pragma unroll
        for (int a = 0; a < K; ++a) {
          if (a == i) continue;
          int cc = 0;
#pragma unroll
          for (int b = 0; b < K; ++b) {
            if (b == j) continue;
            sub[rr * (K - 1) + cc] = m[a * K + b];
            ++cc;
          }
          ++rr;
        }
        long long d = idet<K - 1>(sub);
        cof[i][j] = ((i + j) & 1) ? -d : d;
      }
    long long det = 0;
#pragma unroll
    for (int j = 0; j < K; ++j) det += m[j] * cof[0][j];
    if (det == 0) return;
    const double inv = 1.0 / (double)det;
#pragma unroll
    for (int i = 0; i < K; ++i) {
      // adj = cof^T; G symmetric so cof is symmetric too, but keep the general form
      double s = 0.0;
#pragma unroll
      for (int j = 0; j < K; ++j) s += (double)cof[j][i] * q[j];
      alpha[i] = (float)(s * inv);
    }
  }
}

// 1 / d for an integer-valued d != 0 far from the ends of the exponent range: hardware estimate
// and two Newton steps (error below one unit in the last place of binary64, which disappears when
// the coefficients are rounded to binary32).
__device__ __forceinline__ double recip_f64(double d) {
  double r = __builtin_amdgcn_rcp(d);
  r = __builtin_fma(r, __builtin_fma(-d, r, 1.0), r);
  r = __builtin_fma(r, __builtin_fma(-d, r, 1.0), r);
  return r;
}

// Eq. 5 on the vector unit in binary64, from the disagreement counts d[t] of the plane pairs (order (0,1),
// (0,2), .., (1,2), ..): G_ij = n - 2 d_ij, alpha_i = (sum_j cof_ji q_j) / det with exact cofactors and an
// exact determinant for n <= 16384: the cofactors are integers of at most 45 bits, and at K = 4, where the
// determinant may have 56, it is formed from terms n * cof that are multiples of 16 (every 3 x 3 minor of a
// +-1 matrix is a multiple of 4), hence exact too.  A singular G leaves alpha unchanged (returns false).
template <int K>
__device__ __forceinline__ bool ls_solve_f64(int n, const double* d, const double (&q)[K], float (&alpha)[K]) {
  const double dn = (double)n;
  if constexpr (K == 1) {
    alpha[0] = (float)(q[0] / dn);
  } else if constexpr (K == 2) {
    const double a = dn - 2.0 * d[0];
    const double det = dn * dn - a * a;
    if (det == 0.0) return false;
    const double inv = recip_f64(det);
    alpha[0] = (float)((dn * q[0] + (-a) * q[1]) * inv);
    alpha[1] = (float)(((-a) * q[0] + dn * q[1]) * inv);
  } else if constexpr (K == 3) {
    const double a = dn - 2.0 * d[0], b = dn - 2.0 * d[1], c = dn - 2.0 * d[2];
    const double nn = dn * dn;
    const double c00 = nn - c * c, c01 = c * b - a * dn, c02 = a * c - dn * b;
    const double c11 = nn - b * b, c12 = a * b - dn * c, c22 = nn - a * a;
    const double det = dn * c00 + a * c01 + b * c02;
    if (det == 0.0) return false;
    const double inv = recip_f64(det);
    alpha[0] = (float)((c00 * q[0] + c01 * q[1] + c02 * q[2]) * inv);
    alpha[1] = (float)((c01 * q[0] + c11 * q[1] + c12 * q[2]) * inv);
    alpha[2] = (float)((c02 * q[0] + c12 * q[1] + c22 * q[2]) * inv);
  } else {
    static_assert(K == 4, "at most 4 planes");
    const double a = dn - 2.0 * d[0], b = dn - 2.0 * d[1], c = dn - 2.0 * d[2];   // G01 G02 G03
    const double e = dn - 2.0 * d[3], f = dn - 2.0 * d[4], g = dn - 2.0 * d[5];   // G12 G13 G23
    // 2 x 2 minors of rows 0, 1 (s) and of rows 2, 3 (t), columns (0,1) (0,2) (0,3) (1,2) (1,3) (2,3)
    const double s0 = dn * dn - a * a, s1 = dn * e - b * a, s2 = dn * f - c * a;
    const double s3 = a * e - b * dn, s4 = a * f - c * dn, s5 = b * f - c * e;
    const double t1 = b * g - dn * c, t2 = b * dn - g * c, t3 = e * g - dn * f;
    const double t4 = e * dn - g * f, t5 = dn * dn - g * g;
    const double c00 = dn * t5 - e * t4 + f * t3, c01 = b * t4 - a * t5 - c * t3;
    const double c02 = f * s5 - g * s4 + dn * s3, c03 = dn * s4 - e * s5 - g * s3;
    const double c11 = dn * t5 - b * t2 + c * t1, c12 = g * s2 - c * s5 - dn * s1;
    const double c13 = b * s5 - dn * s2 + g * s1, c22 = c * s4 - f * s2 + dn * s0;
    const double c23 = e * s2 - b * s4 - g * s0, c33 = b * s3 - e * s1 + dn * s0;
    const double det = (dn * c00 + a * c01) + (b * c02 + c * c03);
    if (det == 0.0) return false;
    const double inv = recip_f64(det);
    alpha[0] = (float)((c00 * q[0] + c01 * q[1] + c02 * q[2] + c03 * q[3]) * inv);
    alpha[1] = (float)((c01 * q[0] + c11 * q[1] + c12 * q[2] + c13 * q[3]) * inv);
    alpha[2] = (float)((c02 * q[0] + c12 * q[1] + c22 * q[2] + c23 * q[3]) * inv);
    alpha[3] = (float)((c03 * q[0] + c13 * q[1] + c23 * q[2] + c33 * q[3]) * inv);
  }
  return true;
}

// v_writelane_b32: lane `lane` (a constant) of `old` takes the wave-uniform `value`.  (The compiler's
// intrinsic, reached by its name: this compiler has no builtin for it.)
extern "C" __device__ int amq_writelane_i32(int value, int lane, int old) __asm("llvm.amdgcn.writelane.i32");

// This lane's bit of a wave-uniform 64-bit mask, as a condition (the mask becomes the lane mask of whatever
// selects on it; no vector instruction).
extern "C" __device__ bool amq_inverse_ballot_i64(unsigned long long mask) __asm("llvm.amdgcn.inverse.ballot.i64");
__device__ __forceinline__ bool lane_bit(unsigned long long mask) { return amq_inverse_ballot_i64(mask); }

// Lane j keeps the wave-uniform 64-bit value `mk` (the ballot of slot j): one lane write per half, which
// takes the value straight from the scalar registers the comparison wrote.
__device__ __forceinline__ void keep_in_lane(unsigned long long& mine, unsigned long long mk, int j) {
  int lo = (int)(unsigned)(mine & 0xffffffffull), hi = (int)(unsigned)(mine >> 32);
  lo = amq_writelane_i32((int)(unsigned)(mk & 0xffffffffull), j, lo);
  hi = amq_writelane_i32((int)(unsigned)(mk >> 32), j, hi);
  mine = ((unsigned long long)(unsigned)hi << 32) | (unsigned)lo;
}

__device__ __forceinline__ float readlane_f(float v, int l) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l));
}

template <int CTRL>
__device__ __forceinline__ double dpp_d(double v) {
  // (lanes without a source read 0: no previous value to keep, no register to clear)
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, 0xf, 0xf, true);
  return __hiloint2double(hi, lo);
}

// Sums of NV doubles over the 64 lanes through DPP (no LDS traffic), valid in lane 63.  The NV chains are
// independent and interleave.
template <int NV>
__device__ __forceinline__ void wave_sums_lane63(double (&v)[NV]) {
#pragma unroll
  for (int i = 0; i < NV; ++i) v[i] += dpp_d<0xB1>(v[i]);   // quad_perm [1,0,3,2]
#pragma unroll
  for (int i = 0; i < NV; ++i) v[i] += dpp_d<0x4E>(v[i]);   // quad_perm [2,3,0,1]
#pragma unroll
  for (int i = 0; i < NV; ++i) v[i] += dpp_d<0x141>(v[i]);  // row_half_mirror
#pragma unroll
  for (int i = 0; i < NV; ++i) v[i] += dpp_d<0x140>(v[i]);  // row_mirror: every lane holds its row's sum
#pragma unroll
  for (int i = 0; i < NV; ++i) v[i] += dpp_d<0x142>(v[i]);  // row_bcast15: rows 1 and 3 now hold two rows (0 and 2 are not used again)
#pragma unroll
  for (int i = 0; i < NV; ++i) v[i] += dpp_d<0x143>(v[i]);  // row_bcast31: row 3 holds all four
}

// The same, wave-uniform (read from lane 63).
template <int NV>
__device__ __forceinline__ void wave_totals(double (&v)[NV]) {
  wave_sums_lane63<NV>(v);
#pragma unroll
  for (int i = 0; i < NV; ++i) {
    const int lo = __builtin_amdgcn_readlane(__double2loint(v[i]), 63);
    const int hi = __builtin_amdgcn_readlane(__double2hiint(v[i]), 63);
    v[i] = __hiloint2double(hi, lo);
  }
}

constexpr int kMaxRed = 10;  // K coefficients + K(K-1)/2 plane pairs at K = 4

// Totals over the whole workgroup; one barrier per call, two LDS buffers used alternately.
template <int NW, int NV>
__device__ __forceinline__ void block_totals(double (&v)[NV], double (*sh)[16 * kMaxRed], int& phase) {
  wave_totals<NV>(v);
  if constexpr (NW > 1) {
    const int wv = wave_id();
    if (lane_id() == 0) {
#pragma unroll
      for (int i = 0; i < NV; ++i) sh[phase][wv * NV + i] = v[i];
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      double t = sh[phase][i];
#pragma unroll
      for (int w = 1; w < NW; ++w) t += sh[phase][w * NV + i];
      v[i] = t;
    }
    phase ^= 1;
  }
}


// ---------------------------------------------------------------------------------------------------------
// Alg. 2 on magnitudes.
//
// The code table is symmetric (negating every plane negates the value, exactly, in binary32), so the whole
// algorithm runs on |w|: with s the sign of an entry and H = 2^(K-1), the upper half of the sorted table holds
// H values with H - 1 positive midpoints t_1 <= .. <= t_{H-1}, and plane i of an entry's code is
//     plane_i = f_i(m) ^ s,     m = number of midpoints that |w| reaches,
// f_i(m) being plane i of the code at position H + m (the middle midpoint is exactly 0).  The comparison
// "w >= midpoint" sends ties up, which on magnitudes is >= for w >= 0 and > for w < 0; both are one integer
// comparison u >= bits(t) with u = bits(|w|) for w >= 0 and bits(|w|) - 1 for w < 0 (-0.0 counts as +0.0).
//   - The 2^K - 1 comparisons of a pass become 2^(K-1) - 1: one at 2 bits, three at 3.
//   - Everything Eq. 5 needs from a pass are, per midpoint, C_t = sum of |w| over u >= t_t and N_t = the number
//     of such entries: B_i^T w = +-sum |w| +- 2 C_t .. with signs that depend only on where f_i changes, and the
//     disagreement counts of the plane pairs likewise.  No code is formed before the last pass.
//   - C_t is accumulated by ONE binary64 addition under the comparison's own mask as the lane mask (a masked
//     addition costs 5.3 cycles of a SIMD, measured; selecting +-w first costs 13).
//   - alpha_K of the greedy start is needed only where the first Gram matrix is singular (or T = 0): its sum of |r| is
//     formed there and nowhere else, and at two planes no residual at all (k = 2: 16384 x 4096 73.6 -> 69.3, 42000 x 300
//     25.3 -> 23.4, 20000 x 1500 44.0 -> 40.5; k = 3 2 to 5 %).
//   - the reconstruction is read off the table by position, not put together from the planes (a select per midpoint
//     instead of two lane reads, a select and an addition per plane: 16000 x 4096 at k = 3 / 4 with its copy of the gradient
//     247 / 403 -> 229 / 371, 42000 x 300 67 / 130 -> 57 / 109).
// Bound: vector-instruction issue at k >= 3 and HBM at k <= 2 for many vectors, the chain of reductions for a few.
// Measured (us) against the form that compared w with all midpoints and selected +-w per plane, k = 2 / 3 / 4:
// 16384 x 4096 135 / 239 / 443 -> 65 / 122 / 285, 4096 x 2048 33 / 54 / 100 -> 9.9 / 18.1 / 36, 128 vectors of 1024
// 4.4 / 5.9 / 10.1 -> 3.4 / 4.0 / 6.7 (normal values, launches back to back; with an event around each and heavy tails
// 16384 x 4096 takes 73 / 133 / 298).

// A value the compiler must take as new: keeps it from holding the comparison masks of one pass in scalar registers
// for a later pass (16 slots of them spill), where forming them again is one comparison.
__device__ __forceinline__ int opaque_s(int v) { asm volatile("" : "+s"(v)); return v; }
__device__ __forceinline__ float opaque_v(float v) { asm volatile("" : "+v"(v)); return v; }

// count += number of mask bits, slot by slot: left to itself the compiler sums the counts of all slots at the end of
// a pass and holds (spills) their masks until then.
template <int NJ>
__device__ __forceinline__ void add_count(int& count, unsigned long long m) {
  count += __popcll(m);
  if constexpr (NJ > 4) count = opaque_s(count);
}

// The mask bits of the lanes of slot (base + j) that lie inside a vector of n entries.
__device__ __forceinline__ unsigned long long lanes_inside(int n, int slot) {
  const int left = n - slot * 64;
  return left >= 64 ? ~0ull : left <= 0 ? 0ull : (1ull << left) - 1ull;
}

// c[t] += |x| in the lanes of mask m[t].  The lane mask is set from the mask for the addition and restored to all
// lanes (every wave runs whole and undiverged here).
template <int NT>
__device__ __forceinline__ void masked_add(double (&c)[NT], double x, const unsigned long long (&m)[NT]) {
  static_assert(NT == 1 || NT == 3 || NT == 7, "midpoints of the upper half of the code table");
  if constexpr (NT == 1) {
    asm volatile("s_mov_b64 exec, %[m0]\n\tv_add_f64 %[c0], %[c0], |%[x]|\n\ts_mov_b64 exec, -1"
                 : [c0] "+v"(c[0]) : [x] "v"(x), [m0] "s"(m[0]));
  } else if constexpr (NT == 3) {
    asm volatile("s_mov_b64 exec, %[m0]\n\tv_add_f64 %[c0], %[c0], |%[x]|\n\t"
                 "s_mov_b64 exec, %[m1]\n\tv_add_f64 %[c1], %[c1], |%[x]|\n\t"
                 "s_mov_b64 exec, %[m2]\n\tv_add_f64 %[c2], %[c2], |%[x]|\n\ts_mov_b64 exec, -1"
                 : [c0] "+v"(c[0]), [c1] "+v"(c[1]), [c2] "+v"(c[2])
                 : [x] "v"(x), [m0] "s"(m[0]), [m1] "s"(m[1]), [m2] "s"(m[2]));
  } else {
    asm volatile("s_mov_b64 exec, %[m0]\n\tv_add_f64 %[c0], %[c0], |%[x]|\n\t"
                 "s_mov_b64 exec, %[m1]\n\tv_add_f64 %[c1], %[c1], |%[x]|\n\t"
                 "s_mov_b64 exec, %[m2]\n\tv_add_f64 %[c2], %[c2], |%[x]|\n\t"
                 "s_mov_b64 exec, %[m3]\n\tv_add_f64 %[c3], %[c3], |%[x]|\n\t"
                 "s_mov_b64 exec, %[m4]\n\tv_add_f64 %[c4], %[c4], |%[x]|\n\t"
                 "s_mov_b64 exec, %[m5]\n\tv_add_f64 %[c5], %[c5], |%[x]|\n\t"
                 "s_mov_b64 exec, %[m6]\n\tv_add_f64 %[c6], %[c6], |%[x]|\n\ts_mov_b64 exec, -1"
                 : [c0] "+v"(c[0]), [c1] "+v"(c[1]), [c2] "+v"(c[2]), [c3] "+v"(c[3]), [c4] "+v"(c[4]), [c5] "+v"(c[5]),
                   [c6] "+v"(c[6])
                 : [x] "v"(x), [m0] "s"(m[0]), [m1] "s"(m[1]), [m2] "s"(m[2]), [m3] "s"(m[3]), [m4] "s"(m[4]),
                   [m5] "s"(m[5]), [m6] "s"(m[6]));
  }
}

// Sums over the 64 lanes of up to four doubles on the matrix cores, which add f64 values exactly as the vector unit does
// (v_mfma_f64_4x4x4_4b: four blocks of 4 x 4 x 4; lane i + 4 b + 16 k holds A_b[i][k] and B_b[k][i], and lane
// j + 4 b + 16 i receives D_b[i][j]).  Value j of the lanes times column selector j, accumulated over the values, leaves
// in column j the sums over k; ones times that, the sums over i as well: lane l then holds the sum of value l % 4 over the
// 16 lanes of block (l / 4) % 4.
template <int NV>
__device__ __forceinline__ double matrix_sums(const double* v) {
  static_assert(NV >= 1 && NV <= 4, "columns");
  int j = lane_id() & 3;
  asm volatile("" : "+v"(j));  // (the selectors are formed here, not kept in registers from one exchange to the next)
  double acc = 0.0;
#pragma unroll
  for (int i = 0; i < NV; ++i) acc = __builtin_amdgcn_mfma_f64_4x4x4f64(v[i], j == i ? 1.0 : 0.0, acc, 0, 0, 0);
  return __builtin_amdgcn_mfma_f64_4x4x4f64(1.0, acc, 0.0, 0, 0, 0);
}

// Doubles of LDS for one of the two buffers of the exchanges of a workgroup of NW waves.
template <int NW>
constexpr int kExchange = NW == 1 ? 1 : 2 * 16 * NW;

// Totals over a workgroup of NW waves of the NE per-lane doubles e, left in e[0] and e[4]: value i is in e[i & ~3] of the
// lane total_lane<NW>(i).  Latency is what counts here (the reductions are the serial part of the algorithm): per wave the
// sums of all values take one matrix instruction each and one more, 16 partial sums (value, block) go to LDS in one
// write, and after the one barrier every lane reads one (value, block, wave) entry of each four waves, and two matrix
// instructions sum over waves and blocks.  Measured over four waves: 356 cycles for one value, 530 for four.
// sh: 2 * kExchange<NW> doubles, the two buffers used alternately.  A workgroup may hold several groups of NW waves that work on
// a vector each, with an sh each, in step: all pass the same barriers.
template <int NW>
__device__ __forceinline__ constexpr int total_lane(int i) { return (i & 3) * (NW == 1 ? 1 : 4); }

template <int NW, int NE>
__device__ __forceinline__ void exchange_raw(double (&e)[4 * ((NE + 3) / 4)], double* sh, int& phase) {
  constexpr int NG = (NE + 3) / 4, last = NE - 4 * (NG - 1);
  static_assert(NG <= 2, "LDS buffer");
#pragma unroll
  for (int g = 0; g < NG; ++g) {
    double t = g + 1 < NG ? matrix_sums<4>(e + 4 * g) : matrix_sums<last>(e + 4 * g);
    if constexpr (NW == 1) {
      t += dpp_d<0x124>(t);  // row_ror:4
      t += dpp_d<0x128>(t);  // row_ror:8: over the blocks
      e[4 * g] = t;
    } else {
      const int lane = lane_id();
      if (lane < 16) sh[phase * kExchange<NW> + (g * NW + (wave_id() & (NW - 1))) * 16 + lane] = t;
    }
  }
  if constexpr (NW > 1) {
    lds_barrier();
    const int lane = lane_id();
    const double* mine = sh + phase * kExchange<NW> + ((lane >> 2) & 3) + 4 * (lane & 3);  // value (lane / 4) % 4, block lane % 4
#pragma unroll
    for (int g = 0; g < NG; ++g) {
      double t;
      if constexpr (NW == 2) {
        t = 0.5 * mine[(g * NW + ((lane >> 4) & 1)) * 16];  // (both waves twice)
      } else {
        t = mine[(g * NW + (lane >> 4)) * 16];
#pragma unroll
        for (int w = 4; w < NW; w += 4) t += mine[(g * NW + w + (lane >> 4)) * 16];
      }
      t = __builtin_amdgcn_mfma_f64_4x4x4f64(t, 1.0, 0.0, 0, 0, 0);
      e[4 * g] = __builtin_amdgcn_mfma_f64_4x4x4f64(1.0, t, 0.0, 0, 0, 0);  // lane l: total of value (l / 4) % 4
    }
    phase ^= 1;
  }
}

__device__ __forceinline__ double readlane_d(double x, int l) {
  return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(x), l), __builtin_amdgcn_readlane(__double2loint(x), l));
}

// Up to three counts of at most 16384 (15 bits each) in the last places of 2^52 + packed.
__device__ __forceinline__ int count_of(unsigned long long p, int k) { return (int)((p >> (15 * k)) & 0x7fffu); }

// Totals of NV per-lane doubles v and of NC wave-uniform counts c, the same in every lane.  The counts travel three to a
// double (the sums are exact).
template <int NW, int NV, int NC>
__device__ __forceinline__ void exchange_totals(double (&v)[NV], int (&c)[NC > 0 ? NC : 1], double* sh, int& phase) {
  constexpr int NCW = NW == 1 ? 0 : (NC + 2) / 3;
  constexpr int NE = NV + NCW;
  double e[4 * ((NE + 3) / 4)];
#pragma unroll
  for (int i = 0; i < NV; ++i) e[i] = v[i];
#pragma unroll
  for (int i = 0; i < NCW; ++i) {
    unsigned long long p = 0x42d0000000000000ull;  // 2^46, in whose last place a count stands for itself / 64
#pragma unroll
    for (int k = 0; k < 3; ++k)
      if (3 * i + k < NC) p |= (unsigned long long)(unsigned)c[3 * i + k] << (15 * k);
    e[NV + i] = __longlong_as_double((long long)p) - 0x1p46;  // a 64th of the wave's counts in every lane
  }
  exchange_raw<NW, NE>(e, sh, phase);
#pragma unroll
  for (int i = 0; i < NV; ++i) v[i] = readlane_d(e[i & ~3], total_lane<NW>(i));
#pragma unroll
  for (int i = 0; i < NCW; ++i) {
    const int at = NV + i;
    const unsigned long long p =
        (unsigned long long)__double_as_longlong(readlane_d(e[at & ~3] + 0x1p52, total_lane<NW>(at)));
#pragma unroll
    for (int k = 0; k < 3; ++k)
      if (3 * i + k < NC) c[3 * i + k] = count_of(p, k);
  }
}

// The upper half of the sorted code table: thr[t-1] = bits of the midpoint between positions t-1 and t (wave-
// uniform), and per plane the H-bit mask of f_i over the positions.  Values are the binary32 left-to-right sums
// of Alg. 2; equal values keep the order of their patterns.
template <int K>
struct CodeTable {
  static constexpr int H = 1 << (K - 1);
  int thr[H > 1 ? H - 1 : 1];
  unsigned bm[K];
  int val[H];  // bits of the values, not negative (filled by code_table)
};

__device__ __forceinline__ int uniform_bits(float v) { return __builtin_amdgcn_readfirstlane(__float_as_int(v)); }

template <int K>
__device__ __forceinline__ void code_table_any_order(const float (&alpha)[K], CodeTable<K>& ct) {
  // lane p < H owns the pair of patterns p | H and its complement, represented by the one whose value is not
  // negative; it ranks its (value, pattern) among the H pairs and pushes it to the lane of its rank
  constexpr int H = CodeTable<K>::H;
  const int lane = lane_id();
  const int p = (lane & (H - 1)) | H;
  float v = 0.0f;
#pragma unroll
  for (int i = 0; i < K; ++i) {
    const float term = ((p >> (K - 1 - i)) & 1) ? alpha[i] : -alpha[i];
    v = (i == 0) ? term : v + term;
  }
  const int pat = (v < 0.0f) ? (2 * H - 1) ^ p : p;
  const int vb = __float_as_int(fabsf(v));
  int rank = 0;
#pragma unroll
  for (int o = 0; o < H; ++o) {
    const int vo = __builtin_amdgcn_readlane(vb, o), po = __builtin_amdgcn_readlane(pat, o);
    rank += (vo < vb || (vo == vb && po < pat)) ? 1 : 0;
  }
  if (lane >= H) rank = lane;
  const float sv = __int_as_float(__builtin_amdgcn_ds_permute(rank << 2, vb));
  const int sp = __builtin_amdgcn_ds_permute(rank << 2, pat);
  const float up = __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(sv), 0x101 /* row_shl:1 */, 0xf, 0xf, true));
  const int mid = __float_as_int(0.5f * (sv + up));
#pragma unroll
  for (int t = 0; t < H - 1; ++t) ct.thr[t] = __builtin_amdgcn_readlane(mid, t);
#pragma unroll
  for (int i = 0; i < K; ++i) ct.bm[i] = (unsigned)__ballot((sp & (1 << (K - 1 - i))) != 0) & ((1u << H) - 1u);
#pragma unroll
  for (int t = 0; t < H; ++t) ct.val[t] = __builtin_amdgcn_readlane(__float_as_int(sv), t);
}

template <int K>
__device__ __forceinline__ void code_table(const float (&alpha)[K], CodeTable<K>& ct) {
  static_assert(K >= 2, "one plane has no midpoint but 0");
  if constexpr (K == 2) {
    // alpha_1 >= alpha_2 >= 0, the order after any ordinary least-squares step
    const float v2 = alpha[0] - alpha[1], v3 = alpha[0] + alpha[1];
    if (__ballot(v2 >= 0.0f && alpha[1] >= 0.0f) != 0ull) {
      ct.thr[0] = uniform_bits(0.5f * (v2 + v3));
      ct.bm[0] = 3u;
      ct.bm[1] = 2u;
      ct.val[0] = uniform_bits(v2);
      ct.val[1] = uniform_bits(v3);
      return;
    }
  } else if constexpr (K == 3) {
    // patterns 100 (or its complement 011), 101, 110, 111 in this order: the two cases that occur in practice
    const float d = alpha[0] - alpha[1], s = alpha[0] + alpha[1];
    const float v4 = d - alpha[2], v5 = d + alpha[2], v6 = s - alpha[2], v7 = s + alpha[2];
    const float lo = fabsf(v4);
    if (__ballot(lo <= v5 && v5 <= v6 && v6 <= v7) != 0ull) {
      ct.thr[0] = uniform_bits(0.5f * (lo + v5));
      ct.thr[1] = uniform_bits(0.5f * (v5 + v6));
      ct.thr[2] = uniform_bits(0.5f * (v6 + v7));
      const bool swap = __ballot(v4 < 0.0f) != 0ull;
      ct.bm[0] = swap ? 0xeu : 0xfu;
      ct.bm[1] = swap ? 0xdu : 0xcu;
      ct.bm[2] = swap ? 0xbu : 0xau;
      ct.val[0] = uniform_bits(lo);
      ct.val[1] = uniform_bits(v5);
      ct.val[2] = uniform_bits(v6);
      ct.val[3] = uniform_bits(v7);
      return;
    }
  }
  code_table_any_order<K>(alpha, ct);
}

// Step of f at position t: f(t) - f(t - 1), from the mask of a plane (or of the difference of two planes).
__device__ __forceinline__ int step_at(unsigned bm, int t) { return (int)((bm >> t) & 1u) - (int)((bm >> (t - 1)) & 1u); }

// B_i^T w = sum |w| (2 f_i - 1) = q0 + sum_t 2 (step of f_i at t) C_t with q0 = +-sum |w| by f_i(0); the factors
// are exact powers of two.
template <int NT>
__device__ __forceinline__ double plane_dot(unsigned bm, double q0, const double (&c)[NT]) {
  double q = q0;
#pragma unroll
  for (int t = 1; t <= NT; ++t) q = __builtin_fma(__hiloint2double(step_at(bm, t) << 30, 0), c[t - 1], q);
  return q;
}

// Up to this many slots per lane the sign masks of the slots stay in scalar registers; beyond, a sign is taken from
// the stored value where it is needed (16 slots would fill a third of the scalar registers and spill).
constexpr int kSignMaskSlots = 4;

// Alg. 2 for one vector: x[j] of lane L is entry (base + j) * 64 + L (0 beyond n), NW waves cooperate with nj
// slots each.  On return alpha holds the coefficients and lane j of each wave, in mym[i], the 64 packed codes of
// its slot j of plane i.  Slots below MASKED lie inside the vector; an entry of the others that does not is 0 and its u
// is -1, below every midpoint (branches around absent slots cost a vector of 650 entries twice the time of 640).
template <int K, int NJ, int NW, int MASKED, bool RECON = false>
__device__ __forceinline__ void quantize_magnitudes(const float (&x)[NJ], int n, int base, int nj, int T,
                                                    float (&alpha)[K], unsigned long long (&mym)[K],
                                                    double* sh, int& phase, unsigned long long* marks,
                                                    float* recon = nullptr) {
  (void)marks;  // phase timers of the profiling build: 2 = greedy done, 4 + 4 * cycle + {0: reduction, 1: solve, 2: table, 3: assignment}
  constexpr int H = 1 << (K - 1);
  constexpr int NT = H > 1 ? H - 1 : 1;
  constexpr int NP = K * (K - 1) / 2;
  const double dn = (double)n;
  const double inv_n = recip_f64(dn);  // (exact for a power of two; the last binary64 digit is rounded away)
  auto mean = [&](double s) { return (float)(s * inv_n); };
  const int within = min(n - base * 64, nj * 64) - lane_id();  // this lane has an entry in slot j if j * 64 < within
  const unsigned long long lane_inside = MASKED == NJ ? ~0ull : lanes_inside(n, base + lane_id());

  int u[NJ];                     // order-preserving integer of |w| with the tie rule folded in
  // w: as the binary64 value that the additions take, or (where registers are what limits the waves) as the binary32 value,
  // converted at every use
  constexpr bool kNarrow = NJ > 16 || (K == 2 && NW > 1) || (K == 4 && NW == 16);
  using Held = typename std::conditional<kNarrow, float, double>::type;
  Held held[NJ];
  auto wide = [&](int j) {
    if constexpr (kNarrow) return (double)opaque_v(held[j]);
    else return held[j];
  };
  auto narrow = [&](int j) {
    Held w0 = held[j];
    asm volatile("" : "+v"(w0));  // (otherwise what is formed from it here and earlier is kept in registers from the start)
    return (float)w0;
  };
  auto sign_bits = [&](int j) {
    if constexpr (kNarrow) return __float_as_int(held[j]);
    else return __double2hiint(held[j]);
  };
  float r[NJ];                   // greedy residual
  unsigned long long neg[NJ <= kSignMaskSlots ? NJ : 1];  // w < 0
  unsigned long long lane_neg = 0ull;                     // the same, slot j in lane j
  double sum[1] = {0.0};
  int no_counts[1] = {0};
#pragma unroll
  for (int j = 0; j < NJ; ++j) {
    const float xc = x[j] + 0.0f;  // -0.0 -> +0.0
    const unsigned b = __float_as_uint(xc);
    // b, or bits(|w|) - 1 = b + 0x7fffffff (mod 2^32) for a set sign bit: the smaller of the two in both cases
    u[j] = (int)min(b, b + 0x7fffffffu);
    if (j >= MASKED) u[j] = j * 64 < within ? u[j] : -1;
    held[j] = (Held)xc;
    const unsigned long long ng = __ballot(xc < 0.0f);
    if constexpr (NJ <= kSignMaskSlots) neg[j] = ng;
    keep_in_lane(lane_neg, ng, j);
    r[j] = xc;
    sum[0] = (j == 0) ? fabs(wide(j)) : sum[0] + fabs(wide(j));
    if (NJ > 4 && (j & 3) == 3) __builtin_amdgcn_sched_barrier(0);
  }
  AMQ_PHASE(marks, 12);
  exchange_totals<NW, 1, 0>(sum, no_counts, sh, phase);
  AMQ_PHASE(marks, 13);
  const double l1 = sum[0];
  alpha[0] = mean(l1);
  if constexpr (K == 1) {
    // the sign codes are final: Eq. 5 returns mean |w| again and the only midpoint is 0
    if constexpr (RECON) {
#pragma unroll
      for (int j = 0; j < NJ; ++j) recon[j] = r[j] < 0.0f ? -alpha[0] : alpha[0];
    }
    mym[0] = ~lane_neg & lane_inside;
    return;
  } else {
    // ---- greedy stages 2 .. K (Eq. 4): the residual loses the previous plane, its sign is the next plane.
    // s[i - 1] = sum of |w| where plane i agrees with the sign of w, cnt = disagreement counts of the plane pairs.
    double s[K - 1];
    int cnt[NP];
#pragma unroll
    for (int i = 0; i < NP; ++i) cnt[i] = 0;
#pragma unroll
    for (int i = 1; i < K; ++i) {
      const float a = alpha[i - 1];
      const int abits = uniform_bits(a);
      const int a0bits = opaque_s(uniform_bits(alpha[0]));
      double sr[1] = {0.0}, si[1] = {0.0};
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        const unsigned long long in = j < MASKED ? ~0ull : __ballot(u[j] >= 0);
        unsigned long long before = 0ull;  // previous plane against the sign of w
        if (NJ > 4 && i > 2) r[j] = opaque_v(r[j]);
        if (i > 1) before = __ballot(r[j] < 0.0f);
        float rn = 0.0f;
        if (K > 2) {
          rn = r[j] - copysignf(a, r[j]);  // (a difference is never -0.0)
          if (j >= MASKED) rn = lane_bit(in) ? rn : 0.0f;
          r[j] = rn;
        }
        unsigned long long f[1];
        if (i == 1) {
          f[0] = __ballot(u[j] >= abits);
        } else {
          const unsigned long long ng = __ballot(rn < 0.0f);
          if constexpr (NJ <= kSignMaskSlots) f[0] = ~(ng ^ neg[j]);
          else f[0] = __ballot((__float_as_int(rn) ^ sign_bits(j)) >= 0);
          // pairs (i - 1, i) of planes beyond the first: both signs are at hand
          add_count<NJ>(cnt[K == 3 ? 2 : (i == 2 ? 3 : 5)], (before ^ ng) & in);
          if (K == 4 && i == 3) add_count<NJ>(cnt[4], (__ballot(u[j] >= a0bits) ^ f[0]) & in);
        }
        if (i > 1) f[0] &= in;
        add_count<NJ>(cnt[i - 1], f[0]);
        masked_add<1>(si, wide(j), f);
        if (i + 1 < K) {
          const double ra = (double)fabsf(rn);
          sr[0] = (j == 0) ? ra : sr[0] + ra;
        }
        if (NJ > 4 && (j & 3) == 3) __builtin_amdgcn_sched_barrier(0);
      }
      s[i - 1] = si[0];
      if (i + 1 < K) {
        AMQ_PHASE(marks, 14);
        exchange_totals<NW, 1, 0>(sr, no_counts, sh, phase);
        AMQ_PHASE(marks, 15);
        alpha[i] = mean(sr[0]);
      }
    }
    AMQ_PHASE(marks, 2);
    exchange_totals<NW, K - 1, NP>(s, cnt, sh, phase);
    auto last_greedy_coefficient = [&]() {  // (the whole workgroup or nobody)
      double sr[1] = {0.0};
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        float rj = narrow(j);
#pragma unroll
        for (int i = 0; i + 1 < K; ++i) rj = rj - copysignf(alpha[i], rj);
        if (j >= MASKED) rj = u[j] >= 0 ? rj : 0.0f;
        sr[0] = (j == 0) ? (double)fabsf(rj) : sr[0] + (double)fabsf(rj);
      }
      exchange_totals<NW, 1, 0>(sr, no_counts, sh, phase);
      alpha[K - 1] = mean(sr[0]);
    };
    if (T == 0) {
      last_greedy_coefficient();
      // the greedy result itself: its planes are formed again from the coefficients
#pragma unroll
      for (int i = 0; i < K; ++i) mym[i] = 0ull;
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        float rj = narrow(j);
        float v = 0.0f;
#pragma unroll
        for (int i = 0; i < K; ++i) {
          keep_in_lane(mym[i], __ballot(rj >= 0.0f), j);
          const float term = rj >= 0.0f ? alpha[i] : -alpha[i];
          v = i == 0 ? term : v + term;
          rj = rj - copysignf(alpha[i], rj);
        }
        if constexpr (RECON) recon[j] = v;
      }
#pragma unroll
      for (int i = 0; i < K; ++i) mym[i] &= lane_inside;
      return;
    }
    double q[K], d[NP];
    q[0] = l1;
#pragma unroll
    for (int i = 1; i < K; ++i) {
      q[i] = 2.0 * s[i - 1] - l1;
      d[i - 1] = (double)(n - cnt[i - 1]);
    }
#pragma unroll
    for (int i = K - 1; i < NP; ++i) d[i] = (double)cnt[i];

    CodeTable<K> ct;
    for (int it = 0;; ++it) {
      AMQ_PHASE(marks, 4 + 4 * it);
      if (!ls_solve_f64<K>(n, d, q, alpha) && it == 0) last_greedy_coefficient();
      AMQ_PHASE(marks, 5 + 4 * it);
      code_table<K>(alpha, ct);
      AMQ_PHASE(marks, 6 + 4 * it);
      if (it + 1 == T) break;
      // ---- a pass that another cycle follows: only C_t and N_t
      double c[NT];
      int cn[NT];
#pragma unroll
      for (int t = 0; t < NT; ++t) { c[t] = 0.0; cn[t] = 0; }
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        unsigned long long ge[NT];
#pragma unroll
        for (int t = 0; t < NT; ++t) {
          ge[t] = __ballot(u[j] >= ct.thr[t]);
          add_count<NJ>(cn[t], ge[t]);
        }
        masked_add<NT>(c, wide(j), ge);
        if (NJ > 4 && (j & 3) == 3) __builtin_amdgcn_sched_barrier(0);
      }
      AMQ_PHASE(marks, 7 + 4 * it);
      if constexpr (K == 4) {
        // four plane sums instead of seven C_t through the reduction (this lane's shares, without sum |w|)
        double sp[K];
#pragma unroll
        for (int i = 0; i < K; ++i) sp[i] = plane_dot<NT>(ct.bm[i], 0.0, c);
        exchange_totals<NW, K, NT>(sp, cn, sh, phase);
#pragma unroll
        for (int i = 0; i < K; ++i) q[i] = ((ct.bm[i] & 1u) ? l1 : -l1) + sp[i];
      } else {
        exchange_totals<NW, NT, NT>(c, cn, sh, phase);
#pragma unroll
        for (int i = 0; i < K; ++i) q[i] = plane_dot<NT>(ct.bm[i], (ct.bm[i] & 1u) ? l1 : -l1, c);
      }
      int t0 = 0;
#pragma unroll
      for (int a = 0; a < K; ++a)
#pragma unroll
        for (int b = a + 1; b < K; ++b) {
          const unsigned xo = ct.bm[a] ^ ct.bm[b];
          int dd = (xo & 1u) ? n : 0;
#pragma unroll
          for (int t = 1; t <= NT; ++t) dd += step_at(xo, t) * cn[t - 1];
          d[t0++] = (double)dd;
        }
    }

    if constexpr (RECON) {
      // the value of the position, by selects from the smallest up, with the sign of w (the table is symmetric, exactly)
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        float v = __int_as_float(ct.val[0]);
#pragma unroll
        for (int t = 0; t < NT; ++t) v = u[j] >= ct.thr[t] ? __int_as_float(ct.val[t + 1]) : v;
        recon[j] = sign_bits(j) < 0 ? 0.0f - v : v;
        if (NJ > 4 && (j & 3) == 3) __builtin_amdgcn_sched_barrier(0);
      }
      return;
    }

    // ---- the last pass: the comparison masks, slot j in lane j, then the planes in the lanes
    unsigned long long ge[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) ge[t] = 0ull;
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
#pragma unroll
      for (int t = 0; t < NT; ++t) keep_in_lane(ge[t], __ballot(u[j] >= ct.thr[t]), j);
      if (NJ > 4 && (j & 3) == 3) __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int i = 0; i < K; ++i) {
      unsigned long long p = lane_neg ^ (0ull - (unsigned long long)(ct.bm[i] & 1u));
#pragma unroll
      for (int t = 1; t <= NT; ++t)
        p ^= ge[t - 1] & (0ull - (unsigned long long)(((ct.bm[i] >> t) ^ (ct.bm[i] >> (t - 1))) & 1u));
      mym[i] = p & lane_inside;
    }
    AMQ_PHASE(marks, 11);
  }
}

// ---------------------------------------------------------------------------------------------------------
// The same algorithm where one vector at a time is waited for (on-line quantization: one wave per SIMD, nothing to
// hide behind).  There a wave is bound by the latency of its own instructions, and what is cheap to issue is not what
// is quick: setting the lane mask around an addition takes 38 cycles with the comparison, a selected factor of 0 or 1
// and a fused multiply-add 15; a scalar population count of a comparison waits for the comparison, a second fused
// multiply-add does not.  So
//   - sums under a comparison are c += |w| * m with m = 0 or 1 by one select;
//   - the counts are sums of m * 2^(15 t), three to a double, and go through the same reductions;
//   - thresholds and coefficients stay in vector registers; slots are straight-line code: an entry past the end of the
//     vector is 0 and its u is -1, below every threshold.
//   - coefficients, table and sums of the usual code orders are straight-line code without branches on the data, the
//     rest is out of the way.
// Same arithmetic otherwise.  Measured for a vector of 1024 entries on four waves of one compute unit, k = 2 / 3:
// 2960 / 5730 -> 2650 / 4060 cycles (of which the reductions take about 1100 / 1760).

// 1.0 where `yes`, else 0.0.
__device__ __forceinline__ double one_if(bool yes) { return __hiloint2double(yes ? 0x3ff00000 : 0, 0); }

// Eq. 5 from the inner products g of the planes (integers; pairs in the order of ls_solve_f64), which are exact, as are
// all intermediate values that are in ls_solve_f64.
template <int K>
__device__ __forceinline__ bool ls_solve_gram(int n, double dn, const double* g, const double (&q)[K], float (&alpha)[K]) {
  if constexpr (K == 2) {
    const double a = g[0];
    const double det = __builtin_fma(-a, a, dn * dn);
    const double inv = recip_f64(det);
    const float a0 = (float)(__builtin_fma(-a, q[1], dn * q[0]) * inv);
    const float a1 = (float)(__builtin_fma(-a, q[0], dn * q[1]) * inv);
    alpha[0] = det != 0.0 ? a0 : alpha[0];  // (a select, so that the neighbouring steps stay one block of code)
    alpha[1] = det != 0.0 ? a1 : alpha[1];
    return det != 0.0;
  } else if constexpr (K == 3) {
    const double a = g[0], b = g[1], c = g[2];
    const double nn = dn * dn;
    const double c00 = __builtin_fma(-c, c, nn), c11 = __builtin_fma(-b, b, nn), c22 = __builtin_fma(-a, a, nn);
    const double c01 = __builtin_fma(c, b, -(a * dn)), c02 = __builtin_fma(a, c, -(dn * b)), c12 = __builtin_fma(a, b, -(dn * c));
    const double det = __builtin_fma(b, c02, __builtin_fma(a, c01, dn * c00));
    const double inv = recip_f64(det);
    const float a0 = (float)(__builtin_fma(c02, q[2], __builtin_fma(c01, q[1], c00 * q[0])) * inv);
    const float a1 = (float)(__builtin_fma(c12, q[2], __builtin_fma(c11, q[1], c01 * q[0])) * inv);
    const float a2 = (float)(__builtin_fma(c22, q[2], __builtin_fma(c12, q[1], c02 * q[0])) * inv);
    alpha[0] = det != 0.0 ? a0 : alpha[0];
    alpha[1] = det != 0.0 ? a1 : alpha[1];
    alpha[2] = det != 0.0 ? a2 : alpha[2];
    return det != 0.0;
  } else {
    double d[6];
#pragma unroll
    for (int i = 0; i < 6; ++i) d[i] = 0.5 * (dn - g[i]);
    return ls_solve_f64<K>(n, d, q, alpha);
  }
}

// The code table in vector registers, and which of the usual orders it is in: 0: by pattern (K = 2, 3), 1: by pattern
// with 011 in the place of 100 (K = 3), 2: any other, given by ct.bm.
template <int K>
__device__ __forceinline__ int code_table_kind(const float (&alpha)[K], CodeTable<K>& ct) {
  if constexpr (K == 2) {
    const float v2 = alpha[0] - alpha[1], v3 = alpha[0] + alpha[1];
    if (__builtin_expect(__ballot(v2 >= 0.0f && alpha[1] >= 0.0f) != 0ull, 1)) {
      ct.thr[0] = __float_as_int(0.5f * (v2 + v3));
      return 0;
    }
  } else if constexpr (K == 3) {
    const float d = alpha[0] - alpha[1], s = alpha[0] + alpha[1];
    const float v4 = d - alpha[2], v5 = d + alpha[2], v6 = s - alpha[2], v7 = s + alpha[2];
    const float lo = fabsf(v4);
    if (__builtin_expect(__ballot(lo <= v5 && v5 <= v6 && v6 <= v7) != 0ull, 1)) {
      ct.thr[0] = __float_as_int(0.5f * (lo + v5));
      ct.thr[1] = __float_as_int(0.5f * (v5 + v6));
      ct.thr[2] = __float_as_int(0.5f * (v6 + v7));
      if (__builtin_expect(__ballot(v4 < 0.0f) == 0ull, 1)) return 0;
      ct.bm[0] = 0xeu;
      ct.bm[1] = 0xdu;
      ct.bm[2] = 0xbu;
      return 1;
    }
  }
  code_table_any_order<K>(alpha, ct);
  return 2;
}

// WHOLE: slots below it lie inside the vector in every wave that takes this form.
template <int K, int NJ, int NW, int WHOLE>
__device__ __forceinline__ void quantize_online(const float (&x)[NJ], int n, int base, int nj, int T, float (&alpha)[K],
                                                unsigned long long (&mym)[K], double* sh, int& phase,
                                                unsigned long long* marks) {
  (void)marks;
  constexpr int H = 1 << (K - 1);
  constexpr int NT = H > 1 ? H - 1 : 1;
  constexpr int NP = K * (K - 1) / 2;
  constexpr int NPW = (NP + 2) / 3, NTW = (NT + 2) / 3;  // doubles that carry the counts of the pairs, of the midpoints
  const double dn = (double)n;
  const double inv_n = recip_f64(dn);
  auto mean = [&](double s) { return (float)(s * inv_n); };
  constexpr bool FULL = WHOLE == NJ;
  const unsigned long long lane_inside = FULL ? ~0ull : lanes_inside(n, base + lane_id());
  // all bits set where this lane has an entry in slot j: one bit operation per use in the chain (a comparison with the
  // index, or a mask formed by the scalar unit and a select, take several)
  const int within = min(n - base * 64, nj * 64) - lane_id();
  int in[NJ];
#pragma unroll
  for (int j = WHOLE; j < NJ; ++j) in[j] = (j * 64 - within) >> 31;
  const int outside = NW * NJ * 64 - n;  // entries past the end that the workgroup's slots hold
  const double field[3] = {1.0, 0x1p15, 0x1p30};
  int no_counts[1] = {0};

  int u[NJ];
  float xc[NJ];
  double wd[NJ];
  float r[NJ];
  double sum[1] = {0.0};
#pragma unroll
  for (int j = 0; j < NJ; ++j) {
    xc[j] = x[j] + 0.0f;
    const unsigned b = __float_as_uint(xc[j]);
    u[j] = (int)min(b, b + 0x7fffffffu);
    if (j >= WHOLE) u[j] |= ~in[j];
    wd[j] = fabs((double)xc[j]);
    r[j] = xc[j];
    sum[0] = (j == 0) ? wd[j] : sum[0] + wd[j];
  }
  AMQ_PHASE(marks, 12);
  exchange_totals<NW, 1, 0>(sum, no_counts, sh, phase);
  AMQ_PHASE(marks, 13);
  const double l1 = sum[0];
  alpha[0] = mean(l1);
  auto signs_in_lanes = [&]() {
    unsigned long long m = 0ull;
#pragma unroll
    for (int j = 0; j < NJ; ++j) keep_in_lane(m, __ballot(__float_as_int(xc[j]) < 0), j);
    return m;
  };
  if constexpr (K == 1) {
    mym[0] = ~signs_in_lanes() & lane_inside;
    return;
  } else {
    // ---- greedy stages; red: the sum of |r| of the last stage, s[1 .. K-1], then the packed counts.  A wave on its own
    // forms that sum only where it is needed (a workgroup always: other waves of it may count its barriers).
    constexpr int SK = NW == 1 ? 1 : 0;
    double red[4 * ((K - SK + NPW + 3) / 4)];
    auto tally = [&](int pair, double m) {
      double& acc = red[K - SK + pair / 3];
      acc = __builtin_fma(m, field[pair % 3], acc);
    };
#pragma unroll
    for (int i = 0; i < NPW; ++i) red[K - SK + i] = 0.0;
#pragma unroll
    for (int i = 1; i < K; ++i) {
      const float a = alpha[i - 1];
      double sr = 0.0, si = 0.0;
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        const float before = r[j];
        float rn = before - copysignf(a, before);
        if (j >= WHOLE) rn = __int_as_float(__float_as_int(rn) & in[j]);
        r[j] = rn;
        double m;  // plane i agrees with the sign of w
        if (i == 1) {
          m = one_if(u[j] >= __float_as_int(a));
        } else {
          m = one_if((__float_as_int(rn) ^ __float_as_int(xc[j])) >= 0);
          tally(K == 3 ? 2 : (i == 2 ? 3 : 5), one_if((__float_as_int(before) ^ __float_as_int(rn)) < 0));
          if (K == 4 && i == 3)
            tally(4, one_if((u[j] >= __float_as_int(alpha[0])) != ((__float_as_int(rn) ^ __float_as_int(xc[j])) >= 0)));
        }
        si = __builtin_fma(wd[j], m, si);
        tally(i - 1, m);
        sr += fabs((double)rn);
      }
      red[i - SK] = si;
      if (i + 1 < K) {
        double one[1] = {sr};
        AMQ_PHASE(marks, 14);
        exchange_totals<NW, 1, 0>(one, no_counts, sh, phase);
        AMQ_PHASE(marks, 15);
        alpha[i] = mean(one[0]);
      } else if (SK == 0) {
        red[0] = sr;
      }
    }
    AMQ_PHASE(marks, 2);
    exchange_raw<NW, K - SK + NPW>(red, sh, phase);
    auto total_of = [&](const double* e, int i) { return readlane_d(e[i & ~3], total_lane<NW>(i)); };
    auto counts_of = [&](const double* e, int i) {
      return (unsigned long long)__double_as_longlong(readlane_d(e[i & ~3] + 0x1p52, total_lane<NW>(i)));
    };
    auto last_greedy_coefficient = [&]() {
      if (SK == 0) return;
      double one[1] = {0.0};
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        float rj = xc[j];
#pragma unroll
        for (int i = 0; i + 1 < K; ++i) rj = rj - copysignf(alpha[i], rj);
        if (j >= WHOLE) rj = __int_as_float(__float_as_int(rj) & in[j]);
        one[0] += fabs((double)rj);
      }
      exchange_totals<NW, 1, 0>(one, no_counts, sh, phase);
      alpha[K - 1] = mean(one[0]);
    };
    if (SK == 0) alpha[K - 1] = mean(total_of(red, 0));
    if (T == 0) {
      last_greedy_coefficient();
#pragma unroll
      for (int i = 0; i < K; ++i) mym[i] = 0ull;
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        float rj = xc[j];
#pragma unroll
        for (int i = 0; i < K; ++i) {
          keep_in_lane(mym[i], __ballot(rj >= 0.0f), j);
          rj = rj - copysignf(alpha[i], rj);
        }
      }
#pragma unroll
      for (int i = 0; i < K; ++i) mym[i] &= lane_inside;
      return;
    }
    double q[K], g[NP];
    {
      unsigned long long p[NPW];
#pragma unroll
      for (int i = 0; i < NPW; ++i) p[i] = counts_of(red, K - SK + i);
      q[0] = l1;
#pragma unroll
      for (int i = 1; i < K; ++i) {
        q[i] = __builtin_fma(2.0, total_of(red, i - SK), -l1);
        // plane 0 against plane i; entries past the end agree from the second stage on
        g[i - 1] = (double)(2 * (count_of(p[(i - 1) / 3], (i - 1) % 3) - (i > 1 ? outside : 0)) - n);
      }
      // (planes 1 and 3: past the end plane 1 disagrees with the sign, u being -1, and plane 3 agrees)
#pragma unroll
      for (int i = K - 1; i < NP; ++i) g[i] = (double)(n - 2 * (count_of(p[i / 3], i % 3) - (K == 4 && i == 4 ? outside : 0)));
    }

    CodeTable<K> ct;
    int kind;
    for (int it = 0;; ++it) {
      AMQ_PHASE(marks, 4 + 4 * it);
      const bool solved = ls_solve_gram<K>(n, dn, g, q, alpha);
      if (SK != 0 && it == 0 && __builtin_expect(__ballot(!solved) != 0ull, 0)) last_greedy_coefficient();
      AMQ_PHASE(marks, 5 + 4 * it);
      kind = code_table_kind<K>(alpha, ct);
      AMQ_PHASE(marks, 6 + 4 * it);
      if (it + 1 == T) break;
      double c[4 * ((NT + NTW + 3) / 4)];
#pragma unroll
      for (int t = 0; t < NT + NTW; ++t) c[t] = 0.0;
#pragma unroll
      for (int j = 0; j < NJ; ++j)
#pragma unroll
        for (int t = 0; t < NT; ++t) {
          const double m = one_if(u[j] >= ct.thr[t]);
          c[t] = __builtin_fma(wd[j], m, c[t]);
          c[NT + t / 3] = __builtin_fma(m, field[t % 3], c[NT + t / 3]);
        }
      AMQ_PHASE(marks, 7 + 4 * it);
      if constexpr (K == 4) {
        // four plane sums instead of seven C_t through the reduction (this lane's shares, without sum |w|)
        double sp[8];
        double ct7[NT];
#pragma unroll
        for (int t = 0; t < NT; ++t) ct7[t] = c[t];
#pragma unroll
        for (int i = 0; i < K; ++i) sp[i] = plane_dot<NT>(ct.bm[i], 0.0, ct7);
#pragma unroll
        for (int i = 0; i < NTW; ++i) sp[K + i] = c[NT + i];
        exchange_raw<NW, K + NTW>(sp, sh, phase);
        int cn[3 * NTW];
#pragma unroll
        for (int i = 0; i < NTW; ++i) {
          const unsigned long long p = counts_of(sp, K + i);
#pragma unroll
          for (int k = 0; k < 3; ++k) cn[3 * i + k] = count_of(p, k);
        }
#pragma unroll
        for (int i = 0; i < K; ++i) q[i] = ((ct.bm[i] & 1u) ? l1 : -l1) + total_of(sp, i);
        int t0 = 0;
#pragma unroll
        for (int a = 0; a < K; ++a)
#pragma unroll
          for (int b = a + 1; b < K; ++b) {
            const unsigned xo = ct.bm[a] ^ ct.bm[b];
            int dd = (xo & 1u) ? n : 0;
#pragma unroll
            for (int t = 1; t <= NT; ++t) dd += step_at(xo, t) * cn[t - 1];
            g[t0++] = (double)(n - 2 * dd);
          }
      } else {
        exchange_raw<NW, NT + NTW>(c, sh, phase);
        const unsigned long long p = counts_of(c, NT);
        double cs[NT];
        int cn[NT];
#pragma unroll
        for (int t = 0; t < NT; ++t) {
          cs[t] = total_of(c, t);
          cn[t] = count_of(p, t);
        }
        if (__builtin_expect(kind < 2, 1)) {
          // (what the general form below gives for these two orders)
          if constexpr (K == 2) {
            q[1] = __builtin_fma(2.0, cs[0], -l1);
            g[0] = (double)(2 * cn[0] - n);
          } else {
            g[0] = (double)(2 * cn[1] - n);
            g[1] = (double)(2 * (cn[0] - cn[1] + cn[2]) - n);
            g[2] = (double)(n - 2 * (cn[0] - cn[2]));
            if (__builtin_expect(kind == 0, 1)) {
              q[0] = l1;
              q[1] = __builtin_fma(2.0, cs[1], -l1);
              q[2] = __builtin_fma(2.0, (cs[0] - cs[1]) + cs[2], -l1);
            } else {
              q[0] = __builtin_fma(2.0, cs[0], -l1);
              q[1] = __builtin_fma(2.0, cs[1] - cs[0], l1);
              q[2] = __builtin_fma(2.0, cs[2] - cs[1], l1);
            }
          }
          if constexpr (K == 2) q[0] = l1;
        } else {
#pragma unroll
          for (int i = 0; i < K; ++i) q[i] = plane_dot<NT>(ct.bm[i], (ct.bm[i] & 1u) ? l1 : -l1, cs);
          int t0 = 0;
#pragma unroll
          for (int a = 0; a < K; ++a)
#pragma unroll
            for (int b = a + 1; b < K; ++b) {
              const unsigned xo = ct.bm[a] ^ ct.bm[b];
              int dd = (xo & 1u) ? n : 0;
#pragma unroll
              for (int t = 1; t <= NT; ++t) dd += step_at(xo, t) * cn[t - 1];
              g[t0++] = (double)(n - 2 * dd);
            }
        }
      }
    }

    // ---- the last pass in one of the usual orders: the planes of a slot from the signs of u - threshold and of w,
    // straight into the slot's lane
    auto put_plane = [&](int i, int j, int sign) { keep_in_lane(mym[i], __ballot(sign < 0), j); };
    if constexpr (K == 2) {
      if (__builtin_expect(kind == 0, 1)) {
        mym[0] = mym[1] = 0ull;
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
          const int w = __float_as_int(xc[j]);
          put_plane(0, j, ~w);
          put_plane(1, j, ~(w ^ (u[j] - ct.thr[0])));
        }
        mym[0] &= lane_inside;
        mym[1] &= lane_inside;
        return;
      }
    }
    if constexpr (K == 3) {
      if (__builtin_expect(kind == 0, 1)) {
        mym[0] = mym[1] = mym[2] = 0ull;
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
          const int w = __float_as_int(xc[j]), u1 = u[j] - ct.thr[0], u2 = u[j] - ct.thr[1], u3 = u[j] - ct.thr[2];
          put_plane(0, j, ~w);
          put_plane(1, j, ~(w ^ u2));
          put_plane(2, j, ~(w ^ u1 ^ u2 ^ u3));
        }
#pragma unroll
        for (int i = 0; i < K; ++i) mym[i] &= lane_inside;
        return;
      }
    }

    // ---- the last pass: the comparison masks, slot j in lane j, then the planes in the lanes
    unsigned long long ge[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) ge[t] = 0ull;
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
      for (int t = 0; t < NT; ++t) keep_in_lane(ge[t], __ballot(u[j] >= ct.thr[t]), j);
    const unsigned long long lane_neg = signs_in_lanes();
#pragma unroll
    for (int i = 0; i < K; ++i) {
      unsigned long long p = lane_neg ^ (0ull - (unsigned long long)(ct.bm[i] & 1u));
#pragma unroll
      for (int t = 1; t <= NT; ++t)
        p ^= ge[t - 1] & (0ull - (unsigned long long)(((ct.bm[i] >> t) ^ (ct.bm[i] >> (t - 1))) & 1u));
      mym[i] = p & lane_inside;
    }
    AMQ_PHASE(marks, 11);
  }
}

// Workgroup barriers that quantize_core passes (for waves of the workgroup that take no part in it).
template <int K>
__device__ __forceinline__ int quantize_exchanges(int T) {
  return K == 1 ? 1 : K + (T > 1 ? T - 1 : 0);
}

// The same for a wave that may or may not have all its slots inside the vector (a wave-uniform choice; the
// waves of a workgroup meet at the same barriers either way).
// ONLINE: the latency-bound form.
// RECON (throughput form): recon[j] receives the value of this lane's code in slot j instead of codes in mym.
template <int K, int NJ, int NW, bool ONLINE, bool RECON = false>
__device__ __forceinline__ void quantize_core(const float (&x)[NJ], int n, int base, int nj, int T, float (&alpha)[K],
                                              unsigned long long (&mym)[K], double* sh, int& phase,
                                              unsigned long long* marks = nullptr, float* recon = nullptr) {
  static_assert(!(ONLINE && RECON), "the latency form leaves codes");
  base = __builtin_amdgcn_readfirstlane(base);
  const bool full = nj == NJ && (base + NJ) * 64 <= n;
  if constexpr (ONLINE) {
    if (full) quantize_online<K, NJ, NW, NJ>(x, n, base, nj, T, alpha, mym, sh, phase, marks);
    else if (NW == 1 && nj == NJ && (NJ - 1) * 64 <= n)
      quantize_online<K, NJ, NW, NW == 1 ? NJ - 1 : 0>(x, n, base, nj, T, alpha, mym, sh, phase, marks);
    else quantize_online<K, NJ, NW, 0>(x, n, base, nj, T, alpha, mym, sh, phase, marks);
  } else if (full) {
    quantize_magnitudes<K, NJ, NW, NJ, RECON>(x, n, base, nj, T, alpha, mym, sh, phase, marks, recon);
  } else {
    // a single wave usually takes the form of its own number of slots, one of the even ones (beyond 16 every fourth): only
    // the last two (four) can be short
    constexpr int kLast = NJ > 16 ? 4 : 2;
    if (NW == 1 && (NJ - kLast) * 64 < n)
      quantize_magnitudes<K, NJ, NW, NW == 1 ? NJ - kLast : 0, RECON>(x, n, base, nj, T, alpha, mym, sh, phase, marks, recon);
    else
      quantize_magnitudes<K, NJ, NW, 0, RECON>(x, n, base, nj, T, alpha, mym, sh, phase, marks, recon);
  }
}

}  // namespace amq
