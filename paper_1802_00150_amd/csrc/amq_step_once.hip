// A recurrent step of a small batch in one launch (Eq. 6): quantization of x_t and h_{t-1}, products, cell.
//
// Two launches (quantizer, then products and cell) cost a launch each on the host (2.3 us) and, on the device, the gap between
// dependent kernels, the second kernel's start and the cold fetch of its weights, one after the other.  Here the first workgroups of
// the grid quantize, one batch entry's two vectors each, and the others (amq_pair_body.h: one batch tile and 4 row blocks each)
// fetch their weights, turn them into operand layout and then wait for the codes of their tile.  What is handed over are 8-byte
// {word, tag} pairs, one device-scope store each, polled until all that a lane needs carry the tag of the launch: the data is its own
// arrival signal.
//
// Whom a workgroup waits for comes before it in the grid and waits for nobody.  Should the chip be shared such that those
// workgroups get no room for longer than a wait takes (kHandOverPolls), the waiting workgroup quantizes the vectors of its tile
// itself: it needs nobody then, so results depend neither on the order of the workgroups nor on how many are resident.  The
// inputs are therefore read by workgroups that start late; the host takes this path only where no output overlaps them.
//
// The pairs live in memory of the library (a slot per launch, taken in turn), which is zero at first and is written by nobody else.  A
// tag is used again after 2^32 launches; all slots are cleared four times in between, so that an old pair is not taken for a new one.
// Should that, or as many later launches as there are slots, meet a slot that is still waited for, those waits end as above.  A captured
// launch would carry the same tag at every replay: there the step stays two launches.
//
// The arithmetic and its order are those of the two launches: the results are the same bit for bit.
#include <atomic>
#include <type_traits>

#include "amq_launch.h"
#include "amq_pair_body.h"
#include "amq_quantize_body.h"
#include "amq_seqw_body.h"

namespace amq {

namespace {

constexpr int kOnceWaves = 8;
constexpr unsigned kHandOverPolls = 64;  // about 40 us
constexpr int kHandOverSlots = 32;
constexpr int kSlotPairs = 8192;         // 64 KiB
constexpr unsigned kClearEvery = 1u << 30;
constexpr int kMostCycles = 4;
std::atomic<unsigned> next_tag{1};
static __device__ unsigned long long hand_over[kHandOverSlots][kSlotPairs];

struct OnceArgs {
  BmvArgs b;                 // raw[0], raw[1]: the inputs and the previous state
  // this launch's slot: vectors x_0 .. , then h_0 .., of each the words of its codes, plane by plane, then the coefficients
  unsigned long long* pairs;
  unsigned long long* awaited;  // where the codes are looked for: the same, or (test hook) a slot in which this tag never is
  unsigned tag, polls;
  int rowblocks, gx;         // gx: workgroups of a batch tile
};

__global__ __launch_bounds__(256) void clear_slots_kernel(unsigned long long* pairs) {
  put_pair(pairs + blockIdx.x * 256 + threadIdx.x, 0u, 0u);
}

// NC: stretches of 1024 entries of the longer operand block (1 or 2).  (The register bounds are such that nothing is spilled: a few
// bytes of scratch per lane cost 0.7 us here.)
template <int KW, int KA, int EPI, int NC>
__global__ __launch_bounds__(64 * kOnceWaves, NC == 1 && KW * KA <= 4 ? 4 : 2) void step_once_kernel(OnceArgs o) {
  constexpr int NW = kOnceWaves / 2;  // waves per vector
  constexpr int NJ = 4 * NC;          // slots per lane
  constexpr int kWords = 32 * NC;     // words of a row, padding included
  constexpr int kEntry = (KA * (kWords + 1) + 1) & ~1;  // codes and coefficients of a vector, written in 8-byte pieces
  static_assert(kEntry * sizeof(uint32_t) % sizeof(unsigned long long) == 0, "the second vector's codes are aligned too");
  __shared__ double sh[2][2 * kExchange<NW>];
  __shared__ __attribute__((aligned(8))) uint32_t codes[2][kEntry];
  __shared__ float4 xch[(kOnceWaves / 2) * 64];
  __shared__ int missed;
  extern __shared__ __attribute__((aligned(16))) uint4 turn[];
  const BmvArgs& a = o.b;
  asm volatile("" ::AMQ_ARG(a.blk[0].Wp), AMQ_ARG(a.blk[0].alpha), AMQ_ARG(a.blk[0].n), AMQ_ARG(a.blk[1].Wp),
               AMQ_ARG(a.blk[1].alpha), AMQ_ARG(a.blk[1].n), AMQ_ARG(a.m), AMQ_ARG(a.H), AMQ_ARG(a.batch), AMQ_ARG(a.bias0),
               AMQ_ARG(a.bias1), AMQ_ARG(a.c_prev), AMQ_ARG(a.h_prev), AMQ_ARG(a.h_out), AMQ_ARG(a.c_out), AMQ_ARG(a.raw[0]),
               AMQ_ARG(a.raw[1]), AMQ_ARG(a.T), AMQ_ARG(o.pairs), AMQ_ARG(o.awaited), AMQ_ARG(o.tag), AMQ_ARG(o.rowblocks), AMQ_ARG(o.gx));
  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int batch = a.batch;
  // (formed from the arguments at every use: as captured variables they are kept in memory)
  auto wpr = [&](int k) { return 4 * (((k ? a.blk[1].n : a.blk[0].n) + 127) >> 7); };
  auto vector_at = [&](unsigned long long* slot, int k, int entry) {
    return slot + (k ? batch * seqw_entry_pairs(KA, wpr(0)) + entry * seqw_entry_pairs(KA, wpr(1)) : entry * seqw_entry_pairs(KA, wpr(0)));
  };

  // The codes and coefficients of a batch entry's two vectors in LDS, a half of the waves each; ends with a barrier.
  auto quantize_entry = [&](int entry, int& phase) {
    const int k = wv / NW, n = k ? a.blk[1].n : a.blk[0].n, w = wpr(k);
    const int nslots = w >> 1, nj = (nslots + NW - 1) / NW, base = (wv & (NW - 1)) * nj;
    const float* const x = (k ? a.raw[1] : a.raw[0]) + (size_t)entry * n;
    float beta[KA];
    unsigned long long mym[KA];
    with_slots<NJ, true>(nj, [&](auto slots) {
      float v[slots()];
      load_slots<slots()>(x, n, base, nj, v);
      quantize_core<KA, slots(), NW, true>(v, n, base, nj, a.T, beta, mym, sh[k], phase);
    });
    if (lane < nj && base + lane < nslots) {
#pragma unroll
      for (int i = 0; i < KA; ++i) reinterpret_cast<unsigned long long*>(codes[k] + i * w)[base + lane] = mym[i];
    }
    if ((wv & (NW - 1)) == 0 && lane == 0) {
#pragma unroll
      for (int i = 0; i < KA; ++i) codes[k][KA * w + i] = __float_as_uint(beta[i]);
    }
    lds_barrier();
  };

  if ((int)blockIdx.x < batch) {
    // (ahead of the waiting waves of a workgroup beside it: 650 units batch 13 on two streams 3.84 -> 3.71 us per step)
    __builtin_amdgcn_s_setprio(3);
    int phase = 0;
    const int entry = blockIdx.x, k = wv / NW, t = tid & (64 * NW - 1);
    quantize_entry(entry, phase);
    const int w = wpr(k);
    if (t < KA * (w + 1)) put_pair(vector_at(o.pairs, k, entry) + t, codes[k][t], o.tag);
    return;
  }

  const int at = (int)blockIdx.x - batch, bx = at % o.gx, by = at / o.gx;
  const int b0 = by * kTileB, ncols = batch - b0 < kTileB ? batch - b0 : kTileB;
  if (tid == 0) missed = 0;
  auto stage = [&](uint4* image, int kb, float (&beta)[1]) {
    // thread -> word of a row (plane by plane, block by block) and batch column: adjacent lanes, adjacent pairs
    constexpr int kColsPer = 64 * kOnceWaves / kWords, kColReq = kTileB / kColsPer;
    const int gw = tid & (kWords - 1), gc = tid / kWords;
    const int dst = ((gw >> 5) * kSteps + 4 * ((gw >> 4) & 1) + (gw & 3)) * 64 + 16 * ((gw >> 2) & 3);
    const int swz = (((gw >> 2) & 3) << 1) | (((gw >> 4) & 1) << 3);
    auto place = [&](int k, int j, int col, uint32_t word) {
      image[(k * KA + j) * NC * kSteps * 64 + dst + (col ^ swz)] = expand4_signed(word);
    };
    const int l16 = lane & 15, l4 = lane >> 4, plane = l4 < KA ? l4 : KA - 1;
    lds_barrier();  // (missed is set)
    unsigned long long v[2][KA][kColReq], bv;
    unsigned spins = 0;
    for (;;) {
      bv = get_pair(vector_at(o.awaited, kb, b0 + (l16 < ncols ? l16 : ncols - 1)) + KA * wpr(kb) + plane);
#pragma unroll
      for (int k = 0; k < 2; ++k)
#pragma unroll
        for (int q = 0; q < kColReq; ++q) {
          const int col = q * kColsPer + gc;
          // (columns past the batch and words past the row are not asked for)
#pragma unroll
          for (int j = 0; j < KA; ++j) v[k][j][q] = (unsigned long long)o.tag << 32;
          if (col < ncols && gw < wpr(k)) {
            const unsigned long long* const from = vector_at(o.awaited, k, b0 + col) + gw;
#pragma unroll
            for (int j = 0; j < KA; ++j) v[k][j][q] = get_pair(from + j * wpr(k));
          }
        }
      bool ready = (unsigned)(bv >> 32) == o.tag;
#pragma unroll
      for (int k = 0; k < 2; ++k)
#pragma unroll
        for (int j = 0; j < KA; ++j)
#pragma unroll
          for (int q = 0; q < kColReq; ++q) ready = ready && (unsigned)(v[k][j][q] >> 32) == o.tag;
      if (__all(ready)) break;
      if (++spins >= o.polls) {
        missed = 1;
        break;
      }
    }
#pragma unroll
    for (int k = 0; k < 2; ++k)
#pragma unroll
      for (int j = 0; j < KA; ++j)
#pragma unroll
        for (int q = 0; q < kColReq; ++q)
          place(k, j, q * kColsPer + gc, gw < wpr(k) ? (uint32_t)(v[k][j][q] & 0xffffffffull) : 0u);
    beta[0] = __uint_as_float((unsigned)(bv & 0xffffffffull));
    lds_barrier();
    if (__builtin_expect(__builtin_amdgcn_readfirstlane(missed) != 0, 0)) {
      // the tile's vectors by this workgroup, entry after entry
      int phase = 0;
      for (int col = 0; col < ncols; ++col) {
        quantize_entry(b0 + col, phase);
        for (int t = tid; t < 2 * KA * kWords; t += 64 * kOnceWaves) {  // (whole rounds: kWords is the word's period)
          const int k = t / (KA * kWords), j = t / kWords % KA;
          place(k, j, col, gw < wpr(k) ? codes[k][j * wpr(k) + gw] : 0u);
        }
        if (l16 == col) beta[0] = __uint_as_float(codes[kb][KA * wpr(kb) + plane]);
        lds_barrier();
      }
    }
  };
  pair_body<KW, KA, 1, EPI, kOnceWaves, kPairBoth, NC>(a, o.rowblocks, bx, by, turn, xch, stage);
}

template <int KW, int KA, int EPI, int NC>
hipError_t run_one(const OnceArgs& o, int grid, hipStream_t s) {
  constexpr size_t lds = pair_body_lds<KW, KA, 1, kOnceWaves, kPairBoth, NC>();
  static std::atomic<unsigned long long> configured{0};
  hipError_t e = ensure_dynamic_lds(reinterpret_cast<const void*>(&step_once_kernel<KW, KA, EPI, NC>), (int)lds, configured);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((step_once_kernel<KW, KA, EPI, NC>), dim3((unsigned)grid), dim3(64 * kOnceWaves), lds, s, o);
  return hipGetLastError();
}

template <int KW, int KA>
hipError_t run_k(const OnceArgs& o, int grid, int epi, int nc, hipStream_t s) {
  if (epi == kEpiLstm) return nc == 1 ? run_one<KW, KA, kEpiLstm, 1>(o, grid, s) : run_one<KW, KA, kEpiLstm, 2>(o, grid, s);
  return nc == 1 ? run_one<KW, KA, kEpiGru, 1>(o, grid, s) : run_one<KW, KA, kEpiGru, 2>(o, grid, s);
}

// The slot memory of the current device and its compute units, looked up once per device (null: not to be had).
unsigned long long* hand_over_memory(int& units) {
  struct Device {
    std::atomic<void*> memory;
    std::atomic<int> units;
  };
  static Device known[64];
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return nullptr;
  void* p = known[dev].memory.load(std::memory_order_acquire);
  if (p) {
    units = known[dev].units.load(std::memory_order_relaxed);
  } else {
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(hand_over)) != hipSuccess ||
        hipDeviceGetAttribute(&units, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) {
      (void)hipGetLastError();
      return nullptr;
    }
    known[dev].units.store(units, std::memory_order_relaxed);
    known[dev].memory.store(p, std::memory_order_release);
  }
  return static_cast<unsigned long long*>(p);
}

int row_groups(const BmvArgs& a) { return (int)(((a.H + 3) / 4 + kOnceWaves / 2 - 1) / (kOnceWaves / 2)); }
long long workgroups(const BmvArgs& a) { return a.batch + (long long)row_groups(a) * ((a.batch + kTileB - 1) / kTileB); }

}  // namespace

// Shapes of the paired kernel, 2- and 3-bit weights and 2-bit activations, as long as the workgroups are few.  The quantizing ones carry
// the registers and the LDS of the whole step: on several busy streams they find waiting workgroups of other steps beside them,
// where the quantizer by itself fits anywhere.  Two launches / one, us per LSTM step on one stream, and per step of two and four streams
// that work is queued on; h_t becomes h_{t-1} of the next step:
//   W2/A2 300 units batch 8 (27 workgroups) 6.83 / 6.45, 3.59 / 3.41, 2.01 / 1.87; 650 batch 13 (54) 7.45 / 7.27, 4.02 / 4.07, 2.23 / 2.26;
//   beyond, 1024 batch 16 (80) 7.49 / 7.55, 4.03 / 4.36, 2.27 / 2.49; W3/A2 the same 8.05 / 7.91, 4.34 / 4.54, 2.49 / 2.64.
// Up to four entries have fewer such encounters: 1024 batch 4 (68) W2/A2 7.27 / 6.82, 3.88 / 3.80, 2.16 / 2.04; beyond, 1500 batch 4 (98)
// 8.60 / 8.36, 4.47 / 4.37, 2.49 / 2.65, 2048 batch 4 (132) 9.02 / 8.87, 4.72 / 4.97, 2.96 / 3.90.
// Vectors of up to 512 entries are quantized in less time, and 3-bit weights take longer to turn meanwhile: 200 units batch 48 (87)
// W2/A2 7.31 / 7.00, 3.95 / 3.93, 2.19 / 2.17, W3/A2 256 batch 56 (120) 7.65 / 7.19, 4.23 / 4.12, 2.34 / 2.31; beyond, W2/A2 512 batch 32
// (96) 6.96 / 6.81, 3.86 / 4.02, 2.15 / 2.23, W3/A2 512 batch 40 (136) 7.43 / 7.16, 4.22 / 4.27, 2.35 / 2.37.
// 3-bit activations are quantized slower here than by themselves, which longer vectors and 2-bit weights do not make up for: 650 units batch
// 13 (54) W3/A3 9.08 / 9.31, 4.76 / 4.81, 2.71 / 2.60, 300 batch 16 (35) W2/A3 7.85 / 8.04, 4.15 / 4.14, 2.29 / 2.21, W3/A3 8.32 / 8.33, 4.40 /
// 4.28, 2.39 / 2.28, 512 batch 8 (40) 8.05 / 7.81, 4.22 / 4.01, 2.32 / 2.14.  (One that is waited for 19.3 / 19.5.)
// What the host saves, a launch of 2.3 us, is in none of these: a program that feeds two or more streams from one thread takes 12.3 to
// 13.3 us per step in two launches and 10.2 to 11.0 in one.
bool step_once_supported(const BmvArgs& a, int k_w, int k_a, int epi, hipStream_t s) {
  // Cycles of the quantizer beyond the usual two: four waves per vector beside the workgroups that wait take 0.44 (2 bits) to 0.78 us
  // (3 bits, 1024 entries) per cycle, the quantizer by itself 0.36 and 0.58.  Two launches / one, W2/A2, us, T = 2, 4, 6, 10, 20: 300
  // units batch 4 6.5 / 6.1, 7.2 / 6.9, 7.9 / 7.75, 9.4 / 9.4, 13.0 / 13.7; 650 batch 13 7.0 / 6.8, 7.8 / 7.7, 8.6 / 8.6, 10.3 / 10.4,
  // 14.3 / 15.0.  From about 40 on the waits give up before the codes are there, and every workgroup quantizes its tile: 650 batch 13
  // T = 100 47 / 631.  3-bit activations have no lead to lose.
  if (a.T > (k_a == 2 ? kMostCycles : 2)) return false;
  if (a.batch < 2 || k_w < 2 || k_w > 3 || !a.raw[0] || !a.raw[1]) return false;
  const bool shorter = a.blk[0].n <= 512 && a.blk[1].n <= 512;
  if (k_a != 2 && !(k_a == 3 && k_w == 3 && shorter)) return false;
  if (!mfma4_pair_supported(a, k_w, k_a, epi) || mfma32_cell_supported(a, k_w, k_a, epi)) return false;
  long long pairs = 0;
  for (const BmvBlock& k : a.blk) pairs += (long long)a.batch * seqw_entry_pairs(k_a, 4 * ((k.n + 127) >> 7));
  int units = 0;
  const int most = shorter ? (k_w == 3 && k_a == 2 ? 15 : 11) : a.batch <= 4 ? 12 : 7;  // workgroups per 32 units
  if (pairs > kSlotPairs || !hand_over_memory(units) || 32 * workgroups(a) > most * units) return false;
  return !maybe_captured(s);
}

unsigned step_once_launches(long long next) {
  return next < 0 ? next_tag.load(std::memory_order_relaxed) : next_tag.exchange((unsigned)next, std::memory_order_relaxed);
}

hipError_t launch_step_once(const BmvArgs& a, int k_w, int k_a, int epi, hipStream_t s) {
  int units = 0;
  unsigned long long* const memory = hand_over_memory(units);
  if (!memory) return hipErrorInvalidValue;
  OnceArgs o{};
  o.b = a;
  AMQ_PHASE_ATTACH(o.b);
  do {
    o.tag = next_tag.fetch_add(1, std::memory_order_relaxed);
    if (o.tag % kClearEvery == 0u) {
      static_assert(kHandOverSlots * kSlotPairs % 256 == 0, "whole workgroups");
      hipLaunchKernelGGL(clear_slots_kernel, dim3(kHandOverSlots * kSlotPairs / 256), dim3(256), 0, s, memory);
      const hipError_t e = hipGetLastError();
      if (e != hipSuccess) return e;
    }
  } while (o.tag == 0u);  // (0 is what cleared slots hold)
  o.pairs = memory + (size_t)(o.tag % kHandOverSlots) * kSlotPairs;
  o.polls = sequence_spin_limit() < kHandOverPolls ? sequence_spin_limit() : kHandOverPolls;
  o.awaited = o.polls > 1 ? o.pairs : memory + (size_t)((o.tag + 1) % kHandOverSlots) * kSlotPairs;
  o.rowblocks = (int)((a.H + 3) / 4);
  o.gx = row_groups(a);
  const int grid = (int)workgroups(a);
  const int nc = a.blk[0].n > 1024 || a.blk[1].n > 1024 ? 2 : 1;
  if (k_a == 3) return epi == kEpiLstm ? run_one<3, 3, kEpiLstm, 1>(o, grid, s) : run_one<3, 3, kEpiGru, 1>(o, grid, s);
  return k_w == 2 ? run_k<2, 2>(o, grid, epi, nc, s) : run_k<3, 2>(o, grid, epi, nc, s);
}

}  // namespace amq
