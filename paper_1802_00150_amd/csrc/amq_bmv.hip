// Small-batch binary matrix-vector products (amq_bmv_body.h) on quantized operands: instantiations and launch rules.
#include <atomic>

#include "amq_bmv_body.h"

namespace amq {

namespace {

template <int KW, int KA, int NSEG, int NBLK, int EPI, bool LSE = false>
__global__ __launch_bounds__(256) void bmv_kernel(BmvArgs a) {
  extern __shared__ uint4 xs[];
  bmv_body<KW, KA, NSEG, NBLK, EPI, LSE, false>(a, xs, nullptr, nullptr);
}

// Waves of a plain product that the chip holds at once, asked once per form (one kind of chip is built for).
template <int KW, int KA, int NSEG>
long long resident_waves() {
  static std::atomic<long long> known{0};
  long long waves = known.load(std::memory_order_relaxed);
  if (waves == 0) {
    int dev = 0, units = 0, blocks = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&units, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        hipOccupancyMaxActiveBlocksPerMultiprocessor(
            &blocks, reinterpret_cast<const void*>(&bmv_kernel<KW, KA, NSEG, 1, kEpiStore, false>), 256, 0) != hipSuccess) {
      (void)hipGetLastError();  // (only the split depends on it)
    }
    waves = 4LL * (units > 0 ? units : 256) * (blocks > 0 ? blocks : 4);
    known.store(waves, std::memory_order_relaxed);
  }
  return waves;
}

template <int KW, int KA, int NSEG, int NBLK, int EPI>
hipError_t launch_one(BmvArgs a, long long waves, size_t lds, hipStream_t s, int* lse_slots) {
  const long long blocks = (waves + 3) / 4;
  const dim3 grid((unsigned)blocks, (unsigned)a.groups);
  // every wave that owns at least one row fills one slot per batch entry
  if (a.lse_part && (waves > kLseMaxSlots || waves > a.lse_cap || a.groups != 1)) a.lse_part = nullptr;
  a.lse_slots = (int)waves;
  if (lse_slots) *lse_slots = a.lse_part ? (int)waves : 0;
  if constexpr (EPI == kEpiStore) {
    if (a.lse_part) {
      hipLaunchKernelGGL((bmv_kernel<KW, KA, NSEG, NBLK, EPI, true>), grid, dim3(256), lds, s, a);
      return hipGetLastError();
    }
  }
  hipLaunchKernelGGL((bmv_kernel<KW, KA, NSEG, NBLK, EPI, false>), grid, dim3(256), lds, s, a);
  return hipGetLastError();
}

template <int KW, int KA>
hipError_t launch_epi(const BmvArgs& a, int epi, hipStream_t s, int* lse_slots) {
  const int R = 64 >> a.lg;
  size_t lds = 0;
  const int nblk = (epi == kEpiStore) ? 1 : 2;
  for (int k = 0; k < nblk; ++k) lds += (size_t)KA * a.batch * ((a.blk[k].n + 127) / 128) * 16;
  switch (epi) {
    case kEpiStore: {
      // One row group per wave.  From where that is more waves than the chip holds (8192; `waves4` is a quarter of them): four
      // (all loads in flight) for products read from memory and groups of them, where the pairs of a log-softmax are left (one
      // group would leave more of them than fit), and for 1-bit weights, whose waves have little else to hide their start with
      // (42000 x 4096 W1/A1 batch 2 6.0 us, 6.9 with one).  One vector, and two with 2-bit weights and 1-bit activations (34000 x 4096 7.4,
      // 8.0 with one): two, unless they take more rounds of resident waves (42000 x 2500 W2/A1 5.6 / 6.0); W4/A4 always (25000 x 4096
      // 13.8, 14.8 with four).
      // With several vectors a wave is bound by its own arithmetic, and one group (41 to 65 registers) leaves room for twice the waves
      // of four.  us per product, four groups / two / one: 20000 x 4096 W2/A2 batch 1 4.8 / 4.2 / 4.5, W3/A3 6.7 / 5.9 / 6.5, batch 3
      // 13.1 / 10.9 / 11.0, batch 12 40.6 / 32.8 / 30.5; 42000 x 4096 W3/A3 batch 12 75 / 67 / 60; 25000 x 4096 W4/A1 batch 1 10.8 / 9.8 / -; 42000 x 2048 W3/A3
      // batch 1 (5250 waves of two groups) 6.5 / 7.0; below, 10000 x 4096 W2/A2 4.1 / 3.5 / 3.25.
      const long long waves4 = (a.m + 4LL * R - 1) / (4LL * R), waves2 = (a.m + 2LL * R - 1) / (2LL * R);
      if (waves4 * a.groups >= 2048) {
        if (KW == 1 || a.streaming || a.groups > 1 || a.lse_part) return launch_one<KW, KA, 4, 1, kEpiStore>(a, waves4, lds, s, lse_slots);
        if constexpr (KW > 1) {
          if (a.batch == 1 || (KW * KA == 2 && a.batch == 2)) {
            const long long of2 = resident_waves<KW, KA, 2>(), of4 = resident_waves<KW, KA, 4>();
            if (KW * KA < 16 && (waves2 + of2 - 1) / of2 > (waves4 + of4 - 1) / of4)
              return launch_one<KW, KA, 4, 1, kEpiStore>(a, waves4, lds, s, lse_slots);
            return launch_one<KW, KA, 2, 1, kEpiStore>(a, waves2, lds, s, lse_slots);
          }
        }
      }
      return launch_one<KW, KA, 1, 1, kEpiStore>(a, (a.m + R - 1) / R, lds, s, lse_slots);
    }
    case kEpiLstm: return launch_one<KW, KA, 4, 2, kEpiLstm>(a, (a.H + R - 1) / R, lds, s, nullptr);
    case kEpiGru: return launch_one<KW, KA, 3, 2, kEpiGru>(a, (a.H + R - 1) / R, lds, s, nullptr);
  }
  return hipErrorInvalidValue;
}

template <int KW>
hipError_t launch_ka(const BmvArgs& a, int k_a, int epi, hipStream_t s, int* lse_slots) {
  switch (k_a) {
    case 1: return launch_epi<KW, 1>(a, epi, s, lse_slots);
    case 2: return launch_epi<KW, 2>(a, epi, s, lse_slots);
    case 3: return launch_epi<KW, 3>(a, epi, s, lse_slots);
    case 4: return launch_epi<KW, 4>(a, epi, s, lse_slots);
  }
  return hipErrorInvalidValue;
}

}  // namespace

bool bmv_supported(int n0, int n1, int k_a, long long batch, int epi) {
  const int c0 = (n0 + 127) / 128, c1 = (n1 + 127) / 128;
  const bool fp4 = n0 <= 1024 && n1 <= 1024;  // the fp4 matrix-core kernels are the alternative
  const int limit = !fp4 ? kBmvMaxBatch : epi == kEpiStore ? kBmvMaxBatchStore : kBmvMaxBatchCell;
  if (c0 > 64 || c1 > 64 || batch > limit) return false;
  return (size_t)k_a * batch * (c0 + c1) * 16 <= 48 * 1024;
}

hipError_t launch_bmv(BmvArgs a, int k_w, int k_a, int epi, hipStream_t s, int* lse_slots) {
  if (lse_slots) *lse_slots = 0;
  if (epi != kEpiStore) a.lse_part = nullptr;
  int nmax = a.blk[0].n;
  if (epi != kEpiStore && a.blk[1].n > nmax) nmax = a.blk[1].n;
  const int cpr = (nmax + 127) / 128;
  int lg = 0;
  while ((1 << lg) < cpr) ++lg;
  a.lg = lg;
  {
    long long plane_bytes = (long long)k_w * a.m * ((a.blk[0].n + 127) / 128) * 16;
    if (epi != kEpiStore) plane_bytes += (long long)k_w * a.m * ((a.blk[1].n + 127) / 128) * 16;
    a.streaming = plane_bytes * a.groups > kBmvStreamingBytes;
  }
  switch (k_w) {
    case 1: return launch_ka<1>(a, k_a, epi, s, lse_slots);
    case 2: return launch_ka<2>(a, k_a, epi, s, lse_slots);
    case 3: return launch_ka<3>(a, k_a, epi, s, lse_slots);
    case 4: return launch_ka<4>(a, k_a, epi, s, lse_slots);
  }
  return hipErrorInvalidValue;
}

}  // namespace amq
