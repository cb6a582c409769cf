// Large plain products on the 32 x 32 form of the fp4 matrix instruction (amq_mfma32_body.h): the rule of when they
// apply, and the 2-bit-weight instantiations (those with 3-bit weights are in amq_mfma32_w3.hip).
#include "amq_mfma32_body.h"

namespace amq {

hipError_t launch_mfma32_w3(const BmvArgs& a, int k_a, hipStream_t s, int* lse_slots);

// Plain products (no integer hook) of 2- and 3-bit codes and vectors whose staged planes fit LDS; sizes whose element
// offsets fit 32 bits.  The lines, all measured:
//   - vectors above 1024 entries: from batch 17 on the alternative is the int8 kernel, which takes 1.3 to 2.7 times as
//     long; at 9 .. 16 it is the small-batch kernel, whose time grows with the batch (equal at 10000 x 1500 and batch 8);
//   - of 769 .. 1024 entries (8 pieces per row) the kernel with 16 x 16 tiles wastes nothing either and cuts the work finer, so
//     what decides is how many tasks the SIMD with the most has in either form, and there has to be a task for every SIMD.
//     Six plane products take 0.65 us per 32 x 32 x 1/4 here and 0.7 there: ahead where that SIMD has no more to do (16 x 16 /
//     32 x 32, us: 10000 x 1024 W2/A3 batch 128 9.0 / 8.4, 256 12.8 / 10.8, 4096 x 1024 batch 1024 15.1 / 14.6, 42000 x 1024
//     batch 64 13.1 / 10.9, but batch 32 7.6 / 9.0, 48 9.7 / 11.3 and 16000 x 1024 batch 128 14.1 / 10.0, 129 10.0 / 11.4).
//     Nine (0.88 and 0.97): from two and a half tasks per SIMD on if the one with the most has no more than five quarters of
//     the average (10000 x 1024 batch 128 8.8 / 9.7, 256 12.5 / 13.0, 300 16.4 / 17.8, 512 22.0 / 20.8, 42000 x 1024 batch 64
//     14.8 / 13.0; on the wrong side of it: 16000 x 1024 batch 224 17.0 / 18.2).  Four: from eight, and never where outputs are written (10000 x 1024 batch 512 12.3 / 13.5);
//   - shorter ones: the 16 x 16 kernel always contracts 1024 positions; from one task per SIMD.
bool mfma32_supported(const BmvArgs& a, int k_w, int k_a) {
  using namespace mfma32;
  if (a.D || a.groups > 1 || k_w < 2 || k_w > 3 || k_a < 2 || k_a > 3) return false;
  if (!a.Y && !(a.tgt && a.tgt_out && a.lse_part && a.lse_cap >= 256)) return false;
  if (a.batch <= 8 || lds_bytes(k_w, k_a, 1, a.blk[0].n) > kMaxLds) return false;
  if (a.m * ((a.blk[0].n + 127) / 128) * k_w >= (1LL << 31)) return false;  // weight offsets in 16-byte units
  if ((long long)a.batch * a.m >= (1LL << 31)) return false;
  if (a.blk[0].n > 1024) return a.batch > kBmvMaxBatch || (a.m >= 8192 && a.blk[0].n <= 2048);
  const long long tasks = (a.m + kTileN - 1) / kTileN * ((a.batch + kTileN - 1) / kTileN);
  const int products = k_w * k_a;
  if (half_pieces(a.blk[0].n) == kStaticPieces) {
    if (products == 4) return !a.Y && tasks >= 8192;
    const int rowblocks = (int)((a.m + kTileN - 1) / kTileN), groups = (a.batch + kTileN - 1) / kTileN;
    const int most = (blocks_each(rowblocks, groups) + 3) / 4, other = mfma4w_most_tasks(a, k_w, k_a);
    if (products == 6) return a.batch > 16 && tasks >= 1100 && (other == 0 || other >= 4 * most);
    return a.batch > 16 && tasks >= 2600 && 5 * tasks >= 4 * 1024LL * most;
  }
  return a.batch > 16 && tasks >= 1024;
}

hipError_t launch_mfma32(const BmvArgs& a, int k_w, int k_a, hipStream_t s, int* lse_slots) {
  if (lse_slots) *lse_slots = 0;
  if (k_w == 3) return launch_mfma32_w3(a, k_a, s, lse_slots);
  return k_a == 2 ? mfma32::launch_tiles<2, 2>(a, s, lse_slots) : mfma32::launch_tiles<2, 3>(a, s, lse_slots);
}

}  // namespace amq
