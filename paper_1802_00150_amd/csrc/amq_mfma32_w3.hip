// The 3-bit-weight instantiations of the large plain products (amq_mfma32_body.h).
#include "amq_mfma32_body.h"

namespace amq {

hipError_t launch_mfma32_w3(const BmvArgs& a, int k_a, hipStream_t s, int* lse_slots) {
  return k_a == 2 ? mfma32::launch_tiles<3, 2>(a, s, lse_slots) : mfma32::launch_tiles<3, 3>(a, s, lse_slots);
}

}  // namespace amq
