// Batch-1 sequences in one launch (amq_seq1_body.h): the rule of when, and the forms with 2-bit weights (those with 3-bit
// weights are in amq_seq1_w3.hip).
#include "amq_seq1_body.h"

namespace amq {

hipError_t launch_seq1_w3(const Seq1Args& a, int k_a, int epi, hipStream_t s);

bool seq1_supported(long long I, long long H, long long B, int k_w, int k_a) {
  return B == 1 && I > 0 && H > 0 && I <= 2048 && H <= 2048 && k_w >= 2 && k_w <= 3 && k_a >= 2 && k_a <= 3;
}

hipError_t launch_seq1(Seq1Args a, int k_w, int k_a, int epi, hipStream_t s) {
  if (a.steps > kSeqGMaxSteps || !seq1_supported(a.I, a.H, 1, k_w, k_a)) return hipErrorInvalidValue;
  const int cpr = ((a.I > a.H ? a.I : a.H) + 127) / 128;
  a.lg = 0;
  while ((1 << a.lg) < cpr) ++a.lg;
  a.limit = sequence_spin_limit();
  return k_w == 3 ? launch_seq1_w3(a, k_a, epi, s) : seq1::run_weights<2>(a, k_a, epi, s);
}

}  // namespace amq
