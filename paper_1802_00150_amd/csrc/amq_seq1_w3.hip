// Batch-1 sequences in one launch: the forms with 3-bit weights (amq_seq1_body.h).
#include "amq_seq1_body.h"

namespace amq {

hipError_t launch_seq1_w3(const Seq1Args& a, int k_a, int epi, hipStream_t s) { return seq1::run_weights<3>(a, k_a, epi, s); }

}  // namespace amq
