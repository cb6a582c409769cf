// The quantizer with the reconstruction as its output: w -> w_hat in one pass over memory (Sec. 4, the forward pass
// through quantized weights).  Against quantizing to packed codes and expanding those in a second launch this saves the
// launch and the reading of the codes; the stores hide behind the arithmetic.
#include "amq_quantize_kernels.h"

namespace amq {

hipError_t launch_quantize_recon(const QuantArgs& a, int k, hipStream_t s) { return launch_bits<true>(a, k, s); }

}  // namespace amq
