// Matrix-core path: convolution instantiations with one packed word per lane and load, for a streamed residual.
#include "bnn_mfma_kernel.h"

namespace bnn {

int launch_mfma_conv_v1_stream(const uint32_t* A, const uint32_t* B, const Geom& g, const Epi& e, hipStream_t s) {
    if (g.tw % 2 == 0) return mfma::launch_shape<1, true, false, mfma::KIND_STREAM>(A, B, g, e, s);
    return mfma::launch_shape<1, true, true, mfma::KIND_STREAM>(A, B, g, e, s);
}

}  // namespace bnn
