// 2-bit convolution: instantiations of the streaming implicit-GEMM kernel
// (e2m1 matrix instruction), pixels that are narrow or no whole number of 16-byte items.
#include "conv_stream_impl.h"

namespace qnn {

hipError_t launch_conv_stream_b2x(const StreamArgs &a, int variant, hipStream_t s)
{
    return launch_conv_stream_bits<2, 1>(a, variant, s);
}

}  // namespace qnn
