// 1-bit convolution: instantiations of the streaming implicit-GEMM kernel
// (e2m1 matrix instruction).
#include "conv_stream_impl.h"

namespace qnn {

hipError_t launch_conv_stream_b1(const StreamArgs &a, int variant, hipStream_t s)
{
    return launch_conv_stream_bits<1, 0>(a, variant, s);
}

}  // namespace qnn
