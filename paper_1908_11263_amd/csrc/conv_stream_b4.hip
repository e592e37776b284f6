// 4-bit convolution: instantiations of the streaming implicit-GEMM kernel
// (int8 matrix cores).
#include "conv_stream_impl.h"

namespace qnn {

hipError_t launch_conv_stream_b4(const StreamArgs &a, int variant, hipStream_t s)
{
    return launch_conv_stream_bits<4, 0>(a, variant, s);
}

}  // namespace qnn
