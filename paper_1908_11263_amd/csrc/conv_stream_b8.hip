// 8-bit convolution: instantiations of the streaming implicit-GEMM kernel
// (int8 matrix cores).
#include "conv_stream_impl.h"

namespace qnn {

hipError_t launch_conv_stream_b8(const StreamArgs &a, int variant, hipStream_t s)
{
    return launch_conv_stream_bits<8, 0>(a, variant, s);
}

}  // namespace qnn
