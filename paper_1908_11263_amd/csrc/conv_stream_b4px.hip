// 4-bit convolution: instantiations of the streaming implicit-GEMM kernel
// (int8 matrix cores), packed input tiles, pixels that are no whole number of
// 64-byte staged blocks.
#include "conv_stream_impl.h"

namespace qnn {

hipError_t launch_conv_stream_b4px(const StreamArgs &a, int variant, hipStream_t s)
{
    return launch_conv_stream_bits<4, 1, true>(a, variant, s);
}

}  // namespace qnn
