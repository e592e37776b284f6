// 4-bit convolution: instantiations of the streaming implicit-GEMM kernel
// (int8 matrix cores), pixels that are narrow or no whole number of 16-byte items.
#include "conv_stream_impl.h"

namespace qnn {

hipError_t launch_conv_stream_b4x(const StreamArgs &a, int variant, hipStream_t s)
{
    return launch_conv_stream_bits<4, 1>(a, variant, s);
}

}  // namespace qnn
