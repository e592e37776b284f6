// Max-pooling over packed unsigned codes and signed 8-bit ReLU (Sec. IV-A:
// ReLU is a max with zero, max-pooling the maximum over a window; both split
// over pixels across the parallel units, Sec. IV-B).
//
// Both are bound by HBM, so a lane takes 16 bytes: one load per window tap and
// one store (32-bit words where pixels are no whole number of 16 bytes).
// Measured on 128 images of 112x112x64 bytes, the ReLU and then the 3x3 /
// stride-2 pooling of its output: 100.7 us with one word per lane (2.3 TB/s),
// 51.0 us now (4.5 TB/s; a device copy reaches 5.1).
//
// Pooling compares the packed codes as they are: with everything above field s
// of each 16-bit half masked off, an unsigned 16-bit maximum orders the halves
// by field s first, so the field's bits of the running maximum are the maximum
// of the field (the bits below it only break ties).  One mask (none for the
// top field) and one packed maximum per field pair and tap, no shifts; the
// fields are put together once at the end.
#include "qnn_internal.h"

namespace qnn {

typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));

// workgroup i runs on XCD i mod 8: consecutive parts of the output on one XCD,
// so that overlapping windows find their rows in its L2
__device__ __forceinline__ uint32_t xcd_block()
{
    const uint32_t q = gridDim.x >> 3, r = gridDim.x & 7, x = blockIdx.x & 7;
    return x * q + min(x, r) + (blockIdx.x >> 3);
}

// W: 32-bit words per lane (4 or 1); K: square window of K x K taps known at
// compile time, or 0.
template <int BITS, int W, int K>
__global__ void __launch_bounds__(256) maxpool_kernel(PoolArgs a)
{
    constexpr int S = 16 / BITS;                   // field pairs per word
    const int idx = (int)(xcd_block() * 256 + threadIdx.x);
    if (idx >= a.total)
        return;
    const int pix = (int)fdiv((uint32_t)idx, a.div_pbd);
    const int d = idx - pix * a.pbd;
    const int q = (int)fdiv((uint32_t)pix, a.div_wo);
    const int ox = pix - q * a.wo;
    const int n = (int)fdiv((uint32_t)q, a.div_ho);
    const int oy = q - n * a.ho;
    typedef uint32_t vec __attribute__((ext_vector_type(W)));
    const vec *x = (const vec *)a.x + (((size_t)n * a.h + oy * a.sh) * a.w_ + ox * a.sw) * a.pbd + d;
    u16x2 best[W][S];
#pragma unroll
    for (int j = 0; j < W; ++j)
#pragma unroll
        for (int s = 0; s < S; ++s)
            best[j][s] = (u16x2){0, 0};
    auto take = [&](vec v) {
#pragma unroll
        for (int j = 0; j < W; ++j)
#pragma unroll
            for (int s = 0; s < S; ++s) {
                constexpr uint32_t ones = 0x00010001u;
                const uint32_t mask = (s + 1) * BITS == 16 ? ~0u : ((1u << ((s + 1) * BITS)) - 1u) * ones;
                best[j][s] = __builtin_elementwise_max(best[j][s], __builtin_bit_cast(u16x2, v[j] & mask));
            }
    };
    if constexpr (K > 0) {
        vec v[K][K];
#pragma unroll
        for (int ky = 0; ky < K; ++ky)
#pragma unroll
            for (int kx = 0; kx < K; ++kx)
                v[ky][kx] = x[((size_t)ky * a.w_ + kx) * a.pbd];
#pragma unroll
        for (int ky = 0; ky < K; ++ky)
#pragma unroll
            for (int kx = 0; kx < K; ++kx)
                take(v[ky][kx]);
    } else {
        for (int ky = 0; ky < a.kh; ++ky)
            for (int kx = 0; kx < a.kw; ++kx)
                take(x[((size_t)ky * a.w_ + kx) * a.pbd]);
    }
    vec out;
#pragma unroll
    for (int j = 0; j < W; ++j) {
        uint32_t o = 0;
#pragma unroll
        for (int s = 0; s < S; ++s) {
            const uint32_t field = (((1u << BITS) - 1u) << (s * BITS)) * 0x00010001u;
            o |= __builtin_bit_cast(uint32_t, best[j][s]) & field;
        }
        out[j] = o;
    }
    ((vec *)a.y)[idx] = out;
}

template <int BITS, int W>
hipError_t launch_maxpool_w(const PoolArgs &a, hipStream_t s)
{
    const dim3 grid((a.total + 255) / 256);
    const int k = a.kh == a.kw && a.kh <= 3 ? a.kh : 0;
    if (k == 2)
        hipLaunchKernelGGL((maxpool_kernel<BITS, W, 2>), grid, dim3(256), 0, s, a);
    else if (k == 3)
        hipLaunchKernelGGL((maxpool_kernel<BITS, W, 3>), grid, dim3(256), 0, s, a);
    else
        hipLaunchKernelGGL((maxpool_kernel<BITS, W, 0>), grid, dim3(256), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_maxpool(const PoolArgs &p, int bits, hipStream_t s)
{
    // 16 bytes per lane where pixels are whole quads (buffers are 16-byte
    // aligned), else one word; windows without an instance of their own, whose
    // lanes take their taps one by one, only where that leaves a wave of quads
    // per SIMD (256 compute units of four): 7x7 / stride 2 on 316 images of
    // 56x9x64 INT-2 codes, 15800 quads, 13.4 against 9.1 us, and at 140000 to
    // 260000 quads 0.77 of the words' time (200 random windows)
    PoolArgs a = p;
    const bool built = a.kh == a.kw && (a.kh == 2 || a.kh == 3);
    const bool quads = a.pbd % 4 == 0 && (built || a.total / 4 >= 65536);
    if (quads) {
        a.pbd /= 4;
        a.total /= 4;
        a.div_pbd = make_fastdiv((uint32_t)a.pbd);
    }
    if (bits == 8)
        return quads ? launch_maxpool_w<8, 4>(a, s) : launch_maxpool_w<8, 1>(a, s);
    if (bits == 4)
        return quads ? launch_maxpool_w<4, 4>(a, s) : launch_maxpool_w<4, 1>(a, s);
    if (bits == 2)
        return quads ? launch_maxpool_w<2, 4>(a, s) : launch_maxpool_w<2, 1>(a, s);
    return hipErrorInvalidValue;
}

// max(x, 0) on the four signed bytes of a word: a byte is negative when its
// top bit is set; (neg << 8) - neg turns each such top bit into a 0xFF byte
// mask without carries between bytes.
__device__ __forceinline__ uint32_t relu_word(uint32_t v)
{
    const uint32_t neg = (v >> 7) & 0x01010101u;
    return v & ~((neg << 8) - neg);
}

// 16 bytes per lane, and a lane per byte of what is left (one lane for all of
// it is a chain of up to 15 loads and stores: 1.1 us of 3.3 us at 4207 bytes).
// The input is read once: non-temporal loads leave the memory-side cache to the
// output, which the next layer reads (with the pooling that follows 58.8 ->
// 51.7 us, side by side).
__global__ void __launch_bounds__(256) relu_s8_kernel(const uint8_t *x, uint8_t *y, size_t count)
{
    const size_t quads = count / 16;
    const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (i < quads) {
        typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
        const u32x4 v = __builtin_nontemporal_load((const u32x4 *)x + i);
        ((uint4 *)y)[i] = make_uint4(relu_word(v.x), relu_word(v.y), relu_word(v.z), relu_word(v.w));
    } else if (i < quads + (count & 15)) {
        const size_t b = quads * 16 + (i - quads);
        const int8_t v = (int8_t)x[b];
        y[b] = (uint8_t)(v > 0 ? v : 0);
    }
}

hipError_t launch_relu_s8(const uint8_t *x, uint8_t *y, size_t count, hipStream_t s)
{
    dim3 grid((unsigned)((count / 16 + (count & 15) + 255) / 256));
    hipLaunchKernelGGL(relu_s8_kernel, grid, dim3(256), 0, s, x, y, count);
    return hipGetLastError();
}

}  // namespace qnn
