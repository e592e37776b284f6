// The library's dispatch on the host alone: its argument checks and planners
// with every launch replaced by one that records which kernel was asked for.
// No device code and no device call: hip* functions answer for one gfx950.
#include "../paper_1908_11263_amd/csrc/qnn_abi.hip"

namespace {

// what the last call launched: kernel family, then (streaming kernel) tile,
// mode (0 codes, 1 raw, 2 pooled), lg, tail, one-tap, packed
struct Route {
    int32_t kernel, tile, mode, lg, tail, pw, xp, lds, dw, nblk;
};
enum { NONE, STREAM, XNOR, IMAGE, LINEAR, MFMA16, MFMA32, FP4, POOL, RELU };
Route g_route;

hipError_t stream(const StreamArgs &a, int variant)
{
    g_route = {STREAM, variant, a.pool ? 2 : (a.epi == EPI_RAW32 ? 1 : 0), a.lg, a.tail, a.pw1, a.xp, a.lds_bytes,
               a.dw, a.nblk};
    return hipSuccess;
}

hipError_t other(int kernel, int tile, int mode)
{
    g_route = {kernel, tile, mode, 0, 0, 0, 0, 0, 0, 0};
    return hipSuccess;
}

}  // namespace

namespace qnn {

#define STREAM_(B_) \
    hipError_t launch_conv_stream_##B_(const StreamArgs &a, int v, hipStream_t) { return stream(a, v); }
STREAM_(b8) STREAM_(b8x) STREAM_(b4) STREAM_(b4x) STREAM_(b4p) STREAM_(b4px) STREAM_(b2) STREAM_(b2x) STREAM_(b1) STREAM_(b1x)
#define TILE_(F_, K_) \
    hipError_t launch_conv_##F_(const ConvArgs &a, int x, int y, int, dim3, hipStream_t) { return other(K_, 10 * x + y, a.pool ? 2 : (a.epi == EPI_RAW32 ? 1 : 0)); }
#define TILE8_(F_, K_) \
    hipError_t launch_conv_##F_(const ConvArgs &a, int x, int y, int, int, dim3, hipStream_t) { return other(K_, 10 * x + y, a.pool ? 2 : (a.epi == EPI_RAW32 ? 1 : 0)); }
TILE_(mfma_b8, MFMA16) TILE_(mfma_b4, MFMA16) TILE_(mfma_b2, MFMA16)
TILE8_(m32_b8, MFMA32) TILE8_(m32_b4, MFMA32) TILE8_(m32_b2, MFMA32) TILE8_(m32_f4, FP4) TILE8_(m32_f4b1, FP4)
// (XNOR: the instance: 8, 16, .. 128 resident words, or 1, 2, 4, 8 words per step)
hipError_t launch_conv_xnor(const XnorArgs &a, hipStream_t)
{
    const bool res = a.kd % 8 == 0 && a.kd <= 128;
    return other(XNOR, res ? a.kd : (a.cd % 8 == 0 ? 8 : (a.cd % 4 == 0 ? 4 : (a.cd % 2 == 0 ? 2 : 1))), res ? 1 : 0);
}
hipError_t launch_conv_img_p2(const ImgArgs &, int, int, int, hipStream_t) { return other(IMAGE, 2, 0); }
hipError_t launch_conv_img_p4(const ImgArgs &, int, int, int, hipStream_t) { return other(IMAGE, 4, 0); }
hipError_t launch_conv_img_p16(const ImgArgs &, int, int, int, int, hipStream_t) { return other(IMAGE, 16, 0); }
hipError_t launch_conv_img_p32(const ImgArgs &, int, int, int, int, hipStream_t) { return other(IMAGE, 32, 0); }
hipError_t launch_linear_raw(const uint8_t *, const uint8_t *, const int32_t *, int32_t *, int32_t, int32_t, int32_t, int,
                             hipStream_t) { return other(LINEAR, 0, 1); }
hipError_t launch_maxpool(const PoolArgs &, int, hipStream_t) { return other(POOL, 0, 0); }
hipError_t launch_relu_s8(const uint8_t *, uint8_t *, size_t, hipStream_t) { return other(RELU, 0, 0); }

}  // namespace qnn

extern "C" {

static int g_device, g_attr_calls;
static hipError_t g_attr_status;

hipError_t hipGetDevice(int *d)
{
    *d = g_device;
    return hipSuccess;
}

hipError_t hipFuncSetAttribute(const void *, hipFuncAttribute, int)
{
    ++g_attr_calls;
    return g_attr_status;
}

// allow_large_lds on a device whose runtime answers `status`; attribute calls so far
int32_t probe_large_lds(int32_t device, int32_t status)
{
    static std::atomic<uint64_t> devices{0};
    g_device = device;
    g_attr_status = (hipError_t)status;
    allow_large_lds(nullptr, devices);
    g_device = 0;
    return g_attr_calls;
}

hipError_t hipGetDeviceProperties(hipDeviceProp_t *p, int)
{
    strcpy(p->gcnArchName, "gfx950:sramecc+:xnack-");
    p->multiProcessorCount = 256;
    return hipSuccess;
}

hipError_t hipGetLastError(void)
{
    return hipSuccess;
}

// resident_workgroups of kernel k with a query that answers `status` and n; asked: queries made so far
int32_t probe_resident(int32_t k, int32_t lds, int32_t status, int32_t n, int32_t *asked)
{
    return resident_workgroups((const void *)(intptr_t)(0x1000 * k), (size_t)lds, [&](int *out) {
        ++*asked;
        *out = n;
        return (hipError_t)status;
    });
}

// status of a call of run_conv on pointers that nothing reads; *r: what it launched
int32_t probe_conv(const qnn_tensor *x, int32_t m, const qnn_conv_geom *g, int32_t epi, const qnn_tensor *y, int32_t pool,
                   Route *r)
{
    void *p = (void *)0x1000;
    qnn_epi e;
    memset(&e, 0, sizeof(e));
    e.kind = epi;
    e.mult = e.thresh = (const int32_t *)p;
    e.shift = (const int8_t *)p;
    e.clip_hi = (1 << x->bits) - 1;
    g_route = {NONE, 0, 0, 0, 0, 0, 0, 0, 0, 0};
    const int32_t st = run_conv(x, p, m, p, g, &e, y, p, nullptr, pool != 0);
    *r = g_route;
    return st;
}

}
