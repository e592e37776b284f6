// Implicit-GEMM quantized convolution with the reduction streamed through
// local memory: the general kernel of 8-, 4-, 2- and 1-bit layers.
//
// The tile kernels (conv_mfma_impl.h, conv_m32_impl.h) hold the filters of
// their channels whole in LDS, which caps a channel tile at 160 KB / K and
// leaves the matrix cores waiting for one long staging phase per tile.  Here
// the reduction runs in steps of 64 staged bytes per channel and pixel:
//   for each 64-byte block of a pixel's channels, for each filter tap:
//     one 64-byte slice of the channel tile's filters (two LDS buffers of one
//     or two slices, the next loads in flight) times the block of the input
//     tile, read at the tap's offset
// so LDS holds a few filter slices and one block of the input tile with its
// halo, whatever K is, and each packed byte is unpacked once per tile.
//
// Tiles.  A workgroup (4 waves) owns 32*WM*WCH output channels and
// 32*WN*(4/WCH) consecutive outputs of the flattened (image, row, column)
// order, so odd sizes leave no partly filled tiles but the last one.  Its
// input tile is the consecutive run of padded input rows that those outputs
// touch, running on into the next image where the outputs do.  Each wave
// computes WM x WN 32x32 matrix tiles; per 32-deep step it reads WM + WN KB
// of fragments for WM * WN MFMAs, and at 128 B per clock and 32 clocks per
// MFMA on each of four SIMDs LDS feeds one KB per MFMA: 2x4 wave tiles (0.75
// KB) are matrix bound, 2x2 (1 KB) at the balance.
//
// Narrow pixels (at most 32 / 16 staged bytes) put two / four taps into one
// step instead of padding the step.
//
// 2- and 1-bit layers run on the e2m1 instruction (see conv_mfma_impl.h: every
// code is an e2m1 value and every partial sum an integer below 2^24, so the
// result is the integer one bit for bit) at half the staged bytes and twice
// the rate of int8: 128 channels per 64-byte block.
//
// Measured on the device, passes one after another, against the tile kernels
// (and XNOR / popcount at 1 bit): 256 images of 14x14x256 INT-8 codes, 256 3x3
// filters, 151 -> 39.4 us (1.5 POP/s); INT-1 8x8x256, 256 3x3 filters, batch
// 1024, 90 -> 20.9 us; 1x1 INT-8 28x28x128 -> 256, batch 256, 65.9 -> 30.9 us;
// INT-4 56x56x64 -> 128, stride 2, staircase, batch 256, 84.8 -> 49.4 us;
// 1000x4096 by 4096x1000 INT-8 58 -> 16.6 us.  What bounds it: where K is long,
// the main loop (the first of these layers keeps the matrix cores busy for 35%
// of the kernel's SIMD cycles, 45% on the compute units that hold two of its
// 392 tiles; a wave waits for a third of its time); where K is short, the chain
// of a tile's prologue (parameters, pixel offsets, loads, staging) and its
// compression (the 1x1 layer issues vector instructions in 47% of the SIMD
// cycles and matrix ones in 10%, the strided one in 38% and 12%).
#pragma once

#include "conv_m32_impl.h"

namespace qnn {

// Buffer descriptor of `bytes` bytes (at most 0x7fff0000) at `base`: reads past
// them return zero without touching memory, which replaces predicates on the
// loads.
constexpr uint32_t kStreamOob = 0x80000000u;
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ __amdgpu_buffer_rsrc_t stream_rsrc(const uint8_t *base, uint32_t bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc((void *)base, 0, (int)bytes, 0x00027000);
}

// LB (16, 8 or 4) bytes at offset vo (per lane) + so (uniform).  DW: word by
// word, the words from nvw on come back zero (items that end inside a run).
template <int LB, bool DW>
__device__ __forceinline__ uint4 stream_load(__amdgpu_buffer_rsrc_t r, uint32_t vo, uint32_t so, int nvw)
{
    uint4 v = make_uint4(0, 0, 0, 0);
    if (DW) {
        v.x = __builtin_amdgcn_raw_buffer_load_b32(r, nvw > 0 ? vo : kStreamOob, so, 0);
        if (LB >= 8)
            v.y = __builtin_amdgcn_raw_buffer_load_b32(r, nvw > 1 ? vo + 4 : kStreamOob, so, 0);
        if (LB == 16) {
            v.z = __builtin_amdgcn_raw_buffer_load_b32(r, nvw > 2 ? vo + 8 : kStreamOob, so, 0);
            v.w = __builtin_amdgcn_raw_buffer_load_b32(r, nvw > 3 ? vo + 12 : kStreamOob, so, 0);
        }
    } else if (LB == 4) {
        v.x = __builtin_amdgcn_raw_buffer_load_b32(r, vo, so, 0);
    } else if (LB == 8) {
        const u32x2 d = __builtin_bit_cast(u32x2, __builtin_amdgcn_raw_buffer_load_b64(r, vo, so, 0));
        v.x = d.x;
        v.y = d.y;
    } else {
        const u32x4 d = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(r, vo, so, 0));
        v = make_uint4(d.x, d.y, d.z, d.w);
    }
    return v;
}

// Staged form of one packed word at dst: 4, 8 or 16 bytes.
template <int BITS, bool F4, bool WEIGHT>
__device__ __forceinline__ void stream_word(uint8_t *dst, uint32_t v)
{
    if (BITS == 1)
        *(uint4 *)dst = b1_word_f4(v);
    else if (F4)
        *(uint2 *)dst = WEIGHT ? w2_word_f4(v) : x2_word_f4(v);
    else if (BITS == 8)
        *(uint32_t *)dst = WEIGHT ? v : v ^ 0x80808080u;
    else if (BITS == 4)
        *(uint2 *)dst = WEIGHT ? w4_word(v) : make_uint2(v & 0x0F0F0F0Fu, (v >> 4) & 0x0F0F0F0Fu);
    else
        *(uint4 *)dst = WEIGHT ? w2_word(v)
                               : make_uint4(v & 0x03030303u, (v >> 2) & 0x03030303u, (v >> 4) & 0x03030303u,
                                            (v >> 6) & 0x03030303u);
}

// Staged form of an item of LB packed bytes (16-byte stores).  live_words:
// 1-bit weights only, the words that exist: code 0 is -1 there, so the words
// past a run's end are written as e2m1 zeros.
template <int BITS, bool F4, bool WEIGHT, int LB>
__device__ __forceinline__ void stream_store(uint8_t *dst, uint4 v, int live_words)
{
    constexpr int E = BITS == 1 ? 16 : (F4 ? 8 : 32 / BITS);  // staged bytes per word
    if (BITS == 8) {
        if (!WEIGHT)
            v = make_uint4(v.x ^ 0x80808080u, v.y ^ 0x80808080u, v.z ^ 0x80808080u, v.w ^ 0x80808080u);
        *(uint4 *)dst = v;
        return;
    }
    const uint32_t d[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int i = 0; i < LB / 4; ++i) {
        if (BITS == 1 && WEIGHT && i >= live_words) {
            *(uint4 *)(dst + E * i) = make_uint4(0, 0, 0, 0);
            continue;
        }
        stream_word<BITS, F4, WEIGHT>(dst + E * i, d[i]);
    }
}

// Split barrier: LDS traffic of the wave done, global loads left in flight.
__device__ __forceinline__ void stream_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

template <int V>
struct StreamInt {
    static constexpr int value = V;
};

enum { STREAM_CODES = 0, STREAM_RAW = 1, STREAM_POOL = 2 };

// LG: log2 of the 16-byte chunks a tap takes in a step (2: one tap per step;
// 1, 0: pixels of one block of at most 32 / 16 staged bytes, two / four taps
// per step).  TAIL: the last block's items may end inside their 16 bytes.
// PW: filters of one tap (LG = 2): a slot is an output of the tile, and both
// operands stream, the input in two LDS buffers loaded D steps ahead.
// Otherwise the input block stays for all taps in one LDS buffer; the next
// block's loads are issued in its first two steps, held in registers and
// stored after its last (batches past the second are loaded there).
// G: filter slices per step (between two barriers).  Two save 3-8% unless their
// LDS costs a workgroup of a compute unit.
// XP (4 bits, LG = 2): the input tile stays packed in LDS and its fragments (8
// packed bytes per lane) are unpacked in registers, six instructions beside WM
// matrix instructions of 32 clocks.  Half the LDS per pixel, which is what
// limits the workgroups of a compute unit where strides, tall filters or short
// images make the tile many rows: INT-4 56x56x64 -> 128, stride 2, staircase,
// batch 256, 65.4 -> 49.3 us; 8x30x56 -> 16, pooled, batch 12222, 190 -> 125.
// Where no more workgroups fit it costs up to 7%, except with one-tap filters,
// whose input is read once: 1x1 56x22x64 -> 34, stride 2, pooled, batch 3005,
// 28.8 -> 19.9 us, so these are built packed only.  2- and 1-bit codes take
// more instructions per fragment, beside e2m1 matrix instructions of the same 32
// clocks: not built.
template <int BITS, int WM, int WN, int WCH, int G, int MODE, int LG, bool TAIL, bool PW, bool XP>
__global__ void __launch_bounds__(256, (WM * WN >= 6 ? 2 : (WM * WN >= 4 ? 3 : 4))) conv_stream_kernel(StreamArgs a)
{
    extern __shared__ __align__(16) uint8_t smem[];
    static_assert(!XP || (BITS == 4 && LG == 2), "packed tiles: whole 4-bit blocks");
    static_assert(!PW || G == 1, "one-tap filters bring new input with every slice");
    constexpr bool F4 = BITS <= 2;
    constexpr int WPX = 4 / WCH;
    constexpr int MT = 32 * WM * WCH;
    constexpr int PT = 32 * WN * WPX;
    constexpr int RB = F4 ? 16 * BITS : 8 * BITS;  // packed bytes of a 64-byte staged block
    constexpr int RUN = RB >> (2 - LG);             // ... of one tap's share of a step
    constexpr int LB = RUN < 16 ? RUN : 16;         // packed bytes of an item
    constexpr int QPR = RUN / LB, TPS = 4 >> LG;    // items per run, taps per step
    constexpr int IPR = TPS * QPR;                  // filter items per row and step
    constexpr int WS = 64 * G + 16;                 // LDS strides: odd multiples of 16 bytes
    constexpr int XD = XP ? 2 : 1;                  // staged bytes per byte held
    // (LDS strides that no two lanes of a half-wave's fragment read share banks at)
    constexpr int PS = XP ? 40 : (LG == 2 ? 80 : (LG == 1 ? 48 : 16));
    constexpr int SPX = (16 << LG) / QPR / XD;      // bytes of an input item in LDS
    constexpr int UW = (MT * IPR + 255) / 256;      // filter items per thread and step
    // input items per thread and batch
    constexpr int UX = PW ? (PT * QPR + 255) / 256 : 4;
    // loads are issued D steps ahead.  One-tap filters wait for both operands
    // in every step: four steps where the tile leaves registers for it (1000
    // INT-8 images of 4096 codes to 1000 outputs 21.3 -> 18.5 us in graph
    // replays, 40 drawn linear layers 0.98; packed 4-bit tiles gained nothing
    // and lost 5% on reductions of two steps)
    constexpr int D = PW ? (UX + UW <= 3 && !XP ? 4 : 2) : 3 - G;
    // log2 of the weight scale the accumulator carries (4-bit filters are staged as 16 w)
    constexpr int SL = BITS == 4 ? 4 : 0;
    constexpr int NTH = BITS == 8 ? 1 : (1 << BITS) - 1;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wch = WCH == 2 ? (wv & 1) : 0, wpx = WCH == 2 ? (wv >> 1) : wv;
    const int h = lane >> 5, r32 = lane & 31;

    // consecutive units on one XCD (workgroup i runs on XCD i mod 8): the
    // channel tiles of a pixel tile follow one another there and share its
    // input in that XCD's L2, neighbouring pixel tiles their halo rows
    int unit;
    {
        const int total = a.ptiles * a.mtiles, q = total >> 3, r = total & 7;
        const int xcd = blockIdx.x & 7, loc = blockIdx.x >> 3;
        unit = xcd * q + min(xcd, r) + loc;
    }
    const int pt = (int)fdiv((uint32_t)unit, a.div_mt);
    const int m0 = (unit - pt * a.mtiles) * MT;
    const int p0 = pt * PT;

    // codes: lane = output, register = channel (four consecutive ones per
    // register group): the matrix rows are channels.  Raw sums and pooled
    // codes: lane = channel, so a half-wave stores 32 consecutive sums and a
    // register group is a pooling window.
    constexpr bool CH_ROWS = MODE == STREAM_CODES;
    // per-channel parameters: plan words [7][MT] (e0.xyzw, e1.xyz of
    // requant_plan), or thresholds, [MT][16] (codes; one: [MT]) / [NTH][MT]
    int32_t *sP = (int32_t *)(smem + a.off_epi);
    int32_t *sSum = (int32_t *)(smem + a.off_sum);     // [MT] filter sums, [4] votes
    uint32_t *sPix = (uint32_t *)(smem + a.off_pix);

    // ---- prologue ----
    const int mrows = min(MT, a.m - m0);
    const __amdgpu_buffer_rsrc_t wr = stream_rsrc(a.w + (size_t)m0 * (uint32_t)a.wrow, (uint32_t)(mrows * a.wrow));
    const int nblk = LG == 2 ? a.nblk : 1;
    const int lastb = nblk - 1;
    const int spb = LG == 2 ? a.taps : a.nlast;        // slices per block
    // steps per block: with two register sets an even number, so that each
    // step's set is fixed (the step added loads and multiplies nothing)
    const int ns = PW ? 1 : (spb + 1) / 2 * D;
    const int pb = a.pb, taps = a.taps;

    // filter slice of a step: item u of this thread
    uint4 wq[D][G * UW];
    uint32_t wvo[UW];
    int wsum[UW];
    const int qn = (uint32_t)tid % QPR;                           // the item's place in its run (256 % IPR = 0)
    const int wtap = (int)((uint32_t)tid % IPR / QPR);
    // words of the last block's items that exist
    const int nvw = TAIL ? min(max((pb - lastb * RB - qn * LB) >> 2, 0), LB / 4) : LB / 4;
#pragma unroll
    for (int u = 0; u < UW; ++u) {
        const int row = (int)((uint32_t)(tid + u * 256) / IPR);
        wvo[u] = row < mrows ? (uint32_t)(row * a.wrow + wtap * pb + qn * LB) : kStreamOob;
        wsum[u] = 0;
    }
    // (no load is conditional: one that may or may not be in flight turns the
    // waits around it into waits for everything.  Slices past a block's or the
    // last one load slice 0, which is not stored.)
    auto w_load = [&](uint4 *q, int cb, int t) {
        const uint32_t so = cb < nblk && t < spb ? (uint32_t)(t * TPS * pb + cb * RB) : 0u;
        const bool live = (TPS == 1 || t * TPS + wtap < taps) && (!TAIL || cb != lastb || nvw > 0) &&
                          (!PW || D == 2 || cb < nblk);
        const bool sel = TPS > 1 || TAIL || (PW && D > 2);
        if (TAIL && cb == lastb && a.dw) {
#pragma unroll
            for (int u = 0; u < UW; ++u)
                q[u] = stream_load<LB, true>(wr, live ? wvo[u] : kStreamOob, so, nvw);
        } else {
#pragma unroll
            for (int u = 0; u < UW; ++u)
                q[u] = stream_load<LB, false>(wr, !sel || live ? wvo[u] : kStreamOob, so, 0);
        }
    };
    auto w_store = [&](const uint4 *q, int cb, int t, int buf) {
        uint8_t *sW = smem + buf;
        int live = LB / 4;
        if (BITS == 1) {
            if (TAIL && cb == lastb)
                live = nvw;
            if (TPS > 1 && t * TPS + wtap >= taps)
                live = 0;
        }
#pragma unroll
        for (int u = 0; u < UW; ++u) {
            const uint32_t i = (uint32_t)(tid + u * 256);
            if (MT * IPR >= 256 * UW || i < MT * IPR)
                stream_store<BITS, F4, true, LB>(sW + (i / IPR) * WS + (i % IPR) * (64 / IPR), q[u], live);
            if (BITS == 8) {
                int s = wsum[u];
                s = __builtin_amdgcn_sdot4((int)q[u].x, 0x01010101, s, false);
                s = __builtin_amdgcn_sdot4((int)q[u].y, 0x01010101, s, false);
                s = __builtin_amdgcn_sdot4((int)q[u].z, 0x01010101, s, false);
                wsum[u] = __builtin_amdgcn_sdot4((int)q[u].w, 0x01010101, s, false);
            }
        }
    };
    // the next step whose slices are loaded
    int lcb = 0, lt = 0;
    auto w_next = [&](uint4 *q) {
#pragma unroll
        for (int g = 0; g < G; ++g)
            w_load(q + g * UW, lcb, lt * G + g);
        if (++lt == ns) {
            lt = 0;
            ++lcb;
        }
    };
#pragma unroll
    for (int d = 0; d < D; ++d)
        w_next(wq[d]);

    // the channel tile's parameters (one thread per channel)
    int32_t p_bias = 0, p_mult = 0, p_shift = 0;
    const bool has_ch = tid < MT;
    if (has_ch && tid < mrows) {
        if (a.bias)
            p_bias = a.bias[m0 + tid];
        if (MODE != STREAM_RAW && a.epi == EPI_REQUANT) {
            p_mult = a.mult[m0 + tid];
            p_shift = a.shift[m0 + tid];
        }
    }

    // the tile's first staged row, counted from the first row of image n0
    int n0, v0;
    {
        const int q0 = (MODE == STREAM_POOL ? p0 >> 2 : p0);
        const int R = (int)fdiv((uint32_t)q0, a.div_wo);
        n0 = (int)fdiv((uint32_t)R, a.div_ho);
        v0 = (R - n0 * a.ho) * a.ssh * (MODE == STREAM_POOL ? 2 : 1);
    }
    const __amdgpu_buffer_rsrc_t xr = stream_rsrc(a.x + (size_t)n0 * ((size_t)a.h * a.w_) * (uint32_t)pb, 0x7fff0000u);
    // input offset of every pixel slot of the tile; the entry past them reads
    // as zero.  PW: slot = output of the tile; else slot = staged row and
    // column (with two columns per output the even ones come first)
    const int nslots = PW ? PT : a.nslots;
    for (int s = tid; s <= nslots; s += 256) {
        int dn, iy, ix;
        if (PW) {
            const int p = p0 + s, q = MODE == STREAM_POOL ? p >> 2 : p;
            const int R = (int)fdiv((uint32_t)q, a.div_wo);
            const int nn = (int)fdiv((uint32_t)R, a.div_ho);
            iy = R - nn * a.ho;
            ix = q - R * a.wo;
            if (MODE == STREAM_POOL) {
                iy = 2 * iy + ((p >> 1) & 1);
                ix = 2 * ix + (p & 1);
            }
            iy = iy * a.rsh - a.ph;
            ix = ix * a.rsw - a.pw;
            dn = nn - n0;
        } else {
            const int r = (int)fdiv((uint32_t)s, a.div_hwd);
            int c = s - r * a.hwd;
            if (a.ssw == 2)
                c = c < a.half ? 2 * c : 2 * (c - a.half) + 1;
            const int vr = v0 + r;
            dn = (int)fdiv((uint32_t)vr, a.div_hv);
            iy = (vr - dn * a.hv) * a.rsh - a.ph;
            ix = c * a.rsw - a.pw;
        }
        uint32_t off = kStreamOob;
        if (s < nslots && n0 + dn < a.n && (uint32_t)iy < (uint32_t)a.h && (uint32_t)ix < (uint32_t)a.w_)
            off = (uint32_t)(((dn * a.h + iy) * a.w_ + ix) * pb);
        sPix[s] = off;
    }
    stream_barrier();

    // ---- input tile: a block in batches of UX items per thread ----
    constexpr int NBPW = (PT * QPR + 256 * UX - 1) / (256 * UX);
    static_assert(!PW || NBPW == 1 || LG != 2, "a pointwise tile's block is one batch");
    constexpr int XQ = PW ? D : 2;
    uint4 xq[XQ][UX];
    uint32_t xo[PW ? UX : 1];
    const int nbatch = PW ? 1 : a.nbatch;
    auto x_off = [&](int b, int u) {
        const int slot = (int)((uint32_t)(b * (256 * UX) + tid + u * 256) / QPR);
        return sPix[min(slot, nslots)] + (uint32_t)(qn * LB);
    };
    auto x_load = [&](uint4 *q, int cb, int b) {
        const uint32_t so = (uint32_t)(cb * RB);
        uint32_t o[UX];
#pragma unroll
        for (int u = 0; u < UX; ++u)
            o[u] = PW ? xo[PW ? u : 0] : x_off(b, u);
        if (TAIL && cb == lastb && a.dw) {
#pragma unroll
            for (int u = 0; u < UX; ++u)
                q[u] = stream_load<LB, true>(xr, o[u], so, nvw);
        } else {
            const bool live = cb < nblk && (!TAIL || cb != lastb || nvw > 0);
#pragma unroll
            for (int u = 0; u < UX; ++u)
                q[u] = stream_load<LB, false>(xr, live ? o[u] : kStreamOob, so, 0);
        }
    };
    auto x_store = [&](const uint4 *q, int b, int buf) {
        uint8_t *sX = smem + a.off_x + buf * a.xbuf + qn * SPX;
#pragma unroll
        for (int u = 0; u < UX; ++u) {
            const int first = b * (256 * UX) + u * 256;
            if (!PW && first >= nslots * QPR)
                break;
            const int slot = (int)((uint32_t)(first + tid) / QPR);
            if (slot < nslots) {
                if constexpr (XP) {
                    *(uint2 *)(sX + slot * PS) = make_uint2(q[u].x, q[u].y);
                    *(uint2 *)(sX + slot * PS + 8) = make_uint2(q[u].z, q[u].w);
                } else {
                    stream_store<BITS, F4, false, LB>(sX + slot * PS, q[u], 4);
                }
            }
            if (BITS != 8 && !XP)
                __builtin_amdgcn_sched_barrier(0);  // (unpacked together they would spill)
        }
    };
    if (PW) {
#pragma unroll
        for (int u = 0; u < UX; ++u)
            xo[PW ? u : 0] = x_off(0, u);
    }
    x_load(xq[0], 0, 0);
    if (PW) {
#pragma unroll
        for (int d = 1; d < XQ; ++d)
            x_load(xq[d], d, 0);
    } else {
        x_load(xq[1], 0, 1);
    }

    // plans (their 8-bit filter sums are folded in after the main loop)
    if (MODE != STREAM_RAW) {
        bool v3 = true, v4 = true, sorted = true;
        if (BITS != 8 && (a.epi == EPI_STAIR || a.epi == EPI_THRESH1)) {
            if (has_ch) {
                int32_t T[16];
                stair_thresholds(tid < mrows ? a.thresh + (size_t)(m0 + tid) * NTH : nullptr, NTH, p_bias, SL, T);
#pragma unroll
                for (int i = 0; i < NTH; ++i) {
                    sP[CH_ROWS && NTH > 1 ? tid * 16 + i : i * MT + tid] = T[i];
                    sorted = sorted && (i == 0 || T[i] >= T[i > 0 ? i - 1 : 0]);
                }
            }
        } else if (has_ch) {
            int4 e0 = make_int4(0, 0, 0, 0), e1 = make_int4(0, 0, 3, 0);
            if (tid < mrows) {
                const int sh = p_shift < 0 ? 0 : (p_shift > 62 ? 62 : p_shift);
                requant_plan(p_bias, p_mult, sh, a.clip_lo, a.clip_hi, true, SL, e0, e1);
            }
            const int32_t e[7] = {e0.x, e0.y, e0.z, e0.w, e1.x, e1.y, e1.z};
#pragma unroll
            for (int i = 0; i < 7; ++i)
                sP[i * MT + tid] = e[i];
            v3 = e1.z == 3;
            v4 = e1.z >= 3;
        }
        const bool a3 = __all(v3), a4 = __all(v4), as = __all(sorted);
        if (lane == 0)
            sSum[MT + wv] = (a3 ? 1 : 0) | (a4 ? 2 : 0) | (as ? 4 : 0);
    } else if (has_ch) {
        sP[tid] = p_bias;
    }

    // ---- per-lane pixel bases ----
    int base[WN];
#pragma unroll
    for (int c = 0; c < WN; ++c) {
        const int p = min(p0 + wpx * 32 * WN + c * 32 + r32, a.npix - 1);
        const int q = MODE == STREAM_POOL ? p >> 2 : p;
        const int R = (int)fdiv((uint32_t)q, a.div_wo);
        int ox = q - R * a.wo;
        const int nn = (int)fdiv((uint32_t)R, a.div_ho);
        int oy = R - nn * a.ho;
        if (MODE == STREAM_POOL) {
            oy = 2 * oy + ((p >> 1) & 1);
            ox = 2 * ox + (p & 1);
        }
        const int vr = PW ? 0 : (nn - n0) * a.hv + oy * a.ssh - v0;
        if (PW)
            base[c] = (wpx * 32 * WN + c * 32 + r32) * PS + a.off_x + h * (16 / XD);
        else
            base[c] = (vr * a.hwd + (a.ssw == 2 ? ox : ox * a.ssw)) * PS + a.off_x + (LG > 0 ? h * (16 / XD) : 0);
    }
    const int wlane = (wch * 32 * WM + r32) * WS + h * 16;

    // input block 0 and the first filter slice
    x_store(xq[0], 0, 0);
    if (!PW) {
        x_store(xq[1], 1, 0);
        for (int b = 2; b < nbatch; b += 2) {
            x_load(xq[0], 0, b);
            x_load(xq[1], 0, b + 1);
            x_store(xq[0], b, 0);
            x_store(xq[1], b + 1, 0);
        }
    }
#pragma unroll
    for (int g = 0; g < G; ++g)
        if (g == 0 || g < spb)
            w_store(wq[0] + g * UW, 0, g, a.off_w + 64 * g);
    stream_barrier();

    // ---- main loop ----
    typedef typename AccTile<F4>::type ACC;
    ACC acc[WM][WN];
#pragma unroll
    for (int i = 0; i < WM; ++i)
#pragma unroll
        for (int c = 0; c < WN; ++c)
            acc[i][c] = (ACC){};
    // lane t holds tap t's offset in the input tile (a scalar read per step);
    // taps past the last one meet zero weights and read slot 0
    int tapv = 0;
    if (!PW && lane < taps) {
        const int ky = (int)fdiv((uint32_t)lane, a.div_kw), kx = lane - ky * a.kw;
        tapv = (ky * a.hwd + (a.ssw == 2 ? (kx & 1) * a.half + (kx >> 1) : kx)) * PS;
    }
    // Offsets of a step's two MFMA depths in the input tile.
    auto x_offs = [&](int cb, int t, int &o0, int &o1) {
        if (PW) {
            o0 = (cb & 1) * a.xbuf;
            o1 = o0 + 32 / XD;
        } else if (LG == 2) {
            o0 = __builtin_amdgcn_readlane(tapv, t);
            o1 = o0 + 32 / XD;
        } else if (LG == 1) {
            o0 = __builtin_amdgcn_readlane(tapv, 2 * t);
            o1 = __builtin_amdgcn_readlane(tapv, 2 * t + 1);
        } else {
            const int t0 = __builtin_amdgcn_readlane(tapv, 4 * t), t1 = __builtin_amdgcn_readlane(tapv, 4 * t + 1);
            const int t2 = __builtin_amdgcn_readlane(tapv, 4 * t + 2), t3 = __builtin_amdgcn_readlane(tapv, 4 * t + 3);
            o0 = h ? t1 : t0;
            o1 = h ? t3 : t2;
        }
    };
    int cb = 0, t = 0;
    int rb = a.off_w, wb = a.off_w + MT * WS;  // filter buffers read and written by the step
    // S: the register set of a step's filter loads; XL: issues the loads of
    // the next input block's first two batches
    auto step = [&](auto slot, auto xl) {
        constexpr int S = decltype(slot)::value;
        constexpr bool XL = decltype(xl)::value != 0;
        const bool block_end = t + 1 == ns;
        const int ncb = block_end ? cb + 1 : cb, nt = block_end ? 0 : t + 1;
        w_next(wq[S]);
        if (PW) {
            x_load(xq[S % XQ], cb + D, 0);
        } else if (XL) {
            x_load(xq[0], cb + 1, 0);
            x_load(xq[1], cb + 1, 1);
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int g = 0; g < G; ++g) {
            const int sl = t * G + g;
            if (!PW && sl >= spb)
                break;
            int o0, o1;
            x_offs(cb, sl, o0, o1);
            const uint8_t *wp = smem + rb + wlane + 64 * g;
            v4i xf[2][WN], wf[2][WM];
            uint2 xp[2][WN];
            auto frags = [&](int ks) {
#pragma unroll
                for (int i = 0; i < WM; ++i)
                    wf[ks][i] = *(const v4i *)(wp + i * 32 * WS + ks * 32);
#pragma unroll
                for (int c = 0; c < WN; ++c) {
                    if constexpr (XP)
                        xp[ks][c] = *(const uint2 *)(smem + base[c] + (ks ? o1 : o0));
                    else
                        xf[ks][c] = *(const v4i *)(smem + base[c] + (ks ? o1 : o0));
                }
            };
            auto mfmas = [&](int ks) {
                if constexpr (XP) {
#pragma unroll
                    for (int c = 0; c < WN; ++c) {
                        const uint2 d = xp[ks][c];
                        xf[ks][c] = (v4i){(int)(d.x & 0x0F0F0F0Fu), (int)((d.x >> 4) & 0x0F0F0F0Fu),
                                          (int)(d.y & 0x0F0F0F0Fu), (int)((d.y >> 4) & 0x0F0F0F0Fu)};
                    }
                }
#pragma unroll
                for (int i = 0; i < WM; ++i)
#pragma unroll
                    for (int c = 0; c < WN; ++c) {
                        const v4i row = CH_ROWS ? wf[ks][i] : xf[ks][c], col = CH_ROWS ? xf[ks][c] : wf[ks][i];
                        if constexpr (F4)
                            acc[i][c] = mfma_f4<BITS>(row, col, acc[i][c]);
                        else
                            acc[i][c] = __builtin_amdgcn_mfma_i32_32x32x32_i8(row, col, acc[i][c], 0, 0, 0);
                    }
            };
            frags(0);
            __builtin_amdgcn_sched_barrier(0);
            mfmas(0);
            // (the second half of the last block may be all padding)
            if (!TAIL || cb != lastb || a.last2 || (LG < 2 && sl + 1 != spb)) {
                frags(1);
                mfmas(1);
            }
        }
        if (ncb < nblk) {
#pragma unroll
            for (int g = 0; g < G; ++g)
                if (PW || nt * G + g < spb)
                    w_store(wq[(S + 1) % D] + g * UW, ncb, nt * G + g, wb + 64 * g);
            if (PW)
                x_store(xq[(S + 1) % XQ], 0, ncb & 1);
        }
        stream_barrier();
        cb = ncb;
        t = nt;
        const int sw = rb;
        rb = wb;
        wb = sw;
    };
    using No = StreamInt<0>;
    if constexpr (PW) {
        for (;;) {
            step(StreamInt<0>(), No());
            if (cb == nblk)
                break;
            step(StreamInt<1>(), No());
            if (cb == nblk)
                break;
            if constexpr (D == 4) {
                step(StreamInt<2>(), No());
                if (cb == nblk)
                    break;
                step(StreamInt<3>(), No());
                if (cb == nblk)
                    break;
            }
        }
    } else {
        for (;;) {
            step(StreamInt<0>(), StreamInt<(LG == 2 ? 1 : 0)>());
            if constexpr (D == 1) {
                while (t != 0)
                    step(StreamInt<0>(), No());
            } else {
                step(StreamInt<1>(), No());
                while (t != 0) {
                    step(StreamInt<0>(), No());
                    step(StreamInt<1>(), No());
                }
            }
            if (cb == nblk)
                break;
            // every wave is done with the block: the next one takes its place
            x_store(xq[0], 0, 0);
            x_store(xq[1], 1, 0);
            for (int b = 2; b < nbatch; b += 2) {
                x_load(xq[0], cb, b);
                x_load(xq[1], cb, b + 1);
                x_store(xq[0], b, 0);
                x_store(xq[1], b + 1, 0);
            }
            stream_barrier();
        }
    }

    // ---- epilogue ----
    // register v of a matrix tile: row 8 (v / 4) + 4 h + v % 4, column r32
    if (BITS == 8) {
#pragma unroll
        for (int u = 0; u < UW; ++u) {
            int s = wsum[u];
            s += __shfl_xor(s, 1, 64);
            s += __shfl_xor(s, 2, 64);
            const int row = (tid + u * 256) >> 2;  // four items per row at 8 bits
            if ((tid & 3) == 0 && row < MT)
                sSum[row] = 128 * s;
        }
        stream_barrier();
    }
    if (MODE == STREAM_RAW) {
        int32_t *y = (int32_t *)a.y;
#pragma unroll
        for (int i = 0; i < WM; ++i) {
            const int ch = wch * 32 * WM + i * 32 + r32, mg = m0 + ch;
            const uint32_t bt = (uint32_t)sP[ch] + (BITS == 8 ? (uint32_t)sSum[ch] : 0u);
#pragma unroll
            for (int c = 0; c < WN; ++c) {
                const int pl = p0 + wpx * 32 * WN + c * 32 + 4 * h;
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int p = pl + 8 * (v >> 2) + (v & 3);
                    if (mg < a.m && p < a.npix)
                        y[(size_t)p * a.m + mg] = (int32_t)((uint32_t)((int32_t)acc[i][c][v] >> SL) + bt);
                }
            }
        }
        return;
    }
    int votes = sSum[MT];
#pragma unroll
    for (int w = 1; w < 4; ++w)
        votes &= sSum[MT + w];
    const bool thr = BITS != 8 && (a.epi == EPI_STAIR || a.epi == EPI_THRESH1);
    // the code of one accumulator under the plan words e of its channel
    auto code3 = [&](int32_t x, const int32_t *e) {
        const int32_t d = __builtin_elementwise_sub_sat(x, e[0]);
        const uint32_t dc = (uint32_t)min(max(d, 0), e[1]);
        return (__umul24(dc, (uint32_t)e[2]) + (uint32_t)e[3]) >> e[4];
    };
    auto code4 = [&](int32_t x, const int32_t *e) {
        // the 48-bit product of two 24-bit numbers from its full-rate halves
        // (a 32x32->64 multiply-add and a 64-bit shift take four times as long)
        const int32_t d = __builtin_elementwise_sub_sat(x, e[0]);
        const uint32_t dc = (uint32_t)min(max(d, 0), e[1]);
        uint32_t hi;
        __asm__("v_mul_hi_u32_u24 %0, %1, %2" : "=v"(hi) : "v"(dc), "v"(e[2]));
        const uint32_t lo = __umul24(dc, (uint32_t)e[2]), sum = lo + (uint32_t)e[3];
        hi += (uint32_t)e[5] + (sum < lo ? 1u : 0u);
        return __builtin_amdgcn_alignbit(hi, sum, (uint32_t)e[4]);
    };
    auto code_any = [&](int32_t x, const int32_t *e, int32_t sum) -> uint32_t {
        if (e[6] >= 3)
            return code4(x, e);
        const int32_t x32 = x >> SL;
        int64_t r;
        if (e[6]) {
            const int32_t d = __builtin_elementwise_sub_sat(x32, e[0]);
            const uint32_t dc = (uint32_t)min(max(d, 0), e[1]);
            r = (int64_t)e[4] + (int64_t)(uint32_t)(((uint64_t)dc * (uint32_t)e[2] + (uint32_t)e[3]) >> e[5]);
        } else {
            const int64_t b = (int64_t)(((uint64_t)(uint32_t)e[1] << 32) | (uint32_t)e[0]) + sum;
            r = round_shift(((int64_t)x32 + b) * (int64_t)e[2], e[3]);
        }
        return (uint32_t)(r < a.clip_lo ? a.clip_lo : (r > a.clip_hi ? a.clip_hi : r));
    };
    // 128 sum(w) of 8-bit layers goes into the plan's origin (an origin past
    // int32 saturates, where the clamped difference is the same) or, in the
    // direct form, into the bias
    auto fold = [&](int32_t *e, int32_t sum) {
        if (BITS == 8 && e[6] != 0)
            e[0] = __builtin_elementwise_sub_sat(e[0], sum);
    };
    constexpr int OB = MT * BITS / 8;               // output bytes of the tile's channels per pixel
    const int ob0 = m0 * BITS / 8;
    const int obn = min(OB, a.ypb - ob0);

    if constexpr (CH_ROWS) {
        // Codes of four consecutive channels per register group, packed in the
        // lane: word[c][g] holds the codes of channels 8 g + 4 h .. + 3 of
        // output c*32 + r32.  The two halves then trade registers so that each
        // holds consecutive channels and stores them straight to memory (8
        // bits: 16 bytes per lane, 32 per output and matrix tile); outputs
        // whose rows are not aligned for that go through LDS.
        uint8_t *sC = smem + a.off_out;
        constexpr int CS = OB + 4;                   // LDS bytes per output of the indirect path
        constexpr int TB = 4 * BITS;                 // output bytes of 32 channels
        const bool direct = (a.ypb % (BITS == 1 ? 4 : TB / 2)) == 0 && obn == OB;
        // stores of matrix tile row i (addresses from an opaque copy of p0: they
        // would otherwise be kept in registers through the main loop)
        int pe = p0;
        __asm__ volatile("" : "+s"(pe));
        uint8_t *const yl = a.y + (size_t)(pe + wpx * 32 * WN + r32) * (uint32_t)a.ypb + ob0 + wch * WM * TB;
        auto emit = [&](int i, uint32_t (*word)[4]) {
#pragma unroll
            for (int c = 0; c < WN; ++c) {
                const int pl = wpx * 32 * WN + c * 32 + r32;
                const bool ok = pe + pl < a.npix;
                uint32_t *w = word[c];
                uint8_t *d = yl + (size_t)(c * 32) * (uint32_t)a.ypb + i * TB;
                uint32_t *l = (uint32_t *)(sC + pl * CS + (wch * WM + i) * TB);
                if constexpr (BITS == 8) {
                    // the halves trade groups: 16 consecutive channels each
                    const auto s0 = __builtin_amdgcn_permlane32_swap(w[0], w[2], false, false);
                    const auto s1 = __builtin_amdgcn_permlane32_swap(w[1], w[3], false, false);
                    if (direct) {
                        if (ok)
                            *(uint4 *)(d + 16 * h) = make_uint4(s0[0], s0[1], s1[0], s1[1]);
                    } else {
                        l[4 * h] = s0[0];
                        l[4 * h + 1] = s0[1];
                        l[4 * h + 2] = s1[0];
                        l[4 * h + 3] = s1[1];
                        __asm__ volatile("" ::: "memory");  // keeps the two paths' stores apart
                    }
                } else if constexpr (BITS == 4) {
                    const auto s0 = __builtin_amdgcn_permlane32_swap(w[0] | (w[1] << 16), w[2] | (w[3] << 16), false, false);
                    const uint32_t u0 = __builtin_amdgcn_perm(s0[1], s0[0], 0x05040100u);
                    const uint32_t u1 = __builtin_amdgcn_perm(s0[1], s0[0], 0x07060302u);
                    if (direct) {
                        if (ok)
                            *(uint2 *)(d + 8 * h) = make_uint2(u0, u1);
                    } else {
                        l[2 * h] = u0;
                        l[2 * h + 1] = u1;
                        __asm__ volatile("" ::: "memory");
                    }
                } else if constexpr (BITS == 2) {
                    // bytes (group, half) -> group-major; after the swap of a
                    // register with itself both halves hold the lower half's
                    // bytes in one and the upper half's in the other
                    const uint32_t r = w[0] | (w[1] << 8) | (w[2] << 16) | (w[3] << 24);
                    const auto s0 = __builtin_amdgcn_permlane32_swap(r, r, false, false);
                    const uint32_t u = __builtin_amdgcn_perm(s0[1], s0[0], h ? 0x07030602u : 0x05010400u);
                    if (!direct) {
                        l[h] = u;
                        __asm__ volatile("" ::: "memory");
                    } else if (ok) {
                        *(uint32_t *)(d + 4 * h) = u;
                    }
                } else {
                    const uint32_t r = w[0] | (w[1] << 8) | (w[2] << 16) | (w[3] << 24);
                    const auto s0 = __builtin_amdgcn_permlane32_swap(r, r, false, false);
                    if (!direct) {
                        l[0] = s0[0] | (s0[1] << 4);
                        __asm__ volatile("" ::: "memory");
                    } else if (ok && h == 0) {
                        *(uint32_t *)d = s0[0] | (s0[1] << 4);
                    }
                }
            }
        };
        // plan words f of channels ch .. ch + 3
        auto plan4 = [&](int f, int ch, int32_t *e) {
            const int4 q = *(const int4 *)(sP + f * MT + ch);
            e[0] = q.x;
            e[1] = q.y;
            e[2] = q.z;
            e[3] = q.w;
        };
        // One form of the compression over the wave's tiles: each form is one
        // run of code without the others' in between (a workgroup often runs
        // it once: what it costs is fetching it).  FORM 0: one threshold, 1:
        // sorted staircase, 2: any staircase, 3 / 4: 32- / 64-bit plans, 5:
        // any plan.
        auto run = [&](auto form) {
            constexpr int FORM = decltype(form)::value;
            __asm__ volatile("" ::"n"(FORM) : "memory");  // nothing of it moves above the choice
#pragma unroll
            for (int i = 0; i < WM; ++i) {
                uint32_t word[WN][4];
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const int ch = wch * 32 * WM + i * 32 + 8 * g + 4 * h;
                    int32_t x[WN][4];
#pragma unroll
                    for (int c = 0; c < WN; ++c) {
                        word[c][g] = 0;
#pragma unroll
                        for (int k = 0; k < 4; ++k)
                            x[c][k] = (int32_t)acc[i][c][4 * g + k];
                    }
                    if constexpr (FORM == 0) {
                        int32_t T[4];
                        plan4(0, ch, T);
#pragma unroll
                        for (int c = 0; c < WN; ++c)
#pragma unroll
                            for (int k = 0; k < 4; ++k)
                                word[c][g] |= x[c][k] >= T[k] ? 1u << k : 0u;
                    } else if constexpr (FORM == 1) {
                        // balanced tree; the last two levels' thresholds come
                        // from the channel's row in LDS, the reads of all the
                        // group's codes of a level in flight together
                        uint32_t q[WN][4];
                        int32_t t[WN][4];
                        constexpr int KS = WM * WN >= 6 ? 2 : 4;  // channels at a time (registers)
#pragma unroll
                        for (int k0 = 0; k0 < 4; k0 += KS) {
#pragma unroll
                            for (int k = k0; k < k0 + KS; ++k) {
                                const int32_t *col = sP + (ch + k) * 16;
                                const int32_t t3 = col[3], t7 = col[7], t11 = col[11];
#pragma unroll
                                for (int c = 0; c < WN; ++c) {
                                    q[c][k] = x[c][k] >= t7 ? 1u : 0u;
                                    q[c][k] = stair_bit(q[c][k], x[c][k], q[c][k] ? t11 : t3);
                                }
                            }
#pragma unroll
                            for (int l = 2; l >= 1; --l) {
#pragma unroll
                                for (int k = k0; k < k0 + KS; ++k)
#pragma unroll
                                    for (int c = 0; c < WN; ++c)
                                        t[c][k] = sP[(ch + k) * 16 + 2 * l * q[c][k] + (l - 1)];
#pragma unroll
                                for (int k = k0; k < k0 + KS; ++k)
#pragma unroll
                                    for (int c = 0; c < WN; ++c)
                                        q[c][k] = stair_bit(q[c][k], x[c][k], t[c][k]);
                            }
                            __builtin_amdgcn_sched_barrier(0);
                        }
#pragma unroll
                        for (int c = 0; c < WN; ++c)
                            word[c][g] = q[c][0] | (q[c][1] << BITS) | (q[c][2] << (2 * BITS)) | (q[c][3] << (3 * BITS));
                    } else if constexpr (FORM == 2) {
#pragma unroll
                        for (int k = 0; k < 4; ++k) {
                            const int32_t *col = sP + (ch + k) * 16;
                            if constexpr (NTH == 3) {
                                const int4 T = *(const int4 *)col;
#pragma unroll
                                for (int c = 0; c < WN; ++c)
                                    word[c][g] |= ((x[c][k] >= T.x ? 1u : 0u) + (x[c][k] >= T.y ? 1u : 0u) +
                                                   (x[c][k] >= T.z ? 1u : 0u)) << (k * BITS);
                            } else {
#pragma unroll 1
                                for (int j = 0; j < NTH; ++j) {
                                    const int32_t tj = col[j];
#pragma unroll
                                    for (int c = 0; c < WN; ++c)
                                        word[c][g] += x[c][k] >= tj ? 1u << (k * BITS) : 0u;
                                }
                            }
                        }
                    } else {
                        int32_t e[7][4], sum[4] = {0, 0, 0, 0};
#pragma unroll
                        for (int f = 0; f < (FORM == 3 ? 5 : (FORM == 4 ? 6 : 7)); ++f)
                            plan4(f, ch, e[f]);
                        if (BITS == 8) {
                            const int4 q = *(const int4 *)(sSum + ch);
                            sum[0] = q.x;
                            sum[1] = q.y;
                            sum[2] = q.z;
                            sum[3] = q.w;
#pragma unroll
                            for (int k = 0; k < 4; ++k)
                                if (FORM != 5 || e[6][k] != 0)
                                    e[0][k] = __builtin_elementwise_sub_sat(e[0][k], sum[k]);
                        }
                        if constexpr (FORM < 5) {
#pragma unroll
                            for (int c = 0; c < WN; ++c)
#pragma unroll
                                for (int k = 0; k < 4; ++k) {
                                    const int32_t ek[7] = {e[0][k], e[1][k], e[2][k], e[3][k], e[4][k], FORM == 4 ? e[5][k] : 0, 3};
                                    word[c][g] |= (FORM == 3 ? code3(x[c][k], ek) : code4(x[c][k], ek)) << (k * BITS);
                                }
                        } else {
                            // one code at a time, everything rotated through
                            // the first registers (rare: small code)
                            int32_t z[4 * WN];
                            uint32_t w[WN];
#pragma unroll
                            for (int c = 0; c < WN; ++c) {
                                w[c] = 0;
#pragma unroll
                                for (int k = 0; k < 4; ++k)
                                    z[k * WN + c] = x[c][k];
                            }
                            int c = 0, sh = 0;
#pragma unroll 1
                            for (int t = 0; t < 4 * WN; ++t) {
                                const int32_t ek[7] = {e[0][0], e[1][0], e[2][0], e[3][0], e[4][0], e[5][0], e[6][0]};
                                const uint32_t wn = w[0] | (code_any(z[0], ek, sum[0]) << sh);
#pragma unroll
                                for (int v = 0; v + 1 < 4 * WN; ++v)
                                    z[v] = z[v + 1];
#pragma unroll
                                for (int v = 0; v + 1 < WN; ++v)
                                    w[v] = w[v + 1];
                                w[WN - 1] = wn;
                                if (++c == WN) {
                                    c = 0;
                                    sh += BITS;
#pragma unroll
                                    for (int v = 0; v < 3; ++v) {
#pragma unroll
                                        for (int f = 0; f < 7; ++f)
                                            e[f][v] = e[f][v + 1];
                                        sum[v] = sum[v + 1];
                                    }
                                }
                            }
#pragma unroll
                            for (int v = 0; v < WN; ++v)
                                word[v][g] = w[v];
                        }
                    }
                    // computed here (the compiler would sink it into the
                    // stores' branches and keep its inputs in scratch memory)
#pragma unroll
                    for (int c = 0; c < WN; ++c)
                        __asm__ volatile("" : "+v"(word[c][g]));
                    __builtin_amdgcn_sched_barrier(0);
                }
                emit(i, word);
            }
        };
        if (BITS == 1 || (BITS != 8 && thr)) {
            if constexpr (NTH == 1)
                run(StreamInt<0>());
            else if (NTH == 15 && (votes & 4))
                run(StreamInt<1>());
            else
                run(StreamInt<2>());
        } else if constexpr (BITS != 1) {
            if (votes & 1)
                run(StreamInt<3>());
            else if (votes & 2)
                run(StreamInt<4>());
            else
                run(StreamInt<5>());
        }
        if (direct)
            return;
        stream_barrier();
        const int np = min(PT, a.npix - p0);
        uint8_t *y = a.y + (size_t)p0 * (uint32_t)a.ypb + ob0;
        if ((a.ypb & 3) == 0) {
            constexpr int NQ = OB / 4;
            for (int i = tid; i < np * NQ; i += 256) {
                const int p = i / NQ, q = i % NQ;
                if (4 * q < obn)
                    *(uint32_t *)(y + (size_t)p * (uint32_t)a.ypb + 4 * q) = *(const uint32_t *)(sC + p * CS + 4 * q);
            }
        } else {
            for (int i = tid; i < np * OB; i += 256) {
                const int p = i / OB, q = i % OB;
                if (q < obn)
                    y[(size_t)p * (uint32_t)a.ypb + q] = sC[p * CS + q];
            }
        }
        return;
    }

    // pooled: lane = channel; register group g of a matrix tile is one 2x2
    // window, its code the largest accumulator's (codes are non-decreasing in
    // the accumulator, except where the direct form's multiplier is negative:
    // there the codes are compared); codes to LDS, one byte each
    if constexpr (MODE == STREAM_POOL) {
        uint8_t *sC = smem + a.off_out;
        constexpr int cs = MT + 16;
#pragma unroll
        for (int i = 0; i < WM; ++i) {
            const int ch = wch * 32 * WM + i * 32 + r32;
            int32_t e[7], sum = 0;
            if (!thr) {
#pragma unroll
                for (int f = 0; f < 7; ++f)
                    e[f] = sP[f * MT + ch];
                if (BITS == 8)
                    sum = sSum[ch];
                fold(e, sum);
            }
#pragma unroll
            for (int c = 0; c < WN; ++c) {
                int32_t x[4];
                uint32_t r[4];
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    x[g] = max(max((int32_t)acc[i][c][4 * g], (int32_t)acc[i][c][4 * g + 1]),
                               max((int32_t)acc[i][c][4 * g + 2], (int32_t)acc[i][c][4 * g + 3]));
                    r[g] = 0;
                }
                if (thr) {
                    const int32_t *col = sP + ch;
                    if (NTH == 15 && (votes & 4)) {
                        const int32_t t3 = col[3 * MT], t7 = col[7 * MT], t11 = col[11 * MT];
#pragma unroll
                        for (int g = 0; g < 4; ++g) {
                            uint32_t q = x[g] >= t7 ? 1u : 0u;
                            q = stair_bit(q, x[g], q ? t11 : t3);
                            q = stair_bit(q, x[g], col[MT * (4 * q + 1)]);
                            r[g] = stair_bit(q, x[g], col[MT * (2 * q)]);
                        }
                    } else {
#pragma unroll 1
                        for (int j = 0; j < NTH; ++j) {
                            const int32_t tj = col[j * MT];
#pragma unroll
                            for (int g = 0; g < 4; ++g)
                                r[g] += x[g] >= tj ? 1u : 0u;
                        }
                    }
                } else if (votes & 1) {
#pragma unroll
                    for (int g = 0; g < 4; ++g)
                        r[g] = code3(x[g], e);
                } else if (votes & 2) {
#pragma unroll
                    for (int g = 0; g < 4; ++g)
                        r[g] = code4(x[g], e);
                } else {
                    // rare: one accumulator at a time, rotated through z[0]
                    int32_t z[16];
#pragma unroll
                    for (int v = 0; v < 16; ++v)
                        z[v] = (int32_t)acc[i][c][v];
                    uint32_t packed = 0;
#pragma unroll 1
                    for (int v = 0; v < 16; ++v) {
                        const uint32_t code = code_any(z[0], e, sum);
#pragma unroll
                        for (int k = 0; k < 15; ++k)
                            z[k] = z[k + 1];
                        const uint32_t sh = 8 * (v >> 2);
                        const uint32_t old = (packed >> sh) & 255u;
                        packed = (packed & ~(255u << sh)) | (max(old, code) << sh);
                    }
#pragma unroll
                    for (int g = 0; g < 4; ++g)
                        r[g] = (packed >> (8 * g)) & 255u;
                }
                uint8_t *d = sC + ((wpx * 32 * WN + c * 32) / 4 + h) * cs + ch;
#pragma unroll
                for (int g = 0; g < 4; ++g)
                    d[2 * g * cs] = (uint8_t)r[g];
            }
        }
        stream_barrier();
        // copy-out: the tile's windows are consecutive
        constexpr int CPW = 32 / BITS;              // codes per output word
        const int q0 = p0 >> 2;
        const int np = min(PT / 4, (a.npix >> 2) - q0);
        uint8_t *y = a.y + (size_t)q0 * (uint32_t)a.ypb + ob0;
        if ((a.ypb & 3) == 0) {
            constexpr int NQ = OB / 4;
            for (int i = tid; i < np * NQ; i += 256) {
                const int p = i / NQ, q = i % NQ;
                if (4 * q < obn)
                    *(uint32_t *)(y + (size_t)p * (uint32_t)a.ypb + 4 * q) = pack_codes_word<BITS>(sC + p * cs + q * CPW);
            }
        } else {
            for (int i = tid; i < np * OB; i += 256) {
                const int p = i / OB, q = i % OB;
                if (q < obn)
                    y[(size_t)p * (uint32_t)a.ypb + q] = pack_codes_byte<BITS>(sC + p * cs + q * (8 / BITS));
            }
        }
    }
}

// Part 0: one tap per step, whole items; part 1: the others.  XP: packed input
// tiles (one tap per step).
template <int BITS, int PART, bool XP = false>
hipError_t launch_conv_stream_bits(const StreamArgs &a, int variant, hipStream_t s)
{
    const int mode = a.pool ? STREAM_POOL : (a.epi == EPI_RAW32 ? STREAM_RAW : STREAM_CODES);
    const dim3 grid((unsigned)(a.ptiles * a.mtiles));
#define QNN_STREAM_M(V_, WM_, WN_, WCH_, G_, MODE_, LG_, TAIL_, PW_)                                  \
    if (variant == V_ && mode == MODE_ && a.lg == LG_ && a.pw1 == PW_) {                              \
        auto *k = conv_stream_kernel<BITS, WM_, WN_, WCH_, G_, MODE_, LG_, TAIL_, PW_, XP>;               \
        if (a.lds_bytes > 64 * 1024) {                                                                \
            static std::atomic<uint64_t> devices{0};                                                  \
            allow_large_lds((const void *)k, devices);                                                \
        }                                                                                             \
        hipLaunchKernelGGL(k, grid, dim3(256), a.lds_bytes, s, a);                                    \
        return hipGetLastError();                                                                     \
    }
#define QNN_STREAM_L(V_, WM_, WN_, WCH_, G_, LG_, TAIL_, PW_)                                         \
    QNN_STREAM_M(V_, WM_, WN_, WCH_, G_, STREAM_CODES, LG_, TAIL_, PW_)                               \
    QNN_STREAM_M(V_, WM_, WN_, WCH_, G_, STREAM_RAW, LG_, TAIL_, PW_)                                 \
    if constexpr (BITS != 1) {                                                                        \
        QNN_STREAM_M(V_, WM_, WN_, WCH_, G_, STREAM_POOL, LG_, TAIL_, PW_)                            \
    }
    // one-tap filters (of one tap per step): G = 1 only, packed at 4 bits
#define QNN_STREAM_0(V_, WM_, WN_, WCH_, G_)                                                          \
    QNN_STREAM_L(V_, WM_, WN_, WCH_, G_, 2, false, false)                                             \
    if constexpr (G_ == 1 && (XP || BITS != 4)) {                                                     \
        QNN_STREAM_L(V_, WM_, WN_, WCH_, 1, 2, false, true)                                           \
    }
#define QNN_STREAM_1(V_, WM_, WN_, WCH_, G_)                                                          \
    QNN_STREAM_L(V_, WM_, WN_, WCH_, G_, 2, true, false)                                              \
    if constexpr (G_ == 1 && (XP || BITS != 4)) {                                                     \
        QNN_STREAM_L(V_, WM_, WN_, WCH_, 1, 2, true, true)                                            \
    }                                                                                                 \
    if constexpr (!XP) {                                                                              \
        QNN_STREAM_L(V_, WM_, WN_, WCH_, G_, 1, true, false)                                          \
        QNN_STREAM_L(V_, WM_, WN_, WCH_, G_, 0, true, false)                                          \
    }
    if constexpr (PART == 0) {
        QNN_STREAM_VARIANTS(QNN_STREAM_0)
    } else {
        QNN_STREAM_VARIANTS_TAIL(QNN_STREAM_1)
    }
#undef QNN_STREAM_0
#undef QNN_STREAM_1
#undef QNN_STREAM_L
#undef QNN_STREAM_M
    return hipErrorInvalidValue;
}

}  // namespace qnn
