"""GPU parity of general layers (most on the streaming implicit-GEMM kernel; the
small narrow ones at 4 and 2 bits on the 16x16 tiles) against the oracle,
byte for byte, at the sizes where the streaming kernel's tiles, blocks and
loads end: partly filled channel and output tiles, tiles that run on into the
next image, narrow pixels (several taps per step), pixels that end inside a
16-byte item or a 64-byte block, several channel blocks, one-tap filters,
strides, whole-image filters, every epilogue and plan form."""
import pytest

import layers
import synth
from gpu_helpers import compare, dev, gpu_conv, oracle_conv
from test_parity_pool_gpu import gpu_pool, oracle_pool

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def qnn():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1908_11263_amd as q
    q.device_check()
    return q


def layer(bits, n, h, w, c, m, k, stride=1, epi=None, mult=(1 << 10, 1 << 14), shift=None, seed=5, pad=None,
          stair_sorted=True):
    K = k * k * c
    hi = (1 << bits) - 1
    if shift is None:
        # codes spread over the range: 14-bit multipliers, accumulators of about K^.5 hi 2^(bits-1)
        shift = max(0, min(30, 14 + int(K ** 0.5).bit_length() + (bits - 1 if bits > 1 else 0) - 1))
    span = max(2, int(2 * K ** 0.5 * hi * (1 << max(0, bits - 2))))
    epi = epi or ("thresh1" if bits == 1 else "requant")
    return synth.conv_layer("stream_int%d" % bits, bits, n, h, w, c, m, k, k // 2 if pad is None else pad, seed,
                            (0, hi), (-(1 << (bits - 1)), (1 << (bits - 1)) - 1) if bits > 1 else None,
                            bias_rng=None if bits == 1 else (-span, span), mult_rng=mult, shift=shift,
                            clip=(0, hi) if epi == "requant" else None, thresh_rng=(-span, span), epi=epi,
                            stride=stride, stair_sorted=stair_sorted)


def epilogues(bits):
    return ["thresh1", "raw32"] if bits == 1 else (["requant", "raw32"] + ([] if bits == 8 else ["stair"]))


# packed bytes per pixel: words, parts of a 16-byte item, one item and a word,
# parts of a 64-byte staged block, whole blocks, blocks and a part
PIXELS = [4, 8, 12, 16, 20, 28, 32, 36, 48, 60, 64, 68, 96, 128, 132]


@pytest.mark.parametrize("bits", [8, 4, 2, 1])
@pytest.mark.parametrize("k", [1, 3])
def test_pixel_sizes(qnn, orc, bits, k):
    for i, pb in enumerate(PIXELS):
        if bits == 1 and pb > 68:
            continue
        c = pb * 8 // bits
        for j, epi in enumerate(epilogues(bits)):
            L = layer(bits, 3, 9 + i % 3, 7 + j, c, 33 + 8 * (i % 4), k, epi=epi, seed=100 * i + j)
            compare(gpu_conv(L), oracle_conv(orc, L), "%s pb=%d k=%d %s" % (L.name, pb, k, epi))


@pytest.mark.parametrize("bits", [8, 4, 2, 1])
def test_tiles_and_strides(qnn, orc, bits):
    u = 128 // bits  # channels of a 16-byte pixel
    for i, (n, h, w, c, m, k, s) in enumerate([
            (1, 1, 1, u, 32, 1, 1),             # one output
            (70, 3, 3, u, 32, 3, 1),            # a tile over many images
            (2, 17, 15, 4 * u, 128, 3, 1),      # whole channel tiles, ragged outputs
            (5, 14, 14, 8 * u, 160, 3, 1),      # several channel tiles and blocks
            (3, 33, 21, 4 * u, 72, 3, 2),       # stride 2: even and odd columns apart
            (2, 31, 29, 2 * u, 40, 5, 2),
            (2, 20, 23, u, 48, 3, 3),           # stride 3
            (3, 16, 18, 4 * u, 96, 1, 2),       # strided one-tap filter
            (2, 11, 70, u, 256, 3, 1),          # 256 channels, long rows
            (1, 9, 200, u, 64, 3, 1),           # rows longer than a tile
            (9, 4, 4, 2 * u, 130, 4, 1)]):      # whole-image filter (pad 0)
        L = layer(bits, n, h, w, c, m, k, stride=s, seed=40 + i, pad=0 if k == 4 else None)
        compare(gpu_conv(L), oracle_conv(orc, L), "%s case %d" % (L.name, i))
        if bits != 1 and L.ho > 1 and L.wo > 1:
            compare(gpu_pool(qnn, L), oracle_pool(orc, L), "%s case %d pooled" % (L.name, i))


@pytest.mark.parametrize("epi", ["requant", "raw32", "stair", "pool"])
def test_packed_input_tiles(qnn, orc, epi):
    """4-bit layers whose input tiles stay packed in local memory because more
    workgroups fit (whole and odd blocks; one-tap filters always do)."""
    for i, (n, h, w, c, m, k, s) in enumerate(layers.PACKED_POOLED if epi == "pool" else layers.PACKED):
        L = layer(4, n, h, w, c, m, k, stride=s, seed=60 + i, epi="requant" if epi == "pool" else epi)
        if epi == "pool":
            compare(gpu_pool(qnn, L), oracle_pool(orc, L), "packed case %d pooled" % i)
        else:
            compare(gpu_conv(L), oracle_conv(orc, L), "packed case %d %s" % (i, epi))


@pytest.mark.parametrize("bits", [8, 4, 2])
def test_plan_forms(qnn, orc, bits):
    """Multipliers and shifts of each form of the compression: 32-bit, 64-bit,
    offset (multiplier above 2^shift), negative and zero multipliers, shifts
    past the plans' range; plain and pooled."""
    for j, (mult, shift) in enumerate([((1 << 14, 1 << 15), 18), ((1 << 20, 1 << 21), 26), ((200, 300), 6),
                                       ((-(1 << 12), 1 << 12), 16), ((0, 1), 0), ((1 << 28, 1 << 30), 40)]):
        L = layer(bits, 2, 10, 12, 256 // bits, 44, 3, mult=mult, shift=shift, seed=70 + j)
        compare(gpu_conv(L), oracle_conv(orc, L), "%s plan %d" % (L.name, j))
        compare(gpu_pool(qnn, L), oracle_pool(orc, L), "%s plan %d pooled" % (L.name, j))


@pytest.mark.parametrize("bits", [4, 2])
def test_unsorted_staircase(qnn, orc, bits):
    L = layer(bits, 2, 13, 9, 256 // bits, 50, 3, epi="stair", stair_sorted=False)
    compare(gpu_conv(L), oracle_conv(orc, L), "%s unsorted" % L.name)
    compare(gpu_pool(qnn, L), oracle_pool(orc, L), "%s unsorted pooled" % L.name)


@pytest.mark.parametrize("bits", [8, 4, 2, 1])
def test_linear_long_reduction(qnn, orc, bits):
    """A fully connected layer large enough to leave the 16x16 kernel."""
    n, m, K = 300, 520, 4096
    L = layer(bits, n, 1, 1, K, m, 1, epi="raw32", seed=9)
    y = qnn.linear(dev(L.x), (n, 1, 1, K), bits, dev(L.wt), m, "raw32", bias=dev(L.bias))
    compare(y.cpu().numpy(), oracle_conv(orc, L), "linear int%d" % bits)


def test_wide_binary_rows_take_the_popcount_kernel(qnn, orc):
    """Rows too wide for the streaming kernel's input tile."""
    for (h, w, c, m, k) in layers.WIDE_BINARY:
        L = layer(1, 1, h, w, c, m, k, seed=w)
        compare(gpu_conv(L), oracle_conv(orc, L), "wide int1 %d" % w)
