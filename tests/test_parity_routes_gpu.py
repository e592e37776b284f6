"""GPU parity, byte for byte against the oracle, of every kernel instance that
the library's dispatch picks by itself and no other test names: the streaming
kernel's (one layer for each instance and epilogue), the popcount kernels' and
the pooled 32x32 tiles'.  test_routes_host.py checks that the layers take them.
Images are independent of one another, so of large batches the oracle computes
the first, the last and a few between."""
import numpy as np
import pytest

import layers
from gpu_helpers import EPI, compare, dev, log, threads

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def qnn():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1908_11263_amd as q
    q.device_check()
    return q


# multipliers and added shift of the compression's forms: 32-bit and 64-bit
# plans, multipliers of either sign, multipliers past 2^shift
FORMS = [((1 << 13, 1 << 14), 0), ((1 << 20, 1 << 21), 7), ((-(1 << 13), 1 << 13), 0), ((1 << 28, 1 << 29), 15)]


def check(qnn, orc, layer, seed):
    import torch
    bits, n, h, w, c, m, kh, kw, s, pad, epi, pool = layer
    log("case", layer, "seed", seed)
    rng = np.random.default_rng(seed)
    K, hi = kh * kw * c, (1 << bits) - 1
    x = rng.integers(0, 256, size=(n, h, w, c * bits // 8), dtype=np.uint8)
    wt = rng.integers(0, 256, size=(m, K * bits // 8), dtype=np.uint8)
    # accumulators spread over about sd: outputs over the whole range of codes
    sd = K ** 0.5 * (hi * 2 ** (bits - 1) / 3 if bits > 1 else 1)
    bias = rng.integers(-int(sd) - 1, int(sd) + 2, size=m).astype(np.int32)
    mult = shift = thresh = None
    clip = (0, hi)
    if epi == "requant":
        rg, more = FORMS[seed % len(FORMS)]
        sh = max(0, int(np.log2(3 * sd / (hi + 1))) + 14 + more)
        mult = rng.integers(rg[0], rg[1], size=m).astype(np.int32)
        shift = np.full(m, min(sh, 62), np.int8)
    elif epi != "raw32":
        thresh = rng.integers(-int(2 * sd) - 2, int(2 * sd) + 3, size=(m, hi if epi == "stair" else 1)).astype(np.int32)
        if seed % 3:
            thresh.sort(axis=1)  # (staircases: sorted ones have a form of their own)
    f = qnn.conv2d_maxpool if pool else qnn.conv2d
    y = f(dev(x), (n, h, w, c), bits, dev(wt), m, kh, kw, (s, s), (pad, pad), epi, bias=dev(bias), mult=dev(mult),
          shift=dev(shift), thresh=dev(thresh), clip=clip)
    torch.cuda.synchronize()
    some = sorted({0, 1 % n, n // 3, n // 2, max(0, n - 2), n - 1}) if n > 8 else list(range(n))
    _, want = orc.conv2d(x[some], (len(some), h, w, c), bits, wt, m, kh, kw, (s, s), (pad, pad), EPI[epi], bias, mult,
                         shift, thresh, clip, nthreads=threads())
    if pool:
        ho, wo = (h + 2 * pad - kh) // s + 1, (w + 2 * pad - kw) // s + 1
        want = orc.maxpool2d(want, (len(some), ho, wo, m), bits, 2, 2, 2, 2)
    compare(y.cpu().numpy()[some], want, "%s" % (layer,))


STREAM = layers.stream_layers()


@pytest.mark.parametrize("bits", [8, 4, 2, 1])
@pytest.mark.parametrize("tile", range(9))
def test_streaming_instances(qnn, orc, bits, tile):
    mine = [v for v in enumerate(STREAM) if v[1][0][0] == bits and v[1][1][0] == tile]
    assert mine
    for i, (layer, _) in mine:
        check(qnn, orc, layer, i)


@pytest.mark.parametrize("layer,words,resident", layers.XNOR)
def test_popcount_instances(qnn, orc, layer, words, resident):
    check(qnn, orc, layer, words + resident)


@pytest.mark.parametrize("layer,tile", layers.POOLED_TILES)
def test_pooled_tiles(qnn, orc, layer, tile):
    for seed in range(4):
        check(qnn, orc, layer, seed)


@pytest.mark.parametrize("bits,n,K,m,kernel", layers.EXTREME_SUMS)
def test_largest_sums_of_the_e2m1_instruction(qnn, bits, n, K, m, kernel):
    """Extreme codes throughout, at the longest reductions whose partial sums the
    fp32 accumulator holds exactly (1 bit: and one past it, on the popcount
    kernel): every sum is known, some are +-2^24."""
    import torch
    log("case extreme sums bits=%d K=%d %s" % (bits, K, kernel))
    row = K * bits // 8
    x = torch.full((n, row), 0xFF, dtype=torch.uint8, device="cuda")       # 3; +1
    w = torch.full((m, row), 0xAA if bits == 2 else 0xFF, dtype=torch.uint8, device="cuda")  # -2; +1
    x[1::2] = 0x55 if bits == 2 else 0                                      # 1; -1
    w[1::2] = 0x55 if bits == 2 else 0                                      # 1; -1
    w[2, row // 2:] = 0x55 if bits == 2 else 0                              # half and half
    y = qnn.linear(x, (n, 1, 1, K), bits, w, m, "raw32")
    torch.cuda.synchronize()
    xv = np.where(np.arange(n) % 2, 1, 3) if bits == 2 else np.where(np.arange(n) % 2, -1, 1)
    wv = np.where(np.arange(m) % 2, 1, -2) if bits == 2 else np.where(np.arange(m) % 2, -1, 1)
    total = wv.astype(np.int64) * K
    first = row // 2 * 8 // bits
    total[2] = wv[2] * first + wv[1] * (K - first)
    want = xv.astype(np.int64)[:, None] * total[None, :]
    assert np.abs(want).max() in (6 * K, K)
    compare(y.cpu().numpy().reshape(n, m).astype(np.int64), want, "extreme sums int%d" % bits)
