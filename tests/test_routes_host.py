"""Which kernel the library picks for a layer, worked out on the CPU
(routes.py: the library's own dispatch with its launches recorded)."""
import ctypes
import math
import random

import pytest

import layers
import routes


# layers with both kernels' measured times in us (tile kernel, streaming
# kernel; graph replays): (bits, n, h, w, c, m, kh, kw, stride, pad, epilogue,
# pooled), the kernel that has to be picked
MEASURED = [
    # wide rows: the streaming kernel's input tile is whole rows
    ((4, 3, 166, 640, 8, 64, 7, 7, 1, 3, "requant", False), "mfma32", 29.3, 145.8),
    ((4, 6, 62, 448, 96, 16, 3, 3, 1, 1, "requant", True), "mfma32", 15.7, 74.7),
    ((2, 8, 189, 1024, 16, 32, 3, 3, 1, 1, "requant", True), "mfma32", 45.8, 186.4),
    ((8, 19, 90, 320, 48, 16, 3, 3, 1, 1, "requant", True), "mfma32", 34.4, 134.2),
    ((8, 6, 99, 640, 8, 48, 7, 7, 1, 3, "requant", False), "mfma16", 65.1, 203.7),
    ((4, 29, 22, 640, 64, 16, 3, 3, 1, 1, "raw32", False), "mfma16", 30.5, 82.0),
    ((2, 4, 213, 640, 16, 32, 5, 5, 1, 2, "stair", False), "mfma32", 29.7, 100.6),
    ((8, 80, 50, 113, 48, 32, 3, 3, 1, 1, "requant", False), "mfma32", 28.2, 58.3),
    # small grids: one workgroup per compute unit walks the whole reduction
    ((4, 3, 11, 8, 544, 56, 3, 3, 1, 1, "raw32", False), "mfma16", 14.1, 32.7),
    ((4, 29, 7, 7, 928, 96, 3, 1, 1, (1, 0), "raw32", False), "mfma16", 10.4, 26.6),
    ((4, 6, 3, 25, 224, 12, 3, 3, 1, 1, "requant", True), "mfma32", 9.4, 17.2),
    ((8, 4, 4, 24, 80, 29, 5, 5, 1, 2, "raw32", False), "mfma16", 10.6, 18.6),
    ((2, 2, 5, 8, 704, 43, 3, 3, 1, 1, "stair", False), "mfma16", 15.8, 27.6),
    ((8, 4, 7, 7, 1312, 491, 3, 1, 1, (1, 0), "requant", False), "mfma16", 22.4, 36.5),
    # and layers of both kinds that the streaming kernel is faster at
    ((4, 1, 253, 512, 120, 128, 5, 5, 1, 2, "raw32", False), "stream", 266.9, 96.8),
    ((2, 16, 169, 320, 16, 64, 3, 3, 1, 1, "raw32", False), "stream", 178.1, 49.4),
    ((8, 2, 144, 384, 16, 96, 3, 3, 1, 1, "raw32", False), "stream", 52.3, 17.3),
    ((8, 1, 224, 72, 60, 128, 7, 7, 1, 3, "requant", True), "stream", 146.8, 28.3),
    ((2, 3, 26, 117, 208, 256, 5, 5, 1, 2, "requant", False), "stream", 362.2, 36.5),
    ((2, 23, 13, 10, 1488, 298, 1, 1, 1, 0, "raw32", False), "stream", 71.0, 11.4),
    ((4, 45, 41, 20, 248, 158, 1, 1, 3, 0, "raw32", False), "stream", 65.2, 8.5),
    ((8, 4, 58, 65, 128, 256, 5, 5, 1, 2, "requant", False), "stream", 153.5, 27.5),
    ((2, 27, 27, 29, 96, 48, 1, 1, 3, 0, "stair", True), "stream", 14.7, 4.3),
]


@pytest.mark.parametrize("layer,kernel,tile_us,stream_us", MEASURED)
def test_the_faster_kernel_is_picked(route_lib, layer, kernel, tile_us, stream_us):
    r = routes.route(route_lib, *layer)
    assert r.status == 0 and r.kernel == kernel
    assert (r.kernel == "stream") == (stream_us < tile_us)


def test_a_failed_occupancy_query_is_not_kept(route_lib):
    """The image kernels' resident workgroups: an answer is kept for its kernel
    and local memory, a failure (or no workgroup) is asked again."""
    asked = ctypes.c_int32(0)

    def ask(kernel, lds, status, n):
        return route_lib.probe_resident(kernel, lds, status, n, ctypes.byref(asked))

    assert ask(1, 4096, 1, 0) == 1 and asked.value == 1     # failed
    assert ask(1, 4096, 0, 0) == 1 and asked.value == 2     # no workgroup
    assert ask(1, 4096, 0, 3) == 3 and asked.value == 3
    assert ask(1, 4096, 0, 7) == 3 and asked.value == 3     # kept
    assert ask(1, 8192, 0, 2) == 2 and ask(2, 4096, 0, 5) == 5 and asked.value == 5


def test_large_local_memory_is_asked_for_once_per_device(route_lib):
    calls = [route_lib.probe_large_lds(dev, status) for dev, status in
             ((0, 1), (0, 0), (0, 0), (3, 0), (0, 0), (3, 0), (70, 0), (70, 0))]
    assert calls == [1, 2, 2, 3, 3, 3, 4, 5]  # (a failure, and a device past the table, are asked for again)


def test_stream_layers_take_every_instance_that_is_picked(route_lib):
    """Every layer of the table takes the instance written beside it, and random
    layers take none that the table lacks."""
    table = set()
    for layer, want in layers.stream_layers():
        r = routes.route(route_lib, *layer)
        got = (r.tile, r.lg, r.tail, r.one_tap, r.packed, r.dw, int(r.nblk > 1))
        assert r.kernel == "stream" and got == want, (layer, r)
        table.add((layer[0], layer[10], layer[11]) + want[:5])
    rng = random.Random(17)

    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    seen = 0
    for _ in range(60000):
        bits = rng.choice([8, 4, 2, 1])
        pool = bits != 1 and rng.random() < 0.3
        epi = rng.choice(["thresh1", "raw32"] if bits == 1 else
                         ["requant"] + ([] if pool else ["raw32"]) + (["stair"] if bits < 8 else []))
        n, h, w = log_int(1, 3000), log_int(2, 80), log_int(2, 80)
        c, m = 32 // bits * log_int(1, 64), log_int(1, 300)
        k, s = rng.choice([1, 1, 2, 3, 3, 5]), rng.choice([1, 1, 2, 3])
        pad = rng.choice([0, k // 2])
        if min(h, w) + 2 * pad - k < s:
            continue
        r = routes.route(route_lib, bits, n, h, w, c, m, k, k, s, pad, epi, pool)
        if r.status == 0 and r.kernel == "stream":
            seen += 1
            assert (bits, epi, pool, r.tile, r.lg, r.tail, r.one_tap, r.packed) in table
    assert seen > 20000


@pytest.mark.parametrize("layer,words,resident", layers.XNOR)
def test_xnor_layers_take_the_popcount_kernels(route_lib, layer, words, resident):
    r = routes.route(route_lib, *layer)
    assert (r.status, r.kernel, r.tile, r.mode) == (0, "xnor", words, resident)


@pytest.mark.parametrize("layer,tile", layers.POOLED_TILES)
def test_pooled_layers_on_the_tile_kernel(route_lib, layer, tile):
    r = routes.route(route_lib, *layer)
    assert (r.status, r.kernel, r.tile, r.mode) == (0, "mfma32", tile, 2)


def test_layers_of_the_other_streaming_tests(route_lib):
    """The layers that tests name by their kernel take it."""
    for pool in (False, True):
        for (n, h, w, c, m, k, s) in layers.PACKED_POOLED if pool else layers.PACKED:
            for epi in ("requant",) if pool else ("requant", "raw32", "stair"):
                r = routes.route(route_lib, 4, n, h, w, c, m, k, k, s, k // 2, epi, pool)
                assert r.kernel == "stream" and r.packed, (n, h, w, c, m, k, s, epi, pool)
    for (h, w, c, m, k) in layers.WIDE_BINARY:
        assert routes.route(route_lib, 1, 1, h, w, c, m, k, k, 1, k // 2, "thresh1").kernel == "xnor"
    for bits, n, K, m, kernel in layers.EXTREME_SUMS:
        assert routes.route(route_lib, bits, n, 1, 1, K, m, 1, 1, 1, 0, "raw32").kernel == kernel
