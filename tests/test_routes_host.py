"""Which kernel the library picks for a layer, worked out on the CPU
(routes.py: the library's own dispatch with its launches recorded)."""
import ctypes

import pytest

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
