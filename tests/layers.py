"""Layers that the library's dispatch sends to a kernel that a test is about.
The host tests check that it does (test_routes_host.py), the GPU tests compare
the kernel's output on them with the oracle's."""
import os

HERE = os.path.dirname(os.path.abspath(__file__))


def stream_layers():
    """((bits, n, h, w, c, m, kh, kw, stride, pad, epilogue, pooled), (tile, lg, tail, one_tap, packed, dw, blocks)):
    one layer for every combination of streaming kernel instance, epilogue and channel blocks (dw: the last one ends
    inside a 16-byte item; blocks: more than one) that is picked."""
    out = []
    with open(os.path.join(HERE, "golden", "stream_layers.txt")) as f:
        for line in f:
            if line.startswith("#"):
                continue
            layer, route = line.split("|")
            v = layer.split()
            bits, n, h, w, c, m, k, s, pad = map(int, v[:9])
            out.append(((bits, n, h, w, c, m, k, k, s, pad, v[9], v[10] == "1"), tuple(map(int, route.split()))))
    return out


def _xnor():
    # (layer, words the instance holds, or takes at a time; 1: whole volume in
    # registers).  Rows too wide for the streaming kernel's input tile, or more
    # than 64 taps.
    out = []
    for kd in range(8, 136, 8):
        # words of a pixel a multiple of four (16-byte gather) ...
        out.append(((1, 1, 2, 1100, 16 * kd, 40, 2, 1, 1, 0, "thresh1" if kd % 16 else "raw32", False), kd, 1))
        # ... and not
        cd, taps = (2, kd // 2) if kd <= 64 else (1, kd)
        kh, kw = (taps, 1) if taps <= 64 else (taps // 8, 8)
        w = 10300 // kh + kw if taps <= 64 else 9 + kw
        out.append(((1, 1, kh + 1, w, 32 * cd, 33, kh, kw, 1, 0, "raw32" if kd % 16 else "thresh1", False), kd, 1))
    # volumes that are no multiple of eight words, or more than 128
    out += [((1, 1, 3, 700, 512, 33, 3, 3, 1, 1, "thresh1", False), 8, 0),
            ((1, 1, 3, 1100, 128, 40, 3, 1, 1, 0, "raw32", False), 4, 0),
            ((1, 1, 3, 1200, 64, 31, 3, 1, 1, 0, "thresh1", False), 2, 0),
            ((1, 1, 9, 40, 32, 12, 9, 9, 1, 4, "thresh1", False), 1, 0),
            ((1, 2, 3, 9000, 32, 8, 1, 3, 1, 0, "raw32", False), 1, 0)]
    return out


XNOR = _xnor()

# pooled layers on the 32x32 tile kernel: the layer, its tile (10 x channel tiles + output tiles of a wave)
POOLED_TILES = [
    ((8, 4, 3, 83, 96, 8, 3, 3, 2, 1, "requant", True), 11),
    ((8, 1, 5, 3, 80, 8, 5, 5, 2, 2, "requant", True), 12),
    ((8, 1, 72, 926, 4, 33, 1, 1, 1, 0, "requant", True), 21),
    ((8, 2, 4, 911, 4, 33, 3, 3, 2, 1, "requant", True), 22),
    ((4, 2, 30, 15, 160, 8, 2, 2, 2, 0, "requant", True), 11),
    ((4, 1, 2, 3, 136, 8, 2, 2, 2, 1, "requant", True), 12),
    ((4, 3, 3, 95, 160, 33, 2, 2, 2, 1, "requant", True), 21),
    ((4, 2, 2, 782, 8, 40, 1, 1, 1, 0, "requant", True), 22),
    ((4, 2, 40, 11, 160, 8, 2, 2, 2, 0, "stair", True), 11),
    ((4, 1, 4, 4, 160, 8, 2, 2, 2, 0, "stair", True), 12),
    ((4, 2, 3, 68, 160, 33, 3, 3, 2, 1, "stair", True), 21),
    ((4, 2, 5, 913, 8, 40, 2, 2, 2, 0, "stair", True), 22),
    ((2, 16, 6, 5, 192, 8, 3, 3, 2, 1, "requant", True), 11),
    ((2, 1, 4, 4, 272, 8, 2, 2, 2, 0, "requant", True), 12),
    ((2, 1, 3, 3, 320, 40, 5, 5, 2, 2, "requant", True), 21),
    ((2, 1, 8, 818, 16, 33, 1, 1, 1, 0, "requant", True), 22),
    ((2, 1, 8, 75, 320, 8, 2, 2, 2, 1, "stair", True), 11),
    ((2, 1, 3, 3, 272, 8, 2, 2, 1, 0, "stair", True), 12),
    ((2, 1, 4, 4, 320, 96, 5, 5, 2, 2, "stair", True), 21),
    ((2, 2, 2, 598, 16, 40, 2, 2, 2, 1, "stair", True), 22),
]

# 4-bit layers whose input tile the streaming kernel keeps packed: (n, h, w, c, m, k, stride), plain and pooled
PACKED = [(137, 13, 70, 64, 72, 3, 2), (46, 40, 41, 64, 40, 5, 2), (94, 40, 41, 88, 40, 3, 2),
          (87, 40, 41, 64, 130, 1, 1), (63, 20, 41, 88, 130, 1, 2), (40, 11, 9, 72, 34, 1, 1)]
PACKED_POOLED = [(200, 13, 60, 64, 72, 3, 2)] + PACKED[1:]

# 1-bit layers past the streaming kernel: (h, w, c, m, k) of one image with pads k // 2
WIDE_BINARY = [(3, 1200, 512, 33, 3), (2, 9000, 32, 8, 3), (9, 40, 32, 12, 9)]

# fully connected layers of extreme codes: bits, images, K, outputs, kernel; K up to the largest whose sums the e2m1
# path's fp32 accumulator holds exactly
EXTREME_SUMS = [(2, 640, 2796160, 640, "stream"), (1, 3, 1 << 24, 40, "stream"), (1, 3, (1 << 24) + 32, 40, "xnor")]
