"""Which kernel the library picks, worked out on the CPU: route_probe.hip is
the library's own host code (argument checks, planners, dispatch) with every
launch recorded in place of made.  Needs hipcc; no GPU."""
import collections
import ctypes
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
EPI = {"requant": 0, "thresh1": 1, "raw32": 2, "stair": 3}
KERNELS = ("none", "stream", "xnor", "image", "linear", "mfma16", "mfma32", "fp4", "pool", "relu")

# kernel, then for "stream": tile, mode (0 codes, 1 raw sums, 2 pooled), lg, tail, one_tap, packed (and lds, dw, nblk);
# "xnor": tile = words (resident, mode 1; else per step); "image": tile = bytes of a pixel
Route = collections.namedtuple("Route", "status kernel tile mode lg tail one_tap packed lds dw nblk")


class _Raw(ctypes.Structure):
    _fields_ = [(f, ctypes.c_int32) for f in ("kernel", "tile", "mode", "lg", "tail", "pw", "xp", "lds", "dw", "nblk")]


def build(folder):
    lib = os.path.join(str(folder), "libroute.so")
    subprocess.check_call([HIPCC, "-x", "hip", "--offload-host-only", "--offload-arch=gfx950", "-nogpulib", "-no-hip-rt",
                           "-O2", "-std=c++17", "-fPIC", "-shared", "-Wl,-Bsymbolic",
                           "-I" + os.path.join(ROOT, "include"),
                           os.path.join(ROOT, "tests", "route_probe.hip"), "-o", lib])
    L = ctypes.CDLL(lib)
    P, I = ctypes.c_void_p, ctypes.c_int32
    L.probe_conv.restype = I
    L.probe_conv.argtypes = [P, I, P, I, P, I, P]
    L.probe_resident.restype = I
    L.probe_resident.argtypes = [I, I, I, I, P]
    return L


def route(L, bits, n, h, w, c, m, kh, kw, stride=1, pad=0, epi="requant", pool=False):
    """The route of one layer; stride and pad are numbers or (vertical, horizontal)."""
    sh, sw = stride if isinstance(stride, tuple) else (stride, stride)
    ph, pw = pad if isinstance(pad, tuple) else (pad, pad)
    ho, wo = (h + 2 * ph - kh) // sh + 1, (w + 2 * pw - kw) // sw + 1
    d = 2 if pool else 1
    obits = {"requant": bits, "stair": bits, "thresh1": 1, "raw32": 32}[epi]
    x = (ctypes.c_int32 * 5)(n, h, w, c, bits)
    y = (ctypes.c_int32 * 5)(n, ho // d, wo // d, m, obits)
    g = (ctypes.c_int32 * 6)(kh, kw, sh, sw, ph, pw)
    r = _Raw()
    st = L.probe_conv(x, m, g, EPI[epi], y, int(pool), ctypes.byref(r))
    v = [getattr(r, f) for f, _ in _Raw._fields_]
    return Route(st, KERNELS[v[0]], *v[1:])
