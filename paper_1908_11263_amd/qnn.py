"""ctypes binding of the gfx950 quantized-convolution library (libqnn.so).

Argument marshalling only: every computation runs in the library's HIP
kernels.  Device tensors are torch tensors on the current HIP device; work is
enqueued on torch's current stream.  If the library is not built the import
of any entry point raises, there is no fallback.

Tensor conventions follow the C ABI (include/qnn.h): packed NHWC uint8
activations, packed M x kh x kw x C uint8 weights, the lower channel in the
less significant bits, int32 outputs for the raw epilogue.
"""
import ctypes
import os
import re
import struct

HERE = os.path.dirname(os.path.abspath(__file__))
# QNN_LIBRARY names another build of the same sources (the sanitizer test
# loads a host-instrumented build)
LIB_PATH = os.environ.get("QNN_LIBRARY") or os.path.join(HERE, "libqnn.so")
HEADER = os.path.join(os.path.dirname(HERE), "include", "qnn.h")

EPI_REQUANT, EPI_THRESH1, EPI_RAW32, EPI_STAIR = 0, 1, 2, 3
# qnn_tile.kernel values (include/qnn.h)
TILE_MFMA16, TILE_MFMA32, TILE_FP4, TILE_IMAGE = 16, 32, 4, 1
_EPI_NAMES = {"requant": EPI_REQUANT, "thresh1": EPI_THRESH1, "raw32": EPI_RAW32, "stair": EPI_STAIR}

STATUS = {
    0: "QNN_OK", 1: "QNN_ERR_NULL", 2: "QNN_ERR_BITS", 3: "QNN_ERR_SHAPE", 4: "QNN_ERR_PARAM",
    5: "QNN_ERR_ALIGN", 6: "QNN_ERR_OVERFLOW", 7: "QNN_ERR_UNSUPPORTED", 8: "QNN_ERR_DEVICE",
    9: "QNN_ERR_LAUNCH",
}


class QnnError(RuntimeError):
    def __init__(self, status, where):
        self.status = status
        msg = lib().qnn_status_string(status).decode()
        super().__init__("%s: %s (%s)" % (where, STATUS.get(status, status), msg))


class Tensor(ctypes.Structure):
    _fields_ = [("n", ctypes.c_int32), ("h", ctypes.c_int32), ("w", ctypes.c_int32),
                ("c", ctypes.c_int32), ("bits", ctypes.c_int32)]


class ConvGeom(ctypes.Structure):
    _fields_ = [("kh", ctypes.c_int32), ("kw", ctypes.c_int32), ("stride_h", ctypes.c_int32),
                ("stride_w", ctypes.c_int32), ("pad_h", ctypes.c_int32), ("pad_w", ctypes.c_int32)]


class Tile(ctypes.Structure):
    _fields_ = [("kernel", ctypes.c_int32), ("tile_m", ctypes.c_int32), ("tile_n", ctypes.c_int32),
                ("waves", ctypes.c_int32)]


class Epi(ctypes.Structure):
    _fields_ = [("kind", ctypes.c_int32), ("bias", ctypes.c_void_p), ("mult", ctypes.c_void_p),
                ("shift", ctypes.c_void_p), ("thresh", ctypes.c_void_p),
                ("clip_lo", ctypes.c_int32), ("clip_hi", ctypes.c_int32)]


_lib = None

# The layer entry points once more, with plain pointer arguments: descriptors
# go in as packed bytes.  A call through ctypes structures takes longer on the
# host than most layers run on the device (building them, asking the library
# for the output shape, a stream object: 13 us a call, launch included).
_raw = {}


def lib():
    """Load libqnn.so (raises if it has not been built)."""
    global _lib
    if _lib is None:
        if not os.path.exists(LIB_PATH):
            raise RuntimeError("libqnn.so is not built (run __graft_entry__.build()); "
                               "there is no CPU fallback")
        L = ctypes.CDLL(LIB_PATH)
        P = ctypes.c_void_p
        TP = ctypes.POINTER(Tensor)
        L.qnn_abi_version.restype = ctypes.c_int32
        L.qnn_abi_version.argtypes = []
        L.qnn_status_string.restype = ctypes.c_char_p
        L.qnn_status_string.argtypes = [ctypes.c_int]
        L.qnn_device_check.restype = ctypes.c_int
        L.qnn_device_check.argtypes = []
        L.qnn_pixel_bytes.restype = ctypes.c_size_t
        L.qnn_pixel_bytes.argtypes = [TP]
        L.qnn_tensor_bytes.restype = ctypes.c_size_t
        L.qnn_tensor_bytes.argtypes = [TP]
        L.qnn_conv2d_out_shape.restype = ctypes.c_int
        L.qnn_conv2d_out_shape.argtypes = [TP, ctypes.c_int32, ctypes.POINTER(ConvGeom),
                                           ctypes.c_int32, TP]
        L.qnn_conv2d.restype = ctypes.c_int
        L.qnn_conv2d.argtypes = [TP, P, ctypes.c_int32, P, ctypes.POINTER(ConvGeom),
                                 ctypes.POINTER(Epi), TP, P, P]
        L.qnn_conv2d_tiled.restype = ctypes.c_int
        L.qnn_conv2d_tiled.argtypes = [TP, P, ctypes.c_int32, P, ctypes.POINTER(ConvGeom),
                                       ctypes.POINTER(Epi), ctypes.POINTER(Tile), TP, P, P]
        L.qnn_conv2d_maxpool.restype = ctypes.c_int
        L.qnn_conv2d_maxpool.argtypes = [TP, P, ctypes.c_int32, P, ctypes.POINTER(ConvGeom),
                                         ctypes.POINTER(Epi), ctypes.c_int32, ctypes.c_int32, TP, P, P]
        L.qnn_linear.restype = ctypes.c_int
        L.qnn_linear.argtypes = [TP, P, ctypes.c_int32, P, ctypes.POINTER(Epi), TP, P, P]
        L.qnn_maxpool2d.restype = ctypes.c_int
        L.qnn_maxpool2d.argtypes = [TP, P, ctypes.c_int32, ctypes.c_int32, ctypes.c_int32,
                                    ctypes.c_int32, TP, P, P]
        L.qnn_relu_s8.restype = ctypes.c_int
        L.qnn_relu_s8.argtypes = [P, P, ctypes.c_size_t, P]
        L.qnn_pack_host.restype = ctypes.c_int
        L.qnn_pack_host.argtypes = [P, ctypes.c_size_t, ctypes.c_int32, P]
        L.qnn_unpack_host.restype = ctypes.c_int
        L.qnn_unpack_host.argtypes = [P, ctypes.c_size_t, ctypes.c_int32, ctypes.c_int32, P]
        I = ctypes.c_int32
        for name, args in (("qnn_conv2d", [P, P, I, P, P, P, P, P, P]),
                           ("qnn_conv2d_tiled", [P, P, I, P, P, P, P, P, P, P]),
                           ("qnn_conv2d_maxpool", [P, P, I, P, P, P, I, I, P, P, P]),
                           ("qnn_linear", [P, P, I, P, P, P, P, P]),
                           ("qnn_maxpool2d", [P, P, I, I, I, I, P, P, P])):
            f = L[name]  # a function object of its own
            f.restype = ctypes.c_int
            f.argtypes = args
            _raw[name] = f
        _lib = L
    return _lib


def header_functions():
    """Names of the functions include/qnn.h declares."""
    with open(HEADER) as f:
        text = f.read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(qnn_[a-z0-9_]+)\s*\(", text)))


def _check(status, where):
    if status != 0:
        raise QnnError(status, where)


def _ptr(t):
    return None if t is None else ctypes.c_void_p(t.data_ptr())


def _call(name, *args):
    f = _raw.get(name)
    if f is None:
        lib()
        f = _raw[name]
    status = f(*args)
    if status != 0:
        raise QnnError(status, name)


_current = None  # () -> torch's current stream on the current device, as an integer


def _stream_int(stream):
    global _current
    if stream is not None:
        return stream.cuda_stream
    if _current is None:
        import torch
        raw = getattr(torch._C, "_cuda_getCurrentRawStream", None)
        if raw is None:
            _current = lambda: torch.cuda.current_stream().cuda_stream
        else:
            device = torch.cuda.current_device
            _current = lambda: raw(device())
    return _current()


_pack5 = struct.Struct("@5i").pack
_pack6 = struct.Struct("@6i").pack
_pack_epi = struct.Struct("@i4x4P2i").pack


def _tensor_bytes(*v):
    try:
        return _pack5(*v)
    except struct.error:  # a value past 32 bits: as the structure takes it
        return bytes(Tensor(*v))


def _epi_bytes(kind, bias, mult, shift, thresh, clip):
    try:
        return _pack_epi(kind, bias.data_ptr() if bias is not None else 0,
                         mult.data_ptr() if mult is not None else 0,
                         shift.data_ptr() if shift is not None else 0,
                         thresh.data_ptr() if thresh is not None else 0, clip[0], clip[1])
    except struct.error:
        return bytes(_epi(kind, bias, mult, shift, thresh, clip)[0])


def _epi(kind, bias, mult, shift, thresh, clip):
    if isinstance(kind, str):
        kind = _EPI_NAMES[kind]
    return Epi(kind, _ptr(bias).value if bias is not None else None,
               _ptr(mult).value if mult is not None else None,
               _ptr(shift).value if shift is not None else None,
               _ptr(thresh).value if thresh is not None else None, clip[0], clip[1]), kind


def pixel_bytes(c, bits):
    return 4 * c if bits == 32 else (c * bits + 7) // 8


def out_shape(xshape, bits, m, kh, kw, stride=(1, 1), pad=(0, 0), epi="requant"):
    """(n, ho, wo, m, out_bits) of a convolution, computed by the library."""
    kind = _EPI_NAMES[epi] if isinstance(epi, str) else epi
    x = Tensor(*xshape, bits)
    y = Tensor()
    _check(lib().qnn_conv2d_out_shape(ctypes.byref(x), m, ctypes.byref(ConvGeom(kh, kw, *stride, *pad)),
                                      kind, ctypes.byref(y)), "qnn_conv2d_out_shape")
    return (y.n, y.h, y.w, y.c, y.bits)


# output bits of each epilogue and bit-width that go together
_OUT_BITS = {(kind, bits): {EPI_REQUANT: bits, EPI_STAIR: bits, EPI_THRESH1: 1, EPI_RAW32: 32}[kind]
             for kind, widths in ((EPI_REQUANT, (8, 4, 2)), (EPI_STAIR, (4, 2)), (EPI_THRESH1, (1,)),
                                  (EPI_RAW32, (8, 4, 2, 1))) for bits in widths}


def _conv_layer(xshape, bits, m, kh, kw, stride, pad, kind):
    """(output shape, x's descriptor, geometry's descriptor) of a convolution.
    The shape is worked out here for every layer that the library accepts; the
    others, and arguments that are no plain integers or not as many as they
    should be, take the structures and the library's shape query, which accept
    or refuse them."""
    try:
        n, h, w, c = xshape
        sh, sw = stride
        ph, pw = pad
        xd = _pack5(n, h, w, c, bits)
        g = _pack6(kh, kw, sh, sw, ph, pw)
        obits = _OUT_BITS.get((kind, bits))
        if obits and kh > 0 and kw > 0 and sh > 0 and sw > 0 and ph >= 0 and pw >= 0:
            ho = (h + 2 * ph - kh) // sh + 1
            wo = (w + 2 * pw - kw) // sw + 1
            size = n * h * w * c
            out = n * ho * wo * m
            # (sizes near the library's limits are the library's to judge; a
            # number of another type would make either product one too)
            if (ho > 0 and wo > 0 and h > 0 and w > 0 and c > 0 and 0 < m < 1 << 31 and 0 <= size < 1 << 40 and
                    0 <= out < 1 << 40 and type(n) is int and type(size) is int and type(out) is int and
                    type(kind) is int):
                return (n, ho, wo, m, obits), xd, g
    except (struct.error, TypeError, ValueError, OverflowError):
        pass
    yshape = out_shape(xshape, bits, m, kh, kw, stride, pad, kind)
    return yshape, bytes(Tensor(*xshape, bits)), bytes(ConvGeom(kh, kw, stride[0], stride[1], pad[0], pad[1]))


def _new_out(shape, out, x):
    """_out_tensor, without its detour where x is what it usually is."""
    if out is None:
        n, h, w, c, bits = shape
        if bits != 32 and x.dtype is _uint8():
            return x.new_empty((n, h, w, (c * bits + 7) // 8))
    return _out_tensor(shape, out, x.device)


_u8 = None


def _uint8():
    global _u8
    if _u8 is None:
        import torch
        _u8 = torch.uint8
    return _u8


def _out_tensor(shape, out, device):
    import torch
    n, h, w, c, bits = shape
    if bits == 32:
        want = (n, h, w, c)
        dtype = torch.int32
    else:
        want = (n, h, w, pixel_bytes(c, bits))
        dtype = torch.uint8
    if out is None:
        return torch.empty(want, dtype=dtype, device=device)
    if tuple(out.shape) != want or out.dtype != dtype or not out.is_contiguous():
        raise ValueError("out must be a contiguous %s tensor of shape %s" % (dtype, want))
    return out


def conv2d(x, xshape, bits, w, m, kh, kw, stride=(1, 1), pad=(0, 0), epi="requant", bias=None,
           mult=None, shift=None, thresh=None, clip=(0, 0), out=None, stream=None, tile=None):
    """Quantized convolution (qnn_conv2d).  x: uint8 packed NHWC device tensor
    of logical shape xshape = (n, h, w, c); w: uint8 packed weights.  Returns
    uint8 [N, Ho, Wo, out bytes] codes or int32 [N, Ho, Wo, M] (raw32).
    tile = (kernel, tile_m, tile_n, waves) picks the tile shape
    (qnn_conv2d_tiled) instead of the library."""
    kind = _EPI_NAMES[epi] if isinstance(epi, str) else epi
    yshape, xd, g = _conv_layer(xshape, bits, m, kh, kw, stride, pad, kind)
    y = _new_out(yshape, out, x)
    yd = _tensor_bytes(*yshape)
    e = _epi_bytes(kind, bias, mult, shift, thresh, clip)
    wp = None if w is None else w.data_ptr()  # (None: NULL, the library's to accept or refuse)
    if tile is None:
        _call("qnn_conv2d", xd, x.data_ptr(), m, wp, g, e, yd, y.data_ptr(), _stream_int(stream))
    else:
        _call("qnn_conv2d_tiled", xd, x.data_ptr(), m, wp, g, e, bytes(Tile(*tile)), yd, y.data_ptr(),
              _stream_int(stream))
    return y


def conv2d_maxpool(x, xshape, bits, w, m, kh, kw, stride=(1, 1), pad=(0, 0), epi="requant",
                   bias=None, mult=None, shift=None, thresh=None, clip=(0, 0), out=None, stream=None):
    """Convolution fused with 2x2 / stride-2 max-pooling (qnn_conv2d_maxpool).
    Returns uint8 [N, floor(Ho/2), floor(Wo/2), out bytes] codes."""
    kind = _EPI_NAMES[epi] if isinstance(epi, str) else epi
    (n, ho, wo, c, obits), xd, g = _conv_layer(xshape, bits, m, kh, kw, stride, pad, kind)
    yshape = (n, ho // 2, wo // 2, c, obits)
    y = _new_out(yshape, out, x)
    wp = None if w is None else w.data_ptr()
    _call("qnn_conv2d_maxpool", xd, x.data_ptr(), m, wp, g,
          _epi_bytes(kind, bias, mult, shift, thresh, clip), 2, 2, _tensor_bytes(*yshape), y.data_ptr(),
          _stream_int(stream))
    return y


def linear(x, xshape, bits, w, m, epi="raw32", bias=None, mult=None, shift=None, thresh=None,
           clip=(0, 0), out=None, stream=None):
    """Fully connected layer (qnn_linear) over the whole NHWC image."""
    kind = _EPI_NAMES[epi] if isinstance(epi, str) else epi
    obits = {EPI_REQUANT: bits, EPI_THRESH1: 1, EPI_RAW32: 32}[kind]
    yshape = (xshape[0], 1, 1, m, obits)
    y = _new_out(yshape, out, x)
    wp = None if w is None else w.data_ptr()
    _call("qnn_linear", _tensor_bytes(*xshape, bits), x.data_ptr(), m, wp,
          _epi_bytes(kind, bias, mult, shift, thresh, clip), _tensor_bytes(*yshape), y.data_ptr(),
          _stream_int(stream))
    return y


def maxpool2d(x, xshape, bits, kh, kw, sh, sw, out=None, stream=None):
    """Max-pooling over packed unsigned codes (qnn_maxpool2d)."""
    n, h, w_, c = xshape
    ho = (h - kh) // sh + 1
    wo = (w_ - kw) // sw + 1
    yshape = (n, ho, wo, c, bits)
    y = _new_out(yshape, out, x)
    _call("qnn_maxpool2d", _tensor_bytes(*xshape, bits), x.data_ptr(), kh, kw, sh, sw, _tensor_bytes(*yshape),
          y.data_ptr(), _stream_int(stream))
    return y


def relu_s8(x, out=None, stream=None):
    """Signed 8-bit ReLU (qnn_relu_s8); out may be x (in place)."""
    import torch
    y = torch.empty_like(x) if out is None else out
    _check(lib().qnn_relu_s8(x.data_ptr(), y.data_ptr(), x.numel(), _stream_int(stream)), "qnn_relu_s8")
    return y


def device_check():
    _check(lib().qnn_device_check(), "qnn_device_check")


def pack_host(codes, bits):
    """Host packing of unsigned codes (numpy uint8 array) -> packed bytes."""
    import numpy as np
    codes = np.ascontiguousarray(codes, dtype=np.uint8).reshape(-1)
    out = np.zeros((codes.size * bits + 7) // 8, dtype=np.uint8)
    _check(lib().qnn_pack_host(codes.ctypes.data_as(ctypes.c_void_p), codes.size, bits,
                               out.ctypes.data_as(ctypes.c_void_p)), "qnn_pack_host")
    return out


def unpack_host(packed, count, bits, signed):
    import numpy as np
    packed = np.ascontiguousarray(packed, dtype=np.uint8)
    out = np.zeros(count, dtype=np.int32)
    _check(lib().qnn_unpack_host(packed.ctypes.data_as(ctypes.c_void_p), count, bits,
                                 1 if signed else 0, out.ctypes.data_as(ctypes.c_void_p)),
           "qnn_unpack_host")
    return out
