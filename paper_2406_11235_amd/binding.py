"""Binding of libqtip.so: same names as include/qtip.h, argument marshalling only (ctypes for what runs on
the host, the _call extension for what enqueues GPU work).

GPU entry points take torch tensors that already live on the device (or raw
integer device pointers) and enqueue on torch's current stream unless a stream is
given.  There is no fallback: if the library is missing, loading raises.
"""
import ctypes
import functools
import os

import numpy as np

CODE_1MAD, CODE_3INST, CODE_HYB, CODE_HYB2, CODE_LUT, CODE_HYB1 = 0, 1, 2, 3, 4, 5

_HERE = os.path.dirname(os.path.abspath(__file__))
# The environment variable QTIP_LIBRARY names another build of the same library to load instead
# (two builds compared on one box; the sanitizer build of the host code in tests/test_sanitizers.py).
_LIB_PATH = os.environ.get("QTIP_LIBRARY") or os.path.join(_HERE, "libqtip.so")
_lib = None

EXPORTS = ["qtip_rht", "qtip_rht_f32", "qtip_decode_matvec", "qtip_rht_decode_matvec",
           "qtip_rht_decode_matvec_noalloc", "qtip_decode_matmat",
           "qtip_dequantize", "qtip_decode_states", "qtip_quantize",
           "qtip_quantize_gpu_workspace", "qtip_quantize_gpu", "qtip_block_ldl_workspace",
           "qtip_block_ldl", "qtip_quantize_ldlq_workspace", "qtip_quantize_ldlq", "qtip_last_error",
           "qtip_version"]


class QtipError(RuntimeError):
    def __init__(self, code, message):
        super().__init__(f"qtip error {code}: {message}")
        self.code = code


def library_path():
    return _LIB_PATH


def lib():
    """Load libqtip.so (built by paper_2406_11235_amd.build.build())."""
    global _lib
    if _lib is None:
        if not os.path.exists(_LIB_PATH):
            raise FileNotFoundError(
                f"{_LIB_PATH} is missing: run `python -m paper_2406_11235_amd.build` "
                "(there is no CPU fallback)")
        # torch ships its own HIP runtime; it must be the one libqtip.so binds to, or
        # the process ends up with two runtimes and the second one sees no device.
        import torch  # noqa: F401
        L = ctypes.CDLL(_LIB_PATH)
        c = ctypes
        vp, i32 = c.c_void_p, c.c_int
        L.qtip_version.restype = i32
        L.qtip_version.argtypes = []
        L.qtip_last_error.restype = c.c_char_p
        L.qtip_last_error.argtypes = []
        L.qtip_rht.restype = i32
        L.qtip_rht.argtypes = [vp, vp, i32, i32, i32, i32, vp, vp]
        L.qtip_rht_f32.restype = i32
        L.qtip_rht_f32.argtypes = [vp, vp, i32, i32, i32, i32, vp, vp]
        L.qtip_decode_matvec.restype = i32
        L.qtip_decode_matvec.argtypes = [vp, i32, i32, i32, i32, vp, i32, i32, vp, vp, vp]
        L.qtip_rht_decode_matvec.restype = i32
        L.qtip_rht_decode_matvec.argtypes = [vp, i32, i32, i32, i32, vp, i32, i32, vp, vp, i32, vp, vp, vp, vp]
        L.qtip_rht_decode_matvec_noalloc.restype = i32
        L.qtip_rht_decode_matvec_noalloc.argtypes = [vp, i32, i32, i32, i32, vp, i32, i32, vp, vp, i32, vp, vp, vp]
        L.qtip_decode_matmat.restype = i32
        L.qtip_decode_matmat.argtypes = [vp, i32, i32, i32, i32, vp, i32, i32, vp, i32, vp, vp, vp]
        L.qtip_dequantize.restype = i32
        L.qtip_dequantize.argtypes = [vp, i32, i32, i32, i32, vp, i32, i32, vp, vp]
        L.qtip_decode_states.restype = i32
        L.qtip_decode_states.argtypes = [vp, i32, i32, i32, i32, vp, vp, vp]
        L.qtip_quantize.restype = i32
        L.qtip_quantize.argtypes = [vp, i32, i32, i32, i32, i32, i32, vp, vp, vp]
        L.qtip_quantize_gpu_workspace.restype = c.c_size_t
        L.qtip_quantize_gpu_workspace.argtypes = [i32, i32, c.c_long]
        L.qtip_quantize_gpu.restype = i32
        L.qtip_quantize_gpu.argtypes = [vp, i32, i32, i32, i32, i32, i32, vp, vp, vp, vp,
                                        c.c_size_t, vp]
        L.qtip_block_ldl_workspace.restype = c.c_size_t
        L.qtip_block_ldl_workspace.argtypes = [i32]
        L.qtip_block_ldl.restype = i32
        L.qtip_block_ldl.argtypes = [vp, i32, i32, vp, vp, vp, c.c_size_t, vp]
        L.qtip_quantize_ldlq_workspace.restype = c.c_size_t
        L.qtip_quantize_ldlq_workspace.argtypes = [i32, i32, i32, i32, c.c_long]
        L.qtip_quantize_ldlq.restype = i32
        L.qtip_quantize_ldlq.argtypes = [vp, vp, i32, i32, i32, i32, i32, i32, vp, vp, vp, vp, vp,
                                         c.c_size_t, vp]
        _lib = L
    return _lib


def _ptr(t):
    """Device (or host) address of a torch tensor / numpy array / int / None."""
    if t is None:
        return None
    if isinstance(t, int):
        return t
    if isinstance(t, np.ndarray):
        return t.ctypes.data
    return t.data_ptr()


def _stream(stream):
    if stream is None:
        import torch
        current = torch.cuda.current_stream().cuda_stream  # (initializes torch's GPU state where nothing has yet)
        # from here on _call asks torch's own getters of the current device and of its current stream as an integer,
        # where this torch has them
        device, raw = (getattr(torch._C, name, None) for name in ("_cuda_getDevice", "_cuda_getCurrentRawStream"))
        if _call is not None and device is not None and raw is not None:
            _call.hooks(_ptr, _stream, _check, _connect, device, raw)
        return current
    if isinstance(stream, int):
        return stream
    return stream.cuda_stream


def _check(rc):
    if rc != 0:
        raise QtipError(rc, lib().qtip_last_error().decode())
    return rc


# The entry points that enqueue work are callable objects of the _call extension (csrc/qtip_call.cpp),
# which turns their arguments into the C ones itself.
_GPU_ENTRIES = ["qtip_rht", "qtip_rht_f32", "qtip_decode_matvec", "qtip_rht_decode_matvec",
                "qtip_rht_decode_matvec_noalloc", "qtip_decode_matmat", "qtip_dequantize", "qtip_decode_states",
                "qtip_quantize_gpu", "qtip_block_ldl", "qtip_quantize_ldlq"]
_call = None


def _connect():
    """Give the entry points of _call the addresses of the loaded library's functions."""
    L = lib()
    for name in _GPU_ENTRIES:
        _call.connect(getattr(_call, name), ctypes.cast(getattr(L, name), ctypes.c_void_p).value)


def _ask_torch():
    """Have _call come to _stream() for the current stream."""
    _call.hooks(_ptr, _stream, _check, _connect, None, None)


def _load_call():
    global _call
    if _call is None:
        import importlib
        try:
            _call = importlib.import_module("._call", __package__)
        except ImportError as e:
            raise FileNotFoundError(
                f"the _call extension of {__package__} is missing ({e}): run `python -m paper_2406_11235_amd.build`"
            ) from e
        _ask_torch()
        # (torch refuses GPU work in a forked child of a process that has done some; its getters alone would not)
        os.register_at_fork(after_in_child=_ask_torch)
    return _call


def _entry(signature):
    """The callable for one entry point, which looks like the function it is written as below; a stand-in that looks for
    it when called where nothing is built yet or what is there is from before (it has to be importable to be built)."""
    try:
        return functools.update_wrapper(getattr(_load_call(), signature.__name__), signature)
    except (FileNotFoundError, AttributeError):
        def entry(*args, **kwargs):
            return getattr(_load_call(), signature.__name__)(*args, **kwargs)
        return functools.update_wrapper(entry, signature)


@_entry
def qtip_rht(x, signs, n, block, batch, side, out, stream=None):
    """Random Hadamard transform of fp16 activations: side 0 is V (S .* x), side 1 is S .* (V^T x)."""


@_entry
def qtip_rht_f32(x, signs, n, block, batch, side, out, stream=None):
    """qtip_rht of fp32 values; the result is fp16."""


@_entry
def qtip_decode_matvec(codes, L, k, V, code_id, lut, m, n, x, y, stream=None):
    """y = W~ x, the weights decoded on the way."""


@_entry
def qtip_rht_decode_matvec(codes, L, k, V, code_id, lut, m, n, x, signs_n, block, row_scale, y, xt_scratch=None,
                           stream=None):
    """y = row_scale .* (W~ (V (S_n .* x))): the input side of a layer."""


@_entry
def qtip_rht_decode_matvec_noalloc(codes, L, k, V, code_id, lut, m, n, x, signs_n, block, row_scale, y, stream=None):
    """qtip_rht_decode_matvec with the library's own scratch (n at most 65536)."""


@_entry
def qtip_decode_matmat(codes, L, k, V, code_id, lut, m, n, X, B, row_scale, Y, stream=None):
    """Y[b] = row_scale .* (W~ X[b]) for B rows."""


@_entry
def qtip_dequantize(codes, L, k, V, code_id, lut, m, n, W, stream=None):
    """The weights of a code stream as an m x n fp16 matrix."""


@_entry
def qtip_decode_states(states, count, L, V, code_id, lut, out, stream=None):
    """The values of a list of states."""


@_entry
def qtip_quantize_gpu(W, m, n, L, k, V, code_id, lut, codes_out, tile_err, workspace, workspace_bytes, stream=None):
    """A weight matrix to code streams, block by block."""


@_entry
def qtip_block_ldl(H, n, g, A_out, D_out, workspace, workspace_bytes, stream=None):
    """The block LDL decomposition of a proxy Hessian."""


@_entry
def qtip_quantize_ldlq(W, A, m, n, L, k, V, code_id, lut, codes_out, What_out, tile_err, workspace, workspace_bytes,
                       stream=None):
    """A weight matrix to code streams with feedback (BlockLDLQ)."""


def qtip_version():
    return int(lib().qtip_version())


def qtip_last_error():
    return lib().qtip_last_error().decode()


def qtip_quantize(W, m, n, L, k, V, code_id, lut=None):
    """Host quantizer: W float32 (m, n) numpy -> (codes uint32 (tiles, 8k), mse)."""
    W = np.ascontiguousarray(W, dtype=np.float32)
    assert W.shape == (m, n)
    if lut is not None:
        lut = np.ascontiguousarray(lut)
        assert lut.dtype in (np.float16, np.uint16) and lut.size == {CODE_LUT: 1 << 14, CODE_HYB1: 64}.get(code_id, 1024)
    codes = np.zeros((m * n // 256, 8 * k), dtype=np.uint32)  # one sequence per 256 weights
    mse = ctypes.c_double(0.0)
    _check(lib().qtip_quantize(_ptr(W), m, n, L, k, V, code_id, _ptr(lut), _ptr(codes),
                               ctypes.addressof(mse)))
    return codes, float(mse.value)


def qtip_quantize_gpu_workspace(k, V, tiles):
    return int(lib().qtip_quantize_gpu_workspace(k, V, tiles))


def qtip_block_ldl_workspace(n):
    return int(lib().qtip_block_ldl_workspace(n))


def qtip_quantize_ldlq_workspace(m, n, k, V, tiles):
    return int(lib().qtip_quantize_ldlq_workspace(m, n, k, V, tiles))


