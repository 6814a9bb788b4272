"""HEAL compensated GEMM for MI355X: Python binding of ``libheal.so``.

Argument marshalling only: every step of the computation runs in the HIP
kernels behind the C ABI declared in ``include/heal.h``.  PyTorch supplies
device memory and the current stream; nothing here computes on the host.
If the library is not built (``python -m paper_2606_21023_amd.build``), every
call raises ``HealError``: there is no fallback path.

Functions (names follow the C ABI):
  heal_split_f32(x)                   -> (hi, lo) bf16 bit patterns, torch.uint16
  heal_gemm_f32(A, B, out=None)       -> C = A @ B, bf16x3 compensated, FP32
  heal_gemm_f32_strided_batched(A, B, alpha=1.0, trans_b=False, out=None)
  heal_gemm_f32_instance(instance, A, B, ...)  -- a forced kernel instance
  heal_split_f16(x)                   -> (hi, lo) binary16 bit patterns (HEAL-Full pair)
  heal_maxabs_f32(x)                  -> max|x| as a 1-element float32 CUDA tensor
  heal_f16_weight_exponent(maxabs)    -> int e (host)
  heal_pack_f16_weight(W, e)          -> packed FP16 weight (torch.uint16)
  heal_gemm_f16w(A, W16, N, e, products)  -> HEAL-Base (1) / HEAL-Full (2) GEMM, FP32
  heal_presplit_b(B, trans_b=False)   -> packed bf16 (hi, lo) operand
  heal_gemm_f32_presplit(A, Bp, N)    -> bitwise equal to heal_gemm_f32(A, B)
  heal_quantize_i16(x)                -> (codes int16, max|x| 1-element tensor)
  heal_scores_i16(Q, Kt, maxQ, maxK, alpha)  -> dual-FP16 scores of INT16 codes, FP32
  lib()                               -> the raw ctypes library
  build_id(), check_build()           -> the library's source hash; refuse a stale binary
"""
import ctypes
import os

__all__ = ["HealError", "lib", "library_path", "build_id", "check_build", "heal_split_f32", "heal_gemm_f32",
           "heal_gemm_f32_strided_batched", "heal_gemm_f32_instance", "select_instance",
           "INSTANCE_AUTO", "INSTANCE_LARGE", "INSTANCE_MEDIUM", "INSTANCE_SKINNY", "STATUS",
           "heal_split_f16", "heal_packed_size", "heal_maxabs_f32", "heal_f16_weight_exponent",
           "heal_pack_f16_weight", "heal_gemm_f16w", "heal_presplit_b", "heal_gemm_f32_presplit",
           "heal_quantize_i16", "heal_scores_i16"]

_HERE = os.path.dirname(os.path.abspath(__file__))
library_path = os.path.join(_HERE, "libheal.so")

INSTANCE_AUTO, INSTANCE_LARGE, INSTANCE_MEDIUM, INSTANCE_SKINNY = 0, 1, 2, 3
STATUS = {0: "HEAL_OK", 1: "HEAL_ERR_INVALID_VALUE", 2: "HEAL_ERR_UNSUPPORTED_DEVICE",
          3: "HEAL_ERR_LAUNCH"}


class HealError(RuntimeError):
    """A libheal call failed, or the library is missing."""

    def __init__(self, msg, status=None):
        super().__init__(msg)
        self.status = status


_lib = None
_i64 = ctypes.c_int64
_vp = ctypes.c_void_p


def lib():
    """Load ``libheal.so`` (once) and declare its C signatures."""
    global _lib
    if _lib is not None:
        return _lib
    if not os.path.exists(library_path):
        raise HealError("libheal.so is not built (expected at %s); run "
                        "`python -m paper_2606_21023_amd.build`" % library_path)
    L = ctypes.CDLL(library_path)
    L.heal_status_string.argtypes = [ctypes.c_int]
    L.heal_status_string.restype = ctypes.c_char_p
    L.heal_version.argtypes = []
    L.heal_version.restype = ctypes.c_int
    L.heal_build_id.argtypes = []
    L.heal_build_id.restype = ctypes.c_char_p
    L.heal_split_f32.argtypes = [_vp, _vp, _vp, _i64, _vp]
    L.heal_split_f32.restype = ctypes.c_int
    L.heal_gemm_f32.argtypes = [_i64, _i64, _i64, _vp, _vp, _vp, _i64, _i64, _i64, _vp]
    L.heal_gemm_f32.restype = ctypes.c_int
    L.heal_gemm_f32_strided_batched.argtypes = [_i64, _i64, _i64, ctypes.c_float,
                                                _vp, _i64, _i64, _vp, _i64, _i64, ctypes.c_int,
                                                _vp, _i64, _i64, _i64, _vp]
    L.heal_gemm_f32_strided_batched.restype = ctypes.c_int
    L.heal_gemm_f32_instance.argtypes = [ctypes.c_int] + L.heal_gemm_f32_strided_batched.argtypes
    L.heal_gemm_f32_instance.restype = ctypes.c_int
    L.heal_gemm_select_instance.argtypes = [_i64, _i64]
    L.heal_gemm_select_instance.restype = ctypes.c_int
    _c = ctypes.c_int
    L.heal_gemm_direct_tile.argtypes = [_c, _c, _i64, _i64, _i64, _i64]
    L.heal_gemm_direct_tile.restype = _c
    L.heal_split_f16.argtypes = [_vp, _vp, _vp, _i64, _vp]
    L.heal_split_f16.restype = _c
    L.heal_packed_size.argtypes = [_i64, _i64, _c]
    L.heal_packed_size.restype = _i64
    L.heal_maxabs_f32.argtypes = [_vp, _i64, _i64, _i64, _vp, _vp]
    L.heal_maxabs_f32.restype = _c
    L.heal_f16_weight_exponent.argtypes = [ctypes.c_float, ctypes.POINTER(ctypes.c_int32)]
    L.heal_f16_weight_exponent.restype = _c
    L.heal_pack_f16_weight.argtypes = [_vp, _i64, _i64, _i64, ctypes.c_int32, _vp, _vp]
    L.heal_pack_f16_weight.restype = _c
    L.heal_gemm_f16w.argtypes = [_c, _i64, _i64, _i64, _vp, _i64, _vp, ctypes.c_int32, _vp, _i64,
                                 _vp]
    L.heal_gemm_f16w.restype = _c
    L.heal_gemm_f16w_instance.argtypes = [_c] + L.heal_gemm_f16w.argtypes
    L.heal_gemm_f16w_instance.restype = _c
    L.heal_presplit_b.argtypes = [_vp, _i64, _i64, _i64, _c, _vp, _vp]
    L.heal_presplit_b.restype = _c
    L.heal_gemm_f32_presplit.argtypes = [_i64, _i64, _i64, _vp, _i64, _vp, _vp, _i64, _vp]
    L.heal_gemm_f32_presplit.restype = _c
    L.heal_gemm_f32_presplit_instance.argtypes = [_c] + L.heal_gemm_f32_presplit.argtypes
    L.heal_gemm_f32_presplit_instance.restype = _c
    L.heal_quantize_i16.argtypes = [_vp, _i64, _vp, _vp, _vp]
    L.heal_quantize_i16.restype = _c
    L.heal_scores_i16.argtypes = [_i64, _i64, _i64, _vp, _i64, _i64, _vp, _vp, _i64, _i64, _vp,
                                  ctypes.c_float, _vp, _i64, _i64, _i64, _vp]
    L.heal_scores_i16.restype = _c
    _lib = L
    return L


def build_id():
    """The source hash the loaded ``libheal.so`` was built from."""
    return lib().heal_build_id().decode()


def check_build():
    """Raise ``HealError`` unless the loaded ``libheal.so`` was built from the
    sources beside it (a stale binary would test old code)."""
    from . import build as _build
    want, got = _build.source_hash(), build_id()
    if got != want:
        raise HealError("libheal.so was built from other sources (build id %s, sources %s); "
                        "rebuild with `python -m paper_2606_21023_amd.build`" % (got, want))
    return got


def _check(status, what):
    if status != 0:
        raise HealError("%s failed: %s" % (what, STATUS.get(status, status)), status)


class _Torch:
    """Stands for the module until a call needs it: the C library is built, and
    its host functions are called, without PyTorch."""

    def __getattr__(self, name):
        import importlib
        globals()["torch"] = module = importlib.import_module("torch")
        return getattr(module, name)


torch = _Torch()


def _stream():
    """The current device's current stream, as a raw pointer.  (The Stream object
    of torch.cuda.current_stream costs 3 us, a third of a small call; it stands in
    where torch lacks the raw accessors.)  The first call replaces itself."""
    global _stream
    raw = getattr(torch._C, "_cuda_getCurrentRawStream", None)
    device = getattr(torch._C, "_cuda_getDevice", None)
    if raw is None or device is None:
        _stream = lambda: torch.cuda.current_stream().cuda_stream
    else:
        _stream = lambda: raw(device())
    return _stream()


def _tensor(t, name, dtype, ndim=None):
    """Check a CUDA tensor of a type and number of dimensions whose last one is
    contiguous; returns its shape and strides."""
    if not isinstance(t, torch.Tensor) or not t.is_cuda:
        raise HealError("%s must be a CUDA (HIP) tensor" % name)
    if t.dtype is not dtype:
        raise HealError("%s must be %s, got %s" % (name, str(dtype).replace("torch.", ""), t.dtype))
    shape, stride = t.shape, t.stride()
    if ndim is not None and len(shape) != ndim:
        raise HealError("%s must have %d dimensions, got %d" % (name, ndim, len(shape)))
    if stride[-1] != 1 and shape[-1] > 1 and t.numel():   # (0 dimensions: IndexError)
        # (a last dimension of one element has no stride to respect: torch
        # may report any, e.g. for the transpose of a one-row matrix)
        raise HealError("%s must be contiguous in its last dimension" % name)
    return shape, stride


def _ld(shape, stride):
    """Row stride of the last two dims, in elements."""
    return stride[-2] if shape[-2] > 1 else max(shape[-1], 1)


def _output(out, like, shape):
    """`out`, checked, or a new float32 tensor; and its strides."""
    if out is None:
        # (new_empty is 0.6 us faster, but follows a subclass)
        C = (like.new_empty(shape) if type(like) is torch.Tensor
             else torch.empty(shape, dtype=torch.float32, device=like.device))
        return C, C.stride()
    got, stride = _tensor(out, "out", torch.float32, len(shape))
    if tuple(got) != shape:
        raise HealError("out has shape %s, expected %s" % (tuple(got), shape))
    return out, stride


def heal_split_f32(x, hi=None, lo=None):
    """Split a contiguous float32 CUDA tensor into bf16 (hi, lo) bit patterns."""
    return _split("heal_split_f32", x, hi, lo)


def _split(what, x, hi, lo):
    if not isinstance(x, torch.Tensor) or not x.is_cuda or x.dtype != torch.float32:
        raise HealError("x must be a float32 CUDA tensor")
    if not x.is_contiguous():
        raise HealError("x must be contiguous")
    if hi is None:
        hi = torch.empty(x.shape, dtype=torch.uint16, device=x.device)
    if lo is None:
        lo = torch.empty(x.shape, dtype=torch.uint16, device=x.device)
    _check(getattr(lib(), what)(x.data_ptr(), hi.data_ptr(), lo.data_ptr(), x.numel(), _stream()),
           what)
    return hi, lo


def heal_gemm_f32(A, B, out=None):
    """C = A @ B (A: M x K, B: K x N, row-major float32 CUDA tensors)."""
    shape_a, stride_a = _tensor(A, "A", torch.float32, 2)
    shape_b, stride_b = _tensor(B, "B", torch.float32, 2)
    M, K = shape_a
    N = shape_b[1]
    if shape_b[0] != K:
        raise HealError("inner dimensions differ: %s @ %s" % (tuple(A.shape), tuple(B.shape)))
    C, stride_c = _output(out, A, (M, N))
    _check((_lib or lib()).heal_gemm_f32(
        M, N, K, A.data_ptr(), B.data_ptr(), C.data_ptr(), _ld(shape_a, stride_a),
        _ld(shape_b, stride_b), _ld((M, N), stride_c), _stream()), "heal_gemm_f32")
    return C


def _batched(fn_args_prefix, A, B, alpha, trans_b, out, what):
    shape_a, stride_a = _tensor(A, "A", torch.float32, 3)
    shape_b, stride_b = _tensor(B, "B", torch.float32, 3)
    bat, M, K = shape_a
    N, Kb = (shape_b[1], shape_b[2]) if trans_b else (shape_b[2], shape_b[1])
    if Kb != K or shape_b[0] != bat:
        raise HealError("shapes do not match: A %s, B %s, trans_b=%s"
                        % (tuple(A.shape), tuple(B.shape), trans_b))
    C, stride_c = _output(out, A, (bat, M, N))
    many = bat > 1
    st = fn_args_prefix(M, N, K, ctypes.c_float(alpha), A.data_ptr(), _ld(shape_a, stride_a),
                        stride_a[0] if many else 0, B.data_ptr(), _ld(shape_b, stride_b),
                        stride_b[0] if many else 0, 1 if trans_b else 0, C.data_ptr(),
                        _ld((M, N), stride_c), stride_c[0] if many else 0, bat, _stream())
    _check(st, what)
    return C


def heal_gemm_f32_strided_batched(A, B, alpha=1.0, trans_b=False, out=None):
    """C[b] = alpha * A[b] @ op(B[b]) for 3-D tensors; op(B) = B^T if trans_b."""
    return _batched((_lib or lib()).heal_gemm_f32_strided_batched, A, B, alpha, trans_b, out,
                    "heal_gemm_f32_strided_batched")


def heal_gemm_f32_instance(instance, A, B, alpha=1.0, trans_b=False, out=None):
    """As heal_gemm_f32_strided_batched with a forced kernel instance (2-D or 3-D)."""
    squeeze = A.dim() == 2
    if squeeze:
        A, B = A.unsqueeze(0), B.unsqueeze(0)
        out = out.unsqueeze(0) if out is not None else None
    f = lib().heal_gemm_f32_instance
    C = _batched(lambda *a: f(int(instance), *a), A, B, alpha, trans_b, out,
                 "heal_gemm_f32_instance")
    return C[0] if squeeze else C


def select_instance(M, N):
    """The instance heal_gemm_f32 chooses for an M x N output by its size."""
    return lib().heal_gemm_select_instance(M, N)


# ---- FP16 forms, pre-split operand, INT16 scores ---------------------------

def heal_split_f16(x, hi=None, lo=None):
    """HEAL-Full pair of a contiguous float32 CUDA tensor, binary16 bit patterns."""
    return _split("heal_split_f16", x, hi, lo)


def heal_packed_size(K, N, planes):
    n = (_lib or lib()).heal_packed_size(K, N, planes)
    if n < 0:
        raise HealError("invalid packed size K=%d N=%d planes=%d" % (K, N, planes))
    return n


def heal_maxabs_f32(x, out=None):
    """max|x| of a 2-D (or contiguous) float32 CUDA tensor, as a 1-element tensor."""
    shape, stride = _tensor(x, "x", torch.float32)
    if len(shape) == 2:
        rows, cols, ld = shape[0], shape[1], _ld(shape, stride)
    else:
        if not x.is_contiguous():
            raise HealError("x must be 2-D or contiguous")
        rows, cols, ld = 1, x.numel(), max(x.numel(), 1)
    out = out if out is not None else torch.empty(1, dtype=torch.float32, device=x.device)
    _check(lib().heal_maxabs_f32(x.data_ptr(), rows, cols, ld, out.data_ptr(), _stream()),
           "heal_maxabs_f32")
    return out


def heal_f16_weight_exponent(maxabs):
    """Largest e with maxabs * 2^e <= 65504 (host)."""
    e = ctypes.c_int32()
    _check(lib().heal_f16_weight_exponent(ctypes.c_float(float(maxabs)), ctypes.byref(e)),
           "heal_f16_weight_exponent")
    return e.value


def heal_pack_f16_weight(W, e, out=None):
    """Packed RNE_f16(W * 2^e) of an N x K float32 weight (torch.uint16, 1-D)."""
    shape, stride = _tensor(W, "W", torch.float32, 2)
    N, K = shape
    size = heal_packed_size(K, N, 1)
    out = out if out is not None else torch.empty(size, dtype=torch.uint16, device=W.device)
    _check(lib().heal_pack_f16_weight(W.data_ptr(), N, K, _ld(shape, stride), int(e),
                                      out.data_ptr(), _stream()), "heal_pack_f16_weight")
    return out


def heal_gemm_f16w(A, W16, N, e, products, out=None, instance=INSTANCE_AUTO):
    """HEAL-Base (products=1) or HEAL-Full (products=2): A (M x K float32) times
    the packed FP16 weight of an N x K matrix, scaled back by 2^-e."""
    shape, stride = _tensor(A, "A", torch.float32, 2)
    M, K = shape
    C, stride_c = _output(out, A, (M, N))
    if W16.numel() < heal_packed_size(K, N, 1):
        raise HealError("W16 is smaller than the packed size")
    _check(_lib.heal_gemm_f16w_instance(int(instance), int(products), M, N, K, A.data_ptr(),
                                        _ld(shape, stride), W16.data_ptr(), int(e), C.data_ptr(),
                                        _ld((M, N), stride_c), _stream()), "heal_gemm_f16w")
    return C


def heal_presplit_b(B, trans_b=False, out=None):
    """Packed bf16 (hi, lo) of B (K x N, or N x K with trans_b)."""
    shape, stride = _tensor(B, "B", torch.float32, 2)
    K, N = (shape[1], shape[0]) if trans_b else (shape[0], shape[1])
    size = heal_packed_size(K, N, 2)
    out = out if out is not None else torch.empty(size, dtype=torch.uint16, device=B.device)
    _check(lib().heal_presplit_b(B.data_ptr(), K, N, _ld(shape, stride), 1 if trans_b else 0,
                                 out.data_ptr(), _stream()), "heal_presplit_b")
    return out


def heal_gemm_f32_presplit(A, Bp, N, out=None, instance=INSTANCE_AUTO):
    """C = A @ B from the pre-split packed B of an operand with N columns."""
    shape, stride = _tensor(A, "A", torch.float32, 2)
    M, K = shape
    C, stride_c = _output(out, A, (M, N))
    if Bp.numel() < heal_packed_size(K, N, 2):
        raise HealError("Bp is smaller than the packed size")
    _check(_lib.heal_gemm_f32_presplit_instance(int(instance), M, N, K, A.data_ptr(),
                                                _ld(shape, stride), Bp.data_ptr(), C.data_ptr(),
                                                _ld((M, N), stride_c), _stream()),
           "heal_gemm_f32_presplit")
    return C


def heal_quantize_i16(x, q=None, maxabs=None):
    """INT16 codes of a contiguous float32 CUDA tensor and its max|x| (device)."""
    _tensor(x, "x", torch.float32)
    if not x.is_contiguous():
        raise HealError("x must be contiguous")
    q = q if q is not None else torch.empty(x.shape, dtype=torch.int16, device=x.device)
    maxabs = maxabs if maxabs is not None else torch.empty(1, dtype=torch.float32, device=x.device)
    _check((_lib or lib()).heal_quantize_i16(x.data_ptr(), x.numel(), q.data_ptr(),
                                             maxabs.data_ptr(), _stream()), "heal_quantize_i16")
    return q, maxabs


def heal_scores_i16(Q, Kt, maxQ, maxK, alpha=1.0, out=None):
    """Scores of INT16 codes: Q (batch x M x d), Kt (batch x N x d) -> batch x M x N
    FP32 (2-D inputs give a 2-D result)."""
    squeeze = Q.dim() == 2
    if squeeze:
        Q, Kt = Q.unsqueeze(0), Kt.unsqueeze(0)
        out = out.unsqueeze(0) if out is not None else None
    shape_q, stride_q = _tensor(Q, "Q", torch.int16, 3)
    shape_k, stride_k = _tensor(Kt, "Kt", torch.int16, 3)
    bat, M, K = shape_q
    N = shape_k[1]
    if shape_k[0] != bat or shape_k[2] != K:
        raise HealError("shapes do not match: Q %s, Kt %s" % (tuple(Q.shape), tuple(Kt.shape)))
    S = out if out is not None else torch.empty((bat, M, N), dtype=torch.float32, device=Q.device)
    shape_s, stride_s = _tensor(S, "out", torch.float32, 3)
    many = bat > 1
    _check((_lib or lib()).heal_scores_i16(
        M, N, K, Q.data_ptr(), _ld(shape_q, stride_q), stride_q[0] if many else 0,
        maxQ.data_ptr(), Kt.data_ptr(), _ld(shape_k, stride_k), stride_k[0] if many else 0,
        maxK.data_ptr(), ctypes.c_float(alpha), S.data_ptr(), _ld(shape_s, stride_s), stride_s[0] if many else 0,
        bat, _stream()), "heal_scores_i16")
    return S[0] if squeeze else S
