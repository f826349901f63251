"""Thin ctypes binding over libtpo.so: same names as the C ABI in ``include/tpo.h``, argument
marshalling only.  Every step of the operator runs in the library's HIP kernels; there is no
fallback: if the library has not been built, loading raises.

Pointers are plain integers (``tensor.data_ptr()``), the stream is a ``hipStream_t`` as an
integer (``torch.cuda.current_stream().cuda_stream``).
"""
from __future__ import annotations

import ctypes
import os

TPO_F64, TPO_F32 = 0, 1
TPO_OK = 0
TPO_ERR_INVALID_ARG, TPO_ERR_UNSUPPORTED, TPO_ERR_NOT_INITIALIZED = -1, -2, -3
TPO_ERR_DEVICE, TPO_ERR_ALIAS = -4, -5
TPO_FORWARD, TPO_BACKWARD = 0, 1
TPO_VARIANT_AUTO, TPO_VARIANT_PENCIL, TPO_VARIANT_MFMA, TPO_VARIANT_PENCIL_MM = 0, 1, 2, 3
TPO_MAX_N = 16

LIB_PATH = os.path.join(os.path.dirname(os.path.abspath(__file__)), "libtpo.so")
BENCH_LIB_PATH = os.path.join(os.path.dirname(os.path.abspath(__file__)), "libtpo_bench.so")
_lib = None
_bench_lib = None


class TpoError(RuntimeError):
    def __init__(self, status: int, what: str):
        super().__init__(f"{what}: {status_string(status)} ({status})")
        self.status = status


def lib():
    """Load libtpo.so (once).  Raises if it has not been built."""
    global _lib
    if _lib is None:
        if not os.path.exists(LIB_PATH):
            raise RuntimeError(
                f"{LIB_PATH} is missing: build it with `python -m paper_2604_19906_amd.build`")
        l = ctypes.CDLL(LIB_PATH)
        vp, ci, cll = ctypes.c_void_p, ctypes.c_int, ctypes.c_longlong
        l.tpo_create.argtypes = []
        l.tpo_create.restype = ci
        l.tpo_destroy.argtypes = []
        l.tpo_destroy.restype = ci
        l.tpo_ihelm_apply.argtypes = [vp, vp, vp, vp, vp, vp, ci, cll, ci, vp]
        l.tpo_ihelm_apply.restype = ci
        l.tpo_ihelm_apply_variant.argtypes = [vp, vp, vp, vp, vp, vp, ci, cll, ci, vp, ci]
        l.tpo_ihelm_apply_variant.restype = ci
        l.tpo_ihelm_variant_for.argtypes = [ci, ci, ci]
        l.tpo_ihelm_variant_for.restype = ci
        l.tpo_ihelm_variant_for_batch.argtypes = [ci, ci, ci, cll]
        l.tpo_ihelm_variant_for_batch.restype = ci
        l.tpo_ihelm_has_variant.argtypes = [ci, ci, ci]
        l.tpo_ihelm_has_variant.restype = ci
        l.tpo_ihelm_apply_sep.argtypes = [vp] * 9 + [ci, cll, ci, vp]
        l.tpo_ihelm_apply_sep.restype = ci
        l.tpo_ihelm_apply_sep_variant.argtypes = [vp] * 9 + [ci, cll, ci, vp, ci]
        l.tpo_ihelm_apply_sep_variant.restype = ci
        l.tpo_ihelm_sep_variant_for.argtypes = [ci, ci]
        l.tpo_ihelm_sep_variant_for.restype = ci
        l.tpo_ihelm_sep_variant_for_batch.argtypes = [ci, ci, ci, cll]
        l.tpo_ihelm_sep_variant_for_batch.restype = ci
        l.tpo_ihelm_sep_has_variant.argtypes = [ci, ci, ci]
        l.tpo_ihelm_sep_has_variant.restype = ci
        l.tpo_ihelm_apply_aniso.argtypes = [vp, vp, vp, vp, vp, vp, ci, ci, ci, cll, ci, vp]
        l.tpo_ihelm_apply_aniso.restype = ci
        l.tpo_transform_apply.argtypes = [vp, vp, vp, vp, vp, ci, cll, ci, ci, vp]
        l.tpo_transform_apply.restype = ci
        l.tpo_convection_apply.argtypes = [vp, vp, vp, vp, vp, ci, ci, cll, ci, vp]
        l.tpo_convection_apply.restype = ci
        l.tpo_convection_has_shape.argtypes = [ci, ci, ci]
        l.tpo_convection_has_shape.restype = ci
        l.tpo_status_string.argtypes = [ci]
        l.tpo_status_string.restype = ctypes.c_char_p
        _lib = l
    return _lib


def status_string(status: int) -> str:
    return lib().tpo_status_string(int(status)).decode()


def tpo_create() -> int:
    return lib().tpo_create()


def tpo_destroy() -> int:
    return lib().tpo_destroy()


def tpo_ihelm_apply(u, S_x, S_y, S_z, D, v, n, num_elems, dtype, stream) -> int:
    """Raw call: integer device pointers in, status out."""
    return lib().tpo_ihelm_apply(u, S_x, S_y, S_z, D, v, int(n), int(num_elems), int(dtype),
                                 stream)


def tpo_ihelm_apply_variant(u, S_x, S_y, S_z, D, v, n, num_elems, dtype, stream,
                            variant) -> int:
    return lib().tpo_ihelm_apply_variant(u, S_x, S_y, S_z, D, v, int(n), int(num_elems),
                                         int(dtype), stream, int(variant))


def tpo_ihelm_variant_for(n: int, dtype: int, shared_s: bool = False) -> int:
    return lib().tpo_ihelm_variant_for(int(n), int(dtype), int(bool(shared_s)))


def tpo_ihelm_variant_for_batch(n: int, dtype: int, shared_s: bool, num_elems: int) -> int:
    return lib().tpo_ihelm_variant_for_batch(int(n), int(dtype), int(bool(shared_s)),
                                             int(num_elems))


def tpo_ihelm_has_variant(n: int, dtype: int, variant: int) -> bool:
    return bool(lib().tpo_ihelm_has_variant(int(n), int(dtype), int(variant)))


def tpo_ihelm_apply_sep(u, S_x, S_y, S_z, lam_x, lam_y, lam_z, mu, v, n, num_elems, dtype,
                        stream) -> int:
    """Raw call of the separable-diagonal form: integer device pointers in, status out."""
    return lib().tpo_ihelm_apply_sep(u, S_x, S_y, S_z, lam_x, lam_y, lam_z, mu, v, int(n),
                                     int(num_elems), int(dtype), stream)


def tpo_ihelm_apply_sep_variant(u, S_x, S_y, S_z, lam_x, lam_y, lam_z, mu, v, n, num_elems,
                                dtype, stream, variant) -> int:
    return lib().tpo_ihelm_apply_sep_variant(u, S_x, S_y, S_z, lam_x, lam_y, lam_z, mu, v,
                                             int(n), int(num_elems), int(dtype), stream,
                                             int(variant))


def tpo_ihelm_sep_variant_for(n: int, dtype: int) -> int:
    return lib().tpo_ihelm_sep_variant_for(int(n), int(dtype))


def tpo_ihelm_sep_variant_for_batch(n: int, dtype: int, shared_s: bool, num_elems: int) -> int:
    return lib().tpo_ihelm_sep_variant_for_batch(int(n), int(dtype), int(bool(shared_s)),
                                                 int(num_elems))


def tpo_ihelm_sep_has_variant(n: int, dtype: int, variant: int) -> bool:
    return bool(lib().tpo_ihelm_sep_has_variant(int(n), int(dtype), int(variant)))


def tpo_ihelm_apply_aniso(u, S_x, S_y, S_z, D, v, n_x, n_y, n_z, num_elems, dtype, stream) -> int:
    """Raw call of the operator on anisotropic elements: integer device pointers in, status out."""
    return lib().tpo_ihelm_apply_aniso(u, S_x, S_y, S_z, D, v, int(n_x), int(n_y), int(n_z),
                                       int(num_elems), int(dtype), stream)


def tpo_transform_apply(u, S_x, S_y, S_z, t, n, num_elems, dtype, direction, stream) -> int:
    """Raw call of one half of the operator: integer device pointers in, status out."""
    return lib().tpo_transform_apply(u, S_x, S_y, S_z, t, int(n), int(num_elems), int(dtype),
                                     int(direction), stream)


def tpo_convection_apply(P, M, D_vq, I_vq, F, n_v, n_q, num_elems, dtype, stream) -> int:
    """Raw call of the convection volume term: integer device pointers in, status out."""
    return lib().tpo_convection_apply(P, M, D_vq, I_vq, F, int(n_v), int(n_q), int(num_elems),
                                      int(dtype), stream)


def tpo_convection_has_shape(n_v: int, n_q: int, dtype: int) -> bool:
    return bool(lib().tpo_convection_has_shape(int(n_v), int(n_q), int(dtype)))


def bench_lib():
    """Load libtpo_bench.so, the benchmark's measurement aid (once).  Raises if it is missing."""
    global _bench_lib
    if _bench_lib is None:
        if not os.path.exists(BENCH_LIB_PATH):
            raise RuntimeError(
                f"{BENCH_LIB_PATH} is missing: build it with `python -m paper_2604_19906_amd.build`")
        l = ctypes.CDLL(BENCH_LIB_PATH)
        vp, ci, cll = ctypes.c_void_p, ctypes.c_int, ctypes.c_longlong
        l.tpo_stream_scale.argtypes = [vp, vp, vp, cll, ci, vp]
        l.tpo_stream_scale.restype = ci
        _bench_lib = l
    return _bench_lib


def tpo_stream_scale(u, D, v, count, dtype, stream) -> int:
    """Measurement aid (libtpo_bench.so): v[i] = u[i] * D[i] over flat device arrays."""
    return bench_lib().tpo_stream_scale(u, D, v, int(count), int(dtype), stream)


def check(status: int, what: str = "tpo call") -> None:
    if status != TPO_OK:
        raise TpoError(status, what)


# What the tensor functions below need of torch, looked up once: the dtype codes, the calling
# thread's current device and the raw handle of a device's current stream.  A call on a small
# batch takes less time on the GPU than a Stream object, a module import and repeated attribute
# reads take on the host: fp64 n = 7, 1000 elements, 6.3 us a call against 10.3 with those (4.4 of
# them the library call itself).
_rt = None


def _runtime():
    global _rt
    if _rt is None:
        import torch

        device = getattr(torch._C, "_cuda_getDevice", None)
        stream = getattr(torch._C, "_cuda_getCurrentRawStream", None)
        if device is None or stream is None:    # not part of torch's public interface
            device = torch.cuda.current_device
            stream = lambda dev: torch.cuda.current_stream(dev).cuda_stream
        _rt = ({torch.float64: TPO_F64, torch.float32: TPO_F32}, device, stream)
    return _rt


# The same functions as one native call (csrc/torch_binding.cpp).  It takes the plain case only and returns None for
# everything else, which the Python forms below then check, refuse or compute; a number is a status.  False: not there.
TORCH_BINDING_PATH = os.path.join(os.path.dirname(os.path.abspath(__file__)), "_tpo_torch.so")
_native = None


def binding_versions() -> str:
    """What the native form has compiled in: torch (offsets of a tensor's members), the interpreter, the C header."""
    import hashlib
    import sysconfig

    import torch

    header = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "include", "tpo.h")
    with open(header, "rb") as f:
        digest = hashlib.sha256(f.read()).hexdigest()[:16]
    return f"torch {torch.__version__} {torch.version.git_version}, {sysconfig.get_config_var('SOABI')}, tpo.h {digest}"


def _load_native():
    global _native
    import importlib.util
    import warnings

    import torch  # noqa: F401  (the libraries that the binding is linked to)

    _native = False
    try:
        spec = importlib.util.spec_from_file_location("_tpo_torch", TORCH_BINDING_PATH)
        module = importlib.util.module_from_spec(spec)
        spec.loader.exec_module(module)
        built_for, here = getattr(module, "built_for", "an unknown torch"), binding_versions()
        if built_for != here:
            raise ImportError(f"built for {built_for}, this is {here}")
    except (ImportError, OSError) as e:     # missing, without a symbol it needs, for another torch, interpreter or header
        warnings.warn(f"{TORCH_BINDING_PATH} cannot be used ({e}): tensor functions run in their Python form")
        return _native
    l = lib()
    module.bind(*(ctypes.cast(f, ctypes.c_void_p).value for f in (
        l.tpo_ihelm_apply_variant, l.tpo_ihelm_apply_sep_variant, l.tpo_transform_apply, l.tpo_convection_apply,
        l.tpo_ihelm_apply_aniso)))
    _native = module
    return _native


def _done(r, what):
    if type(r) is int:
        raise TpoError(r, what)
    return r


_CONTIG = "all tensors must be contiguous device tensors of one dtype"


def _plain(t, dtype) -> bool:
    return t.is_contiguous() and t.dtype == dtype and t.is_cuda


def _output(v, u, what):
    """``v`` checked against ``u``, or a new tensor like it."""
    if v is None:
        import torch

        return torch.empty_like(u)
    if not (v.shape == u.shape and _plain(v, u.dtype)):
        raise ValueError(what)
    return v


def _mats_plain(S_x, S_y, S_z, dtype) -> bool:
    return (_plain(S_x, dtype) and (S_y is S_x or _plain(S_y, dtype))
            and (S_z is S_x or _plain(S_z, dtype)))


def _mats_square(S_x, S_y, S_z, n) -> bool:
    return (S_x.shape == (n, n) and (S_y is S_x or S_y.shape == (n, n))
            and (S_z is S_x or S_z.shape == (n, n)))


def _mat_ptrs(S_x, S_y, S_z):
    p = S_x.data_ptr()
    return p, p if S_y is S_x else S_y.data_ptr(), p if S_z is S_x else S_z.data_ptr()


def apply_tensors(u, S_x, S_y, S_z, D, v=None, variant: int = TPO_VARIANT_AUTO):
    """Convenience over torch device tensors: marshals pointers, shape and the current
    stream; raises TpoError on a non-zero status.  Returns ``v`` (allocated if None)."""
    fast = _native if _native is not None else _load_native()
    if fast:
        r = fast.apply(u, S_x, S_y, S_z, D, v, variant)
        if r is not None:
            return r if r is v else _done(r, "tpo_ihelm_apply")
    shape = u.shape
    if len(shape) != 4 or not u.is_cuda:
        raise ValueError("u must be a device tensor of shape [E,n,n,n]")
    dt = u.dtype
    if not (u.is_contiguous() and _mats_plain(S_x, S_y, S_z, dt) and _plain(D, dt)):
        raise ValueError(_CONTIG)
    e, n, n1, n2 = shape
    if n1 != n or n2 != n or D.shape != shape:
        raise ValueError("u and D must both be [E,n,n,n]")
    if not _mats_square(S_x, S_y, S_z, n):
        raise ValueError("S matrices must be [n,n]")
    v = _output(v, u, "v must match u")
    codes, device, stream = _rt or _runtime()
    status = (_lib or lib()).tpo_ihelm_apply_variant(
        u.data_ptr(), *_mat_ptrs(S_x, S_y, S_z), D.data_ptr(), v.data_ptr(), n, e, codes[dt],
        stream(device()), int(variant))
    if status != TPO_OK:
        raise TpoError(status, "tpo_ihelm_apply")
    return v


def apply_sep_tensors(u, S_x, S_y, S_z, lam_x, lam_y, lam_z, mu, v=None,
                      variant: int = TPO_VARIANT_AUTO):
    """Separable-diagonal form over torch device tensors (``lam_*`` are ``[n]``, ``mu`` is
    ``[E]``); marshalling only, like :func:`apply_tensors`."""
    fast = _native if _native is not None else _load_native()
    if fast:
        r = fast.apply_sep(u, S_x, S_y, S_z, lam_x, lam_y, lam_z, mu, v, variant)
        if r is not None:
            return r if r is v else _done(r, "tpo_ihelm_apply_sep")
    shape = u.shape
    if len(shape) != 4 or not u.is_cuda:
        raise ValueError("u must be a device tensor of shape [E,n,n,n]")
    dt = u.dtype
    if not (u.is_contiguous() and _mats_plain(S_x, S_y, S_z, dt)
            and _mats_plain(lam_x, lam_y, lam_z, dt) and _plain(mu, dt)):
        raise ValueError(_CONTIG)
    e, n, n1, n2 = shape
    if n1 != n or n2 != n:
        raise ValueError("u must be [E,n,n,n]")
    if not _mats_square(S_x, S_y, S_z, n):
        raise ValueError("S matrices must be [n,n]")
    if not (lam_x.shape == (n,) and (lam_y is lam_x or lam_y.shape == (n,))
            and (lam_z is lam_x or lam_z.shape == (n,))):
        raise ValueError("lam vectors must be [n]")
    if mu.shape != (e,):
        raise ValueError("mu must be [E]")
    v = _output(v, u, "v must match u")
    codes, device, stream = _rt or _runtime()
    status = (_lib or lib()).tpo_ihelm_apply_sep_variant(
        u.data_ptr(), *_mat_ptrs(S_x, S_y, S_z), *_mat_ptrs(lam_x, lam_y, lam_z), mu.data_ptr(),
        v.data_ptr(), n, e, codes[dt], stream(device()), int(variant))
    if status != TPO_OK:
        raise TpoError(status, "tpo_ihelm_apply_sep")
    return v


def transform_tensors(u, S_x, S_y, S_z, direction: int, t=None):
    """One half of the operator over torch device tensors; marshalling only."""
    fast = _native if _native is not None else _load_native()
    if fast:
        r = fast.transform(u, S_x, S_y, S_z, direction, t)
        if r is not None:
            return r if r is t else _done(r, "tpo_transform_apply")
    shape = u.shape
    if len(shape) != 4 or not u.is_cuda:
        raise ValueError("u must be a device tensor of shape [E,n,n,n]")
    dt = u.dtype
    if not (u.is_contiguous() and _mats_plain(S_x, S_y, S_z, dt)):
        raise ValueError(_CONTIG)
    e, n, n1, n2 = shape
    if n1 != n or n2 != n:
        raise ValueError("u must be [E,n,n,n]")
    if not _mats_square(S_x, S_y, S_z, n):
        raise ValueError("S matrices must be [n,n]")
    t = _output(t, u, "t must match u")
    codes, device, stream = _rt or _runtime()
    status = (_lib or lib()).tpo_transform_apply(
        u.data_ptr(), *_mat_ptrs(S_x, S_y, S_z), t.data_ptr(), n, e, codes[dt],
        int(direction), stream(device()))
    if status != TPO_OK:
        raise TpoError(status, "tpo_transform_apply")
    return t


def convection_tensors(P, M, D_vq, I_vq, F=None):
    """Convection volume term over torch device tensors (``P`` ``[3,3,E,nq,nq,nq]``, ``M``
    ``[E,nq,nq,nq]``, ``D_vq``/``I_vq`` ``[nv,nq]``); marshalling only.  Returns ``F``
    ``[3,E,nv,nv,nv]``."""
    fast = _native if _native is not None else _load_native()
    if fast:
        r = fast.convection(P, M, D_vq, I_vq, F)
        if r is not None:
            return r if r is F else _done(r, "tpo_convection_apply")
    dt = P.dtype
    if not (_plain(P, dt) and _plain(M, dt) and _plain(D_vq, dt) and _plain(I_vq, dt)):
        raise ValueError(_CONTIG)
    if D_vq.dim() != 2 or I_vq.shape != D_vq.shape:
        raise ValueError("D_vq and I_vq must both be [nv,nq]")
    nv, nq = D_vq.shape
    m_shape = M.shape
    if len(m_shape) != 4 or m_shape[1:] != (nq, nq, nq):
        raise ValueError("M must be [E,nq,nq,nq]")
    e = m_shape[0]
    if P.shape != (3, 3, e, nq, nq, nq):
        raise ValueError("P must be [3,3,E,nq,nq,nq]")
    if F is None:
        import torch

        F = torch.empty((3, e, nv, nv, nv), dtype=dt, device=P.device)
    elif not (F.shape == (3, e, nv, nv, nv) and _plain(F, dt)):
        raise ValueError("F must be [3,E,nv,nv,nv]")
    codes, device, stream = _rt or _runtime()
    status = (_lib or lib()).tpo_convection_apply(
        P.data_ptr(), M.data_ptr(), D_vq.data_ptr(), I_vq.data_ptr(), F.data_ptr(), nv, nq, e,
        codes[dt], stream(device()))
    if status != TPO_OK:
        raise TpoError(status, "tpo_convection_apply")
    return F


def apply_aniso_tensors(u, S_x, S_y, S_z, D, v=None):
    """The operator on anisotropic elements over torch device tensors (``u``, ``D``
    ``[E,nx,ny,nz]``; ``S_x`` ``[nx,nx]``, ``S_y`` ``[ny,ny]``, ``S_z`` ``[nz,nz]``);
    marshalling only."""
    fast = _native if _native is not None else _load_native()
    if fast:
        r = fast.apply_aniso(u, S_x, S_y, S_z, D, v)
        if r is not None:
            return r if r is v else _done(r, "tpo_ihelm_apply_aniso")
    shape = u.shape
    if len(shape) != 4 or not u.is_cuda or D.shape != shape:
        raise ValueError("u and D must be device tensors of shape [E,nx,ny,nz]")
    dt = u.dtype
    if not (u.is_contiguous() and _mats_plain(S_x, S_y, S_z, dt) and _plain(D, dt)):
        raise ValueError(_CONTIG)
    e, nx, ny, nz = shape
    if S_x.shape != (nx, nx) or S_y.shape != (ny, ny) or S_z.shape != (nz, nz):
        raise ValueError("S matrices must be [nx,nx], [ny,ny], [nz,nz]")
    v = _output(v, u, "v must match u")
    codes, device, stream = _rt or _runtime()
    status = (_lib or lib()).tpo_ihelm_apply_aniso(
        u.data_ptr(), *_mat_ptrs(S_x, S_y, S_z), D.data_ptr(), v.data_ptr(), nx, ny, nz, e,
        codes[dt], stream(device()))
    if status != TPO_OK:
        raise TpoError(status, "tpo_ihelm_apply_aniso")
    return v
