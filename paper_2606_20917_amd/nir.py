"""Thin ctypes binding of libnir.so (argument marshalling only).

Every function has the name of the C entry point it calls and takes torch
tensors (or raw integer addresses) where the C ABI takes pointers.  Device
tensors must be contiguous CUDA/HIP tensors; the current torch stream is
used unless a stream is given.  Nothing here computes: if the library is
missing the first call raises, there is no fallback.
"""
import ctypes
import os

HERE = os.path.dirname(os.path.abspath(__file__))
LIBPATH = os.path.join(HERE, "libnir.so")

HEX, PRISM, TET, PYR = 0, 1, 2, 3
F64, F32 = 0, 1
MATH_NATIVE, MATH_F16SPLIT = 0, 1
MAP_VERTEX, MAP_VERTEX_SIN = 0, 1
MIXED_AUTO, MIXED_PERSISTENT, MIXED_PER_BATCH = range(3)
(VARIANT_AUTO, VARIANT_GENERIC, VARIANT_PENCIL, VARIANT_PENCIL_U2, VARIANT_PENCIL_E1, VARIANT_PENCIL_PF,
 VARIANT_PENCIL_SPLIT, VARIANT_PENCIL_GP, VARIANT_PENCIL_SPLIT_GP, VARIANT_PENCIL_EO,
 VARIANT_PENCIL_EO_SPLIT, VARIANT_DENSE) = range(12)
CG_FP64, CG_MIXED_F32, CG_MIXED_F16SPLIT = 0, 1, 2

(TAB_Z1, TAB_Z2, TAB_Z3, TAB_W1, TAB_W2, TAB_W3, TAB_T1, TAB_DT1, TAB_T2, TAB_DT2, TAB_T3, TAB_DT3,
 TAB_D1, TAB_D2, TAB_D3, TAB_WQ, TAB_XI, TAB_MODE_PQR, TAB_POINT_IJK, TAB_PAIR) = range(20)
INT_TABLES = (TAB_MODE_PQR, TAB_POINT_IJK, TAB_PAIR)

STATUS = {0: "NIR_OK", 1: "NIR_EINVAL", 2: "NIR_ENOTSUP", 3: "NIR_ENOMEM", 4: "NIR_EHIP",
          5: "NIR_ENONFINITE", 6: "NIR_EBREAKDOWN", 7: "NIR_ENOCONV"}


class NirError(RuntimeError):
    def __init__(self, status, msg):
        super().__init__(f"{STATUS.get(status, status)}: {msg}")
        self.status = status


class nir_batch(ctypes.Structure):
    _fields_ = [("shape", ctypes.c_int32), ("nmodes", ctypes.c_int32), ("nquad", ctypes.c_int32),
                ("deformed", ctypes.c_int32), ("nelmt", ctypes.c_int64), ("dtype", ctypes.c_int32),
                ("math", ctypes.c_int32)]


class nir_geom(ctypes.Structure):
    _fields_ = [("dxi_dx", ctypes.c_void_p), ("jac", ctypes.c_void_p), ("helm", ctypes.c_void_p)]


class nir_cg_info(ctypes.Structure):
    _fields_ = [("outer_iters", ctypes.c_int32), ("inner_iters", ctypes.c_int32),
                ("rel_residual", ctypes.c_double), ("seconds", ctypes.c_double)]


_lib = None
_vp, _i32, _i64, _dbl = ctypes.c_void_p, ctypes.c_int32, ctypes.c_int64, ctypes.c_double
_SIGS = {
    "nir_nmodes": (_i64, [_i32, _i32]),
    "nir_last_error": (ctypes.c_char_p, []),
    "nir_version": (ctypes.c_char_p, []),
    "nir_quadrature_host": (_i32, [_i32, _i32, _i32, _vp, _vp]),
    "nir_table_size": (_i64, [_i32, _i32, _i32, _i32]),
    "nir_table_host": (_i32, [_i32, _i32, _i32, _i32, _vp]),
    "nir_basis_create": (_i32, [_i32, _i32, _i32, ctypes.POINTER(_vp)]),
    "nir_basis_destroy": (_i32, [_vp]),
    "nir_basis_table_device": (_vp, [_vp, _i32]),
    "nir_geom_from_vertices": (_i32, [ctypes.POINTER(nir_batch), _vp, _vp, _i32, _dbl, _vp, _vp, _vp, _vp, _vp]),
    "nir_geom_prepare": (_i32, [ctypes.POINTER(nir_batch), _vp, _vp, _vp, _vp, _vp, _vp, _vp]),
    "nir_bwd_trans": (_i32, [ctypes.POINTER(nir_batch), _vp, _vp, _vp, _vp]),
    "nir_phys_deriv": (_i32, [ctypes.POINTER(nir_batch), _vp, ctypes.POINTER(nir_geom), _vp, _vp, _vp, _vp, _vp]),
    "nir_iprod_wrt_base": (_i32, [ctypes.POINTER(nir_batch), _vp, ctypes.POINTER(nir_geom), _vp, _vp, _vp]),
    "nir_iprod_wrt_deriv_base": (_i32, [ctypes.POINTER(nir_batch), _vp, ctypes.POINTER(nir_geom), _vp, _vp, _vp,
                                        _vp, _vp]),
    "nir_helmholtz_apply": (_i32, [ctypes.POINTER(nir_batch), _vp, ctypes.POINTER(nir_geom), _dbl, _vp, _vp, _vp]),
    "nir_helmholtz_apply_fields": (_i32, [ctypes.POINTER(nir_batch), _vp, ctypes.POINTER(nir_geom), _dbl, _i32, _vp,
                                          _vp, _vp]),
    "nir_helmholtz_apply_trilinear": (_i32, [ctypes.POINTER(nir_batch), _vp, _vp, _dbl, _vp, _vp, _vp]),
    "nir_helmholtz_apply_nodal": (_i32, [ctypes.POINTER(nir_batch), _vp, ctypes.POINTER(nir_geom), _dbl, _vp, _vp,
                                         _vp]),
    "nir_set_helmholtz_variant": (_i32, [_i32, _i32, _i32, _i32]),
    "nir_points_from_vertices": (_i32, [ctypes.POINTER(nir_batch), _vp, _vp, _i32, _dbl, _vp, _vp]),
    "nir_c0_nglobal_hex": (_i64, [_i32, _i32]),
    "nir_c0_map_hex_host": (_i32, [_i32, _i32, _vp]),
    "nir_c0_map_hex": (_i32, [_i32, _i32, _vp, _vp]),
    "nir_assembly_create": (_i32, [_vp, _i64, _i32, _i64, ctypes.POINTER(_vp)]),
    "nir_assembly_destroy": (_i32, [_vp]),
    "nir_gather": (_i32, [_vp, _i32, _vp, _vp, _vp]),
    "nir_scatter_add": (_i32, [_vp, _i32, _vp, _vp, _vp]),
    "nir_helmholtz_diagonal": (_i32, [ctypes.POINTER(nir_batch), _vp, ctypes.POINTER(nir_geom), _dbl, _vp, _vp]),
    "nir_cg_plan_create": (_i32, [ctypes.POINTER(nir_batch), _vp, ctypes.POINTER(nir_geom), _vp, _vp, _dbl,
                                  ctypes.POINTER(_vp)]),
    "nir_cg_solve": (_i32, [_vp, _i32, _vp, _vp, _dbl, _i32, _dbl, ctypes.POINTER(nir_cg_info), _vp]),
    "nir_cg_plan_destroy": (_i32, [_vp]),
    "nir_mixed_plan_create": (_i32, [_i32, _vp, _vp, _vp, ctypes.POINTER(_vp)]),
    "nir_mixed_helmholtz_apply": (_i32, [_vp, _dbl, _vp, _vp, _vp]),
    "nir_mixed_plan_info": (_i32, [_vp, _vp, _vp, _vp, _vp, _vp]),
    "nir_mixed_plan_set_strategy": (_i32, [_vp, _i32]),
    "nir_mixed_plan_timings": (_i32, [_vp, _vp, _vp, _vp]),
    "nir_mixed_plan_destroy": (_i32, [_vp]),
    "nir_mixed_helmholtz_apply_noalloc": (_i32, [_i32, _vp, _vp, _vp, _dbl, _vp, _vp, _vp]),
    "nir_get_helmholtz_variant": (_i32, [_i32, _i32, _i32]),
    "nir_get_helmholtz_variant_of": (_i32, [ctypes.POINTER(nir_batch)]),
    "nir_autotune_helmholtz": (_i32, [ctypes.POINTER(nir_batch), _vp, ctypes.POINTER(nir_geom), _dbl, _vp, _vp, _i32,
                                      _vp, _vp, _vp]),
    "nir_autotune_save": (_i32, [ctypes.c_char_p]),
    "nir_autotune_load": (_i32, [ctypes.c_char_p]),
}


def lib():
    """The loaded libnir.so; raises if it has not been built."""
    global _lib
    if _lib is None:
        if not os.path.exists(LIBPATH):
            raise RuntimeError(f"{LIBPATH} is missing: build it with `python -m paper_2606_20917_amd.build`")
        L = ctypes.CDLL(LIBPATH)
        for name, (res, args) in _SIGS.items():
            f = getattr(L, name, None)
            if f is None:
                continue
            f.restype, f.argtypes = res, args
        _lib = L
    return _lib


def _check(st):
    if st != 0:
        raise NirError(st, lib().nir_last_error().decode())


def _ptr(x):
    """Address of a contiguous device tensor, or an int (a raw address, passed unchecked);
    None -> NULL.  Host tensors are rejected: the library would read them as device memory."""
    if x is None:
        return None
    if isinstance(x, int):
        return x
    if not x.is_contiguous():
        raise NirError(1, "tensor must be contiguous")
    if not x.is_cuda:
        raise NirError(1, f"tensor on {x.device}: the library takes device memory")
    return x.data_ptr()


_TORCH_DT = {F64: "float64", F32: "float32"}
_dtypes = {}     # F64, F32, "int32" -> torch.dtype, filled at the first match by name
_modes = {}      # (shape, P) -> mode count of valid shapes and orders


def _need(x, name, count, dt, device=False):
    """Check a tensor argument before its address crosses the ABI: element type `dt` (F64, F32
    or "int32") and at least `count` elements; with `device`, also contiguous device memory
    (the other tensors get that check from _ptr when the call is marshalled).  None and raw
    integer addresses pass through (the C side rejects NULL where it needs a pointer)."""
    if x is None or isinstance(x, int):
        return
    if x.dtype is not _dtypes.get(dt):
        want = _TORCH_DT.get(dt, dt)
        got = str(x.dtype).replace("torch.", "")
        if got != want:
            raise NirError(1, f"{name}: element type {got}, the call needs {want}")
        _dtypes[dt] = x.dtype
    if x.numel() < count:
        raise NirError(1, f"{name}: {x.numel()} elements, the call needs at least {count}")
    if device:
        _ptr(x)


def _dims(b):
    """(nelmt, M, Q^3, geometry points per element) of a batch; M = 0 for an invalid shape/order."""
    key = b.shape, b.nmodes
    M = _modes.get(key)
    if M is None:
        M = max(0, int(lib().nir_nmodes(*key)))
        if M and key[1] <= 16:
            _modes[key] = M
    nq = b.nquad ** 3
    return b.nelmt, M, nq, (nq if b.deformed else 1)


def _need_geom(b, g, dxi=False, jac=False, helm=False, dt=None, dims=None):
    """Check the tensors a nir_geom was built from (nir.geom keeps them) against the batch (whose
    _dims the caller may pass)."""
    ne, _, _, ng = _dims(b) if dims is None else dims
    dt = b.dtype if dt is None else dt
    t = getattr(g, "_tensors", (None, None, None))
    if dxi:
        _need(t[0], "geom.dxi_dx", ne * 9 * ng, dt, device=True)
    if jac:
        _need(t[1], "geom.jac", ne * ng, dt, device=True)
    if helm:
        _need(t[2], "geom.helm", ne * 7 * ng, dt, device=True)


_current = None   # (device index, its current stream's address) getters of an initialised torch


def _stream(stream):
    """Address of the stream to enqueue on: the one given, or torch's current stream of the current
    device, asked for at every call (through torch's own getters once torch is initialised: a
    Stream object for each call costs as much as the kernel launch, 1.7 us)."""
    global _current
    if stream is not None:
        return stream if isinstance(stream, int) else stream.cuda_stream
    if _current is not None:
        return _current[1](_current[0]())
    import torch
    s = torch.cuda.current_stream().cuda_stream   # initialises torch
    get = getattr(torch._C, "_cuda_getCurrentRawStream", None), getattr(torch._C, "_cuda_getDevice", None)
    if None not in get:
        _current = get[1], get[0]
    return s


def _forget_stream_getters():
    """In a forked child: torch refuses the GPU there, so its first call goes through torch again."""
    global _current
    _current = None


os.register_at_fork(after_in_child=_forget_stream_getters)


def batch(shape, P, nelmt, dtype=F64, deformed=1, math=MATH_NATIVE, Q=None):
    return nir_batch(shape, P, P + 1 if Q is None else Q, deformed, nelmt, dtype, math)


def _addr(x):
    if x is None or isinstance(x, int):
        return x
    if not x.is_contiguous():
        raise NirError(1, "tensor must be contiguous")
    return x.data_ptr()


def geom(dxi_dx=None, jac=None, helm=None):
    """A nir_geom of device tensors.  It keeps the tensors: each call checks the fields it
    uses (device, element type, size against its batch) before the addresses cross the ABI."""
    g = nir_geom(_addr(dxi_dx), _addr(jac), _addr(helm))
    g._tensors = (dxi_dx, jac, helm)
    return g


class Basis:
    """Owner of a nir_basis handle."""

    def __init__(self, shape, P, Q=None):
        self.shape, self.P, self.Q = shape, P, P + 1 if Q is None else Q
        h = ctypes.c_void_p()
        _check(lib().nir_basis_create(shape, P, self.Q, ctypes.byref(h)))
        self.handle = h

    def __del__(self):
        if getattr(self, "handle", None) is not None and _lib is not None:
            _lib.nir_basis_destroy(self.handle)
            self.handle = None

    @property
    def _as_parameter_(self):
        return self.handle


def _basis(b):
    return b.handle if isinstance(b, Basis) else b


# ------------------------------------------------------------------ entry points
def nir_nmodes(shape, P):
    return lib().nir_nmodes(shape, P)


def nir_version():
    return lib().nir_version().decode()


def nir_last_error():
    return lib().nir_last_error().decode()


def nir_quadrature_host(rule, alpha, Q):
    import numpy as np
    z, w = np.zeros(Q), np.zeros(Q)
    _check(lib().nir_quadrature_host(rule, alpha, Q, z.ctypes.data, w.ctypes.data))
    return z, w


def nir_table_size(shape, P, Q, tid):
    return lib().nir_table_size(shape, P, Q, tid)


def nir_table_host(shape, P, Q, tid):
    import numpy as np
    n = nir_table_size(shape, P, Q, tid)
    if n < 0:
        raise NirError(1, "invalid table request")
    out = np.zeros(n, dtype=np.int32 if tid in INT_TABLES else np.float64)
    _check(lib().nir_table_host(shape, P, Q, tid, out.ctypes.data))
    return out


def nir_basis_create(shape, P, Q=None):
    return Basis(shape, P, Q)


_NVERT = {HEX: 8, PRISM: 6, TET: 4, PYR: 5}


def nir_geom_from_vertices(b, basis, verts, map_, amp, dxi_dx=None, jac=None, helm64=None, helm32=None,
                           stream=None):
    ne, _, _, ng = _dims(b)
    _need(verts, "verts", ne * _NVERT.get(b.shape, 0) * 3, F64)
    _need(dxi_dx, "dxi_dx", ne * 9 * ng, F64)
    _need(jac, "jac", ne * ng, F64)
    _need(helm64, "helm64", ne * 7 * ng, F64)
    _need(helm32, "helm32", ne * 7 * ng, F32)
    _check(lib().nir_geom_from_vertices(ctypes.byref(b), _basis(basis), _ptr(verts), map_, amp, _ptr(dxi_dx),
                                        _ptr(jac), _ptr(helm64), _ptr(helm32), _stream(stream)))


def nir_geom_prepare(b, basis, jacobian, dxi_dx=None, jac=None, helm64=None, helm32=None, stream=None):
    ne, _, _, ng = _dims(b)
    _need(jacobian, "jacobian", ne * 9 * ng, F64)
    _need(dxi_dx, "dxi_dx", ne * 9 * ng, F64)
    _need(jac, "jac", ne * ng, F64)
    _need(helm64, "helm64", ne * 7 * ng, F64)
    _need(helm32, "helm32", ne * 7 * ng, F32)
    _check(lib().nir_geom_prepare(ctypes.byref(b), _basis(basis), _ptr(jacobian), _ptr(dxi_dx), _ptr(jac),
                                  _ptr(helm64), _ptr(helm32), _stream(stream)))


def nir_bwd_trans(b, basis, coef, phys, stream=None):
    ne, M, nq, _ = _dims(b)
    _need(coef, "coef", ne * M, b.dtype)
    _need(phys, "phys", ne * nq, b.dtype)
    _check(lib().nir_bwd_trans(ctypes.byref(b), _basis(basis), _ptr(coef), _ptr(phys), _stream(stream)))


def nir_phys_deriv(b, basis, g, phys, d0, d1, d2, stream=None):
    dims = _dims(b)
    ne, M, nq, _ = dims
    for name, t in (("phys", phys), ("d0", d0), ("d1", d1), ("d2", d2)):
        _need(t, name, ne * nq, b.dtype)
    _need_geom(b, g, dxi=True, dims=dims)
    _check(lib().nir_phys_deriv(ctypes.byref(b), _basis(basis), ctypes.byref(g), _ptr(phys), _ptr(d0), _ptr(d1),
                                _ptr(d2), _stream(stream)))


def nir_iprod_wrt_base(b, basis, g, phys, coef, stream=None):
    dims = _dims(b)
    ne, M, nq, _ = dims
    _need(phys, "phys", ne * nq, b.dtype)
    _need(coef, "coef", ne * M, b.dtype)
    _need_geom(b, g, jac=True, dims=dims)
    _check(lib().nir_iprod_wrt_base(ctypes.byref(b), _basis(basis), ctypes.byref(g), _ptr(phys), _ptr(coef),
                                    _stream(stream)))


def nir_iprod_wrt_deriv_base(b, basis, g, f0, f1, f2, coef, stream=None):
    dims = _dims(b)
    ne, M, nq, _ = dims
    for name, t in (("f0", f0), ("f1", f1), ("f2", f2)):
        _need(t, name, ne * nq, b.dtype)
    _need(coef, "coef", ne * M, b.dtype)
    _need_geom(b, g, dxi=True, jac=True, dims=dims)
    _check(lib().nir_iprod_wrt_deriv_base(ctypes.byref(b), _basis(basis), ctypes.byref(g), _ptr(f0), _ptr(f1),
                                          _ptr(f2), _ptr(coef), _stream(stream)))


def nir_helmholtz_apply(b, basis, g, lam, coef_in, coef_out, stream=None):
    dims = _dims(b)
    ne, M, _, _ = dims
    _need(coef_in, "coef_in", ne * M, b.dtype)
    _need(coef_out, "coef_out", ne * M, b.dtype)
    _need_geom(b, g, helm=True, dims=dims)
    _check(lib().nir_helmholtz_apply(ctypes.byref(b), _basis(basis), ctypes.byref(g), lam, _ptr(coef_in),
                                     _ptr(coef_out), _stream(stream)))


def nir_helmholtz_apply_fields(b, basis, g, lam, nfields, coef_in, coef_out, stream=None):
    dims = _dims(b)
    ne, M, _, _ = dims
    _need(coef_in, "coef_in", ne * max(nfields, 0) * M, b.dtype)
    _need(coef_out, "coef_out", ne * max(nfields, 0) * M, b.dtype)
    _need_geom(b, g, helm=True, dims=dims)
    _check(lib().nir_helmholtz_apply_fields(ctypes.byref(b), _basis(basis), ctypes.byref(g), lam, nfields,
                                            _ptr(coef_in), _ptr(coef_out), _stream(stream)))


def nir_helmholtz_apply_trilinear(b, basis, verts, lam, coef_in, coef_out, stream=None):
    ne, M, _, _ = _dims(b)
    _need(verts, "verts", ne * 24, F64)
    _need(coef_in, "coef_in", ne * M, b.dtype)
    _need(coef_out, "coef_out", ne * M, b.dtype)
    _check(lib().nir_helmholtz_apply_trilinear(ctypes.byref(b), _basis(basis), _ptr(verts), lam, _ptr(coef_in),
                                               _ptr(coef_out), _stream(stream)))


def nir_helmholtz_apply_nodal(b, basis, g, lam, u_in, u_out, stream=None):
    dims = _dims(b)
    ne, _, nq, _ = dims
    _need(u_in, "u_in", ne * nq, b.dtype)
    _need(u_out, "u_out", ne * nq, b.dtype)
    _need_geom(b, g, helm=True, dims=dims)
    _check(lib().nir_helmholtz_apply_nodal(ctypes.byref(b), _basis(basis), ctypes.byref(g), lam, _ptr(u_in),
                                           _ptr(u_out), _stream(stream)))


def nir_set_helmholtz_variant(shape, P, dtype, variant):
    _check(lib().nir_set_helmholtz_variant(shape, P, dtype, variant))


def nir_get_helmholtz_variant(shape, P, dtype):
    return lib().nir_get_helmholtz_variant(shape, P, dtype)


def nir_get_helmholtz_variant_of(b):
    """The variant that nir_helmholtz_apply would run now on the batch b; -1 if it is invalid."""
    return lib().nir_get_helmholtz_variant_of(ctypes.byref(b))


def nir_points_from_vertices(b, basis, verts, map_, amp, xyz, stream=None):
    ne, _, nq, _ = _dims(b)
    _need(verts, "verts", ne * _NVERT.get(b.shape, 0) * 3, F64)
    _need(xyz, "xyz", ne * 3 * nq, F64)
    _check(lib().nir_points_from_vertices(ctypes.byref(b), _basis(basis), _ptr(verts), map_, amp, _ptr(xyz),
                                          _stream(stream)))


def nir_c0_nglobal_hex(n, P):
    return lib().nir_c0_nglobal_hex(n, P)


def nir_c0_map_hex_host(n, P):
    import numpy as np
    out = np.zeros((n ** 3, P ** 3), dtype=np.int32)
    _check(lib().nir_c0_map_hex_host(n, P, out.ctypes.data))
    return out


def nir_c0_map_hex(n, P, l2g, stream=None):
    _need(l2g, "l2g", n ** 3 * P ** 3, "int32")
    _check(lib().nir_c0_map_hex(n, P, _ptr(l2g), _stream(stream)))


class Assembly:
    """Owner of a nir_assembly handle (built from a device l2g tensor)."""

    def __init__(self, l2g, nglobal):
        _need(l2g, "l2g", l2g.numel(), "int32")
        h = ctypes.c_void_p()
        _check(lib().nir_assembly_create(_ptr(l2g), l2g.shape[0], l2g.shape[1], nglobal, ctypes.byref(h)))
        self.handle, self.nglobal, self.nlocal = h, nglobal, l2g.numel()

    def __del__(self):
        if getattr(self, "handle", None) is not None and _lib is not None:
            _lib.nir_assembly_destroy(self.handle)
            self.handle = None


def nir_assembly_create(l2g, nglobal):
    return Assembly(l2g, nglobal)


def nir_gather(a, dtype, xg, xl, stream=None):
    _need(xg, "xg", a.nglobal, dtype)
    _need(xl, "xl", a.nlocal, dtype)
    _check(lib().nir_gather(a.handle, dtype, _ptr(xg), _ptr(xl), _stream(stream)))


def nir_scatter_add(a, dtype, yl, yg, stream=None):
    _need(yl, "yl", a.nlocal, dtype)
    _need(yg, "yg", a.nglobal, dtype)
    _check(lib().nir_scatter_add(a.handle, dtype, _ptr(yl), _ptr(yg), _stream(stream)))


def nir_helmholtz_diagonal(b, basis, g, lam, dl, stream=None):
    ne, M, _, _ = _dims(b)
    _need(dl, "dl", ne * M, b.dtype)
    _need_geom(b, g, helm=True)
    _check(lib().nir_helmholtz_diagonal(ctypes.byref(b), _basis(basis), ctypes.byref(g), lam, _ptr(dl),
                                        _stream(stream)))


class CGPlan:
    """Owner of a nir_cg_plan handle; keeps the objects it points into alive."""

    def __init__(self, b64, basis, g64, helm32, assembly, lam):
        ne, _, _, ng = _dims(b64)
        _need_geom(b64, g64, helm=True, dt=F64)
        _need(helm32, "helm32", ne * 7 * ng, F32)
        h = ctypes.c_void_p()
        _check(lib().nir_cg_plan_create(ctypes.byref(b64), _basis(basis), ctypes.byref(g64), _ptr(helm32),
                                        assembly.handle, lam, ctypes.byref(h)))
        self.handle = h
        self._keep = (b64, basis, g64, helm32, assembly)

    def __del__(self):
        if getattr(self, "handle", None) is not None and _lib is not None:
            _lib.nir_cg_plan_destroy(self.handle)
            self.handle = None


def nir_cg_plan_create(b64, basis, g64, helm32, assembly, lam):
    return CGPlan(b64, basis, g64, helm32, assembly, lam)


def nir_cg_solve(plan, mode, b, x, rtol=1e-10, maxit=100000, inner_rtol=1e-4, stream=None, check=True):
    """Returns (status, nir_cg_info); raises on a non-OK status when check is True."""
    _need(b, "b", plan._keep[4].nglobal, F64)
    _need(x, "x", plan._keep[4].nglobal, F64)
    info = nir_cg_info()
    st = lib().nir_cg_solve(plan.handle, mode, _ptr(b), _ptr(x), rtol, maxit, inner_rtol, ctypes.byref(info),
                            _stream(stream))
    if check:
        _check(st)
    return st, info


class MixedPlan:
    """Owner of a nir_mixed_plan: batches (list of nir_batch), bases (list of Basis), geoms (list of
    nir_geom, helm used).  Keeps them alive with the plan."""

    def __init__(self, batches, bases, geoms):
        n = len(batches)
        for bb, gg in zip(batches, geoms):
            _need_geom(bb, gg, helm=True)
        self._b = (nir_batch * n)(*batches)
        self._h = (ctypes.c_void_p * n)(*[_basis(x).value if hasattr(_basis(x), "value") else _basis(x)
                                          for x in bases])
        self._g = (nir_geom * n)(*geoms)
        h = ctypes.c_void_p()
        _check(lib().nir_mixed_plan_create(n, ctypes.cast(self._b, _vp), ctypes.cast(self._h, _vp),
                                           ctypes.cast(self._g, _vp), ctypes.byref(h)))
        self.handle, self.n, self._keep = h, n, (batches, bases, geoms)

    def __del__(self):
        if getattr(self, "handle", None) is not None and _lib is not None:
            _lib.nir_mixed_plan_destroy(self.handle)
            self.handle = None

    def info(self):
        ni, g = ctypes.c_int32(), ctypes.c_int32()
        ms = ctypes.c_double()
        by, dof = ctypes.c_int64(), ctypes.c_int64()
        _check(lib().nir_mixed_plan_info(self.handle, ctypes.byref(ni), ctypes.byref(g), ctypes.byref(ms),
                                         ctypes.byref(by), ctypes.byref(dof)))
        st, mp, mb = ctypes.c_int32(), ctypes.c_double(), ctypes.c_double()
        _check(lib().nir_mixed_plan_timings(self.handle, ctypes.byref(st), ctypes.byref(mp), ctypes.byref(mb)))
        return dict(nitems=ni.value, grid=g.value, tuned_ms=ms.value, bytes=by.value, dof=dof.value,
                    strategy=st.value, ms_persistent=mp.value, ms_per_batch=mb.value)

    def set_strategy(self, strategy):
        _check(lib().nir_mixed_plan_set_strategy(self.handle, strategy))


def nir_mixed_plan_create(batches, bases, geoms):
    return MixedPlan(batches, bases, geoms)


def nir_mixed_helmholtz_apply(plan, lam, coef_in, coef_out, stream=None):
    n = plan.n
    for k, bb in enumerate(plan._keep[0]):
        ne, M, _, _ = _dims(bb)
        _need(coef_in[k], f"coef_in[{k}]", ne * M, bb.dtype)
        _need(coef_out[k], f"coef_out[{k}]", ne * M, bb.dtype)
    ins = (ctypes.c_void_p * n)(*[_ptr(x) for x in coef_in])
    outs = (ctypes.c_void_p * n)(*[_ptr(x) for x in coef_out])
    _check(lib().nir_mixed_helmholtz_apply(plan.handle, lam, ctypes.cast(ins, _vp), ctypes.cast(outs, _vp),
                                           _stream(stream)))


def nir_mixed_helmholtz_apply_noalloc(batches, bases, geoms, lam, coef_in, coef_out, stream=None):
    """One persistent mixed apply with no plan and no allocation (lists of nir_batch, Basis,
    nir_geom and coefficient tensors, one entry per batch)."""
    n = len(batches)
    if not (len(bases) == len(geoms) == len(coef_in) == len(coef_out) == n):
        raise NirError(1, "batches, bases, geoms, coef_in and coef_out differ in length")
    for k, bb in enumerate(batches):
        ne, M, _, _ = _dims(bb)
        _need_geom(bb, geoms[k], helm=True)
        _need(coef_in[k], f"coef_in[{k}]", ne * M, bb.dtype)
        _need(coef_out[k], f"coef_out[{k}]", ne * M, bb.dtype)
    b = (nir_batch * n)(*batches)
    h = (ctypes.c_void_p * n)(*[_basis(x).value if hasattr(_basis(x), "value") else _basis(x) for x in bases])
    g = (nir_geom * n)(*geoms)
    ins = (ctypes.c_void_p * n)(*[_ptr(x) for x in coef_in])
    outs = (ctypes.c_void_p * n)(*[_ptr(x) for x in coef_out])
    _check(lib().nir_mixed_helmholtz_apply_noalloc(n, ctypes.cast(b, _vp), ctypes.cast(h, _vp), ctypes.cast(g, _vp),
                                                   lam, ctypes.cast(ins, _vp), ctypes.cast(outs, _vp),
                                                   _stream(stream)))


def nir_autotune_helmholtz(b, basis, g, lam, coef_in, coef_out, reps=10, stream=None):
    """Returns (chosen variant, {variant: ms})."""
    ne, M, _, _ = _dims(b)
    _need(coef_in, "coef_in", ne * M, b.dtype)
    _need(coef_out, "coef_out", ne * M, b.dtype)
    _need_geom(b, g, helm=True)
    ch = ctypes.c_int32()
    ms = (ctypes.c_double * 11)(*([-1.0] * 11))
    _check(lib().nir_autotune_helmholtz(ctypes.byref(b), _basis(basis), ctypes.byref(g), lam, _ptr(coef_in),
                                        _ptr(coef_out), reps, ctypes.byref(ch), ctypes.cast(ms, _vp), _stream(stream)))
    return ch.value, {v + 1: ms[v] for v in range(11) if ms[v] >= 0}


def nir_autotune_save(path):
    _check(lib().nir_autotune_save(path.encode()))


def nir_autotune_load(path):
    _check(lib().nir_autotune_load(path.encode()))
