"""ctypes binding of libamgpoly.so.  Argument marshalling only."""
from __future__ import annotations

import ctypes
import os

LIB_PATH = os.path.join(os.path.dirname(os.path.abspath(__file__)), "libamgpoly.so")

AMG_OK, AMG_NOT_CONVERGED = 0, 1
AMG_EINVAL, AMG_ENOTSPD, AMG_ENOMEM, AMG_EHIP, AMG_EBREAKDOWN, AMG_ENAN, AMG_ECAPACITY = -1, -2, -3, -4, -5, -6, -7
AMG_L1JAC, AMG_CHEB4, AMG_OPTCHEB4, AMG_OPTCHEB1 = 0, 1, 2, 3
AMG_FP64, AMG_FP32 = 0, 1
AMG_AGG_BOX, AMG_AGG_MATCHING, AMG_AGG_VBM = 0, 1, 2
AMG_MAX_DEGREE = 12
AMG_HBM_PARTIALS = 16384
AMG_TRANSFER_RESIDUAL, AMG_TRANSFER_PRODUCT, AMG_TRANSFER_EXPLICIT = 0, 1, 2

__all__ = [
    "LIB_PATH", "AmgError", "lib", "amg_setup", "amg_destroy", "amg_num_levels", "amg_level_info", "amg_level_layout",
    "amg_level_transfer", "amg_level_patterns", "amg_level_rows_per_lane",
    "AMG_TRANSFER_RESIDUAL", "AMG_TRANSFER_PRODUCT", "AMG_TRANSFER_EXPLICIT",
    "amg_level_export", "amg_level_aggregates", "amg_default_beta", "amg_default_astar", "amg_set_beta",
    "amg_reset_beta",
    "amg_spmv", "smoother_apply", "smoother_apply_f32", "amg_restrict_residual", "amg_prolong_add", "amg_coarse_solve",
    "vcycle_apply", "pcg_solve", "pcg_solve_smoother", "amg_strerror", "amg_ckpt_bytes", "vcycle_fwd_ckpt", "vcycle_bwd",
    "amg_train_loss_grad", "amg_level_features", "mlp_num_params", "mlp_fwd", "mlp_bwd", "mlp_bwd_noalloc",
    "mlp_adam",
    "amg_beta_valid", "amg_learned_beta", "amg_learned_beta_grad", "amg_hbm_read", "amg_hbm_copy",
    "AMG_HBM_PARTIALS", "VCycleFunction",
    "AMG_OK", "AMG_NOT_CONVERGED", "AMG_EINVAL", "AMG_ENOTSPD", "AMG_ENOMEM", "AMG_EHIP",
    "AMG_EBREAKDOWN", "AMG_ENAN", "AMG_ECAPACITY", "AMG_L1JAC", "AMG_CHEB4", "AMG_OPTCHEB4",
    "AMG_OPTCHEB1", "AMG_FP64", "AMG_FP32", "AMG_MAX_DEGREE", "AMG_AGG_BOX", "AMG_AGG_MATCHING",
    "AMG_AGG_VBM",
]


class AmgOpts(ctypes.Structure):
    _fields_ = [("nx", ctypes.c_int32), ("ny", ctypes.c_int32), ("nz", ctypes.c_int32),
                ("nbatch", ctypes.c_int32), ("max_coarse", ctypes.c_int32), ("precision", ctypes.c_int32),
                ("agg_edge", ctypes.c_int32), ("smoothed", ctypes.c_int32), ("coarse_sweeps", ctypes.c_int32),
                ("aggregation", ctypes.c_int32), ("match_steps", ctypes.c_int32), ("vbm_theta", ctypes.c_double),
                ("drop_fine_csr", ctypes.c_int32)]


class AmgError(RuntimeError):
    def __init__(self, code: int, where: str):
        self.code = code
        super().__init__(f"{where}: {amg_strerror(code)} ({code})")


_lib = None
_P = ctypes.c_void_p
_I = ctypes.c_int
_I64 = ctypes.c_int64
_D = ctypes.c_double

_SIGS = {
    "amg_setup": (_I, [_I64, _I64, _P, _P, _P, ctypes.POINTER(AmgOpts), _P, ctypes.POINTER(_P)]),
    "amg_destroy": (_I, [_P]),
    "amg_num_levels": (_I, [_P, ctypes.POINTER(_I)]),
    "amg_level_info": (_I, [_P, _I, ctypes.POINTER(_I64), ctypes.POINTER(_I64)]),
    "amg_level_export": (_I, [_P, _I, _P, _P, _P, _P, _P]),
    "amg_level_aggregates": (_I, [_P, _I, _P, _P]),
    "amg_level_layout": (_I, [_P, _I, ctypes.POINTER(_I64), ctypes.POINTER(_I), ctypes.POINTER(_I)]),
    "amg_level_patterns": (_I, [_P, _I, _I, ctypes.POINTER(_I64), ctypes.POINTER(_I64), ctypes.POINTER(_I64)]),
    "amg_level_rows_per_lane": (_I, [_P, _I, ctypes.POINTER(_I)]),
    "amg_level_transfer": (_I, [_P, _I, ctypes.POINTER(_I), ctypes.POINTER(_I64)]),
    "amg_default_beta": (_I, [_I, ctypes.POINTER(_D)]),
    "amg_default_astar": (_I, [_I, ctypes.POINTER(_D)]),
    "amg_set_beta": (_I, [_P, _I, _I, ctypes.POINTER(_D)]),
    "amg_reset_beta": (_I, [_P]),
    "amg_spmv": (_I, [_P, _I, _P, _P, _P]),
    "smoother_apply": (_I, [_P, _I, _I, _I, _P, _P, _I, _P]),
    "smoother_apply_f32": (_I, [_P, _I, _I, _I, _P, _P, _I, _P]),
    "amg_restrict_residual": (_I, [_P, _I, _P, _P, _P, _P]),
    "amg_prolong_add": (_I, [_P, _I, _P, _P, _P]),
    "amg_coarse_solve": (_I, [_P, _P, _P, _P]),
    "vcycle_apply": (_I, [_P, _I, _I, _P, _P, _P]),
    "pcg_solve": (_I, [_P, _I, _I, _P, _P, _I, _D, _I, _I, ctypes.POINTER(_I), ctypes.POINTER(_D),
                       ctypes.POINTER(_D), _P]),
    "pcg_solve_smoother": (_I, [_P, _I, _I, _P, _P, _I, _D, _I, _I, ctypes.POINTER(_I), ctypes.POINTER(_D),
                                ctypes.POINTER(_D), _P]),
    "amg_strerror": (ctypes.c_char_p, [_I]),
    "amg_ckpt_bytes": (_I, [_P, ctypes.POINTER(_I64)]),
    "vcycle_fwd_ckpt": (_I, [_P, _I, _P, _P, _P, _P, _P]),
    "vcycle_bwd": (_I, [_P, _I, _P, _P, _P, _P, _P, _P]),
    "amg_train_loss_grad": (_I, [_P, _I, _P, _P, ctypes.POINTER(_D), _P, _P]),
    "amg_level_features": (_I, [_P, _I, ctypes.POINTER(_D), _P, _P]),
    "mlp_num_params": (_I, []),
    "mlp_fwd": (_I, [_P, _P, _I, _P, _P, _P]),
    "mlp_bwd": (_I, [_P, _P, _I, _P, _P, _P, _P, _P]),
    "mlp_bwd_noalloc": (_I, [_P, _P, _I, _P, _P, _P, _P]),
    "mlp_adam": (_I, [_P, _P, _P, _P, _I, _I, ctypes.c_float, ctypes.c_float, ctypes.c_float, ctypes.c_float, _P]),
    "amg_beta_valid": (_I, [_P, _I, _I, _I, _P, _P]),
    "amg_learned_beta": (_I, [_P, _I, _P, _I, _P, _P, _P]),
    "amg_learned_beta_grad": (_I, [_P, _I, _P, _P, _P, _P]),
    "amg_hbm_read": (_I, [_P, _I64, _P, _P]),
    "amg_hbm_copy": (_I, [_P, _P, _I64, _P]),
}


def lib():
    """Load libamgpoly.so (raises ImportError if it is not built: there is no fallback)."""
    global _lib
    if _lib is None:
        if not os.path.exists(LIB_PATH):
            raise ImportError(f"{LIB_PATH} is missing; build it with python -m paper_2407_09848_amd.build")
        L = ctypes.CDLL(LIB_PATH)
        for name, (res, args) in _SIGS.items():
            fn = getattr(L, name)
            fn.restype = res
            fn.argtypes = args
        _lib = L
    return _lib


def _stream():
    import torch
    return ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)


def _ptr(t, dtype=None, n=None, name="tensor"):
    import torch
    if t is None:
        return None
    if not isinstance(t, torch.Tensor) or not t.is_cuda:
        raise TypeError(f"{name} must be a device tensor")
    if not t.is_contiguous():
        raise ValueError(f"{name} must be contiguous")
    if dtype is not None and t.dtype != dtype:
        raise TypeError(f"{name} must be {dtype}, got {t.dtype}")
    if n is not None and t.numel() != n:
        raise ValueError(f"{name} has {t.numel()} entries, expected {n}")
    return ctypes.c_void_p(t.data_ptr())


def _check(rc, where, allow=(AMG_OK,)):
    if rc not in allow:
        raise AmgError(rc, where)
    return rc


def amg_strerror(code: int) -> str:
    return lib().amg_strerror(code).decode()


def amg_setup(row_ptr, col, val, nx, ny, nz, nbatch=1, max_coarse=4096, precision=AMG_FP64, agg_edge=2,
              smoothed=False, coarse_sweeps=0, aggregation=AMG_AGG_BOX, match_steps=3, vbm_theta=0.08,
              drop_fine_csr=False):
    """Build the hierarchy for the device CSR matrix (int32 row_ptr/col, float64 val); returns the handle."""
    import torch
    n = row_ptr.numel() - 1
    nnz = col.numel()
    o = AmgOpts(nx, ny, nz, nbatch, max_coarse, precision, agg_edge, int(bool(smoothed)), coarse_sweeps,
                aggregation, match_steps, float(vbm_theta), int(bool(drop_fine_csr)))
    h = ctypes.c_void_p()
    rc = lib().amg_setup(n, nnz, _ptr(row_ptr, torch.int32, name="row_ptr"), _ptr(col, torch.int32, name="col"),
                         _ptr(val, torch.float64, nnz, "val"), ctypes.byref(o), _stream(), ctypes.byref(h))
    _check(rc, "amg_setup")
    return h


def amg_destroy(h):
    return lib().amg_destroy(h)


def amg_num_levels(h) -> int:
    v = _I()
    _check(lib().amg_num_levels(h, ctypes.byref(v)), "amg_num_levels")
    return v.value


def amg_level_info(h, level):
    n, nnz = _I64(), _I64()
    _check(lib().amg_level_info(h, level, ctypes.byref(n), ctypes.byref(nnz)), "amg_level_info")
    return n.value, nnz.value


def amg_level_layout(h, level):
    """(stored entries including padding, lanes per row, offset-aligned) of level l's operator."""
    padded, lanes, aligned = _I64(), _I(), _I()
    _check(lib().amg_level_layout(h, level, ctypes.byref(padded), ctypes.byref(lanes), ctypes.byref(aligned)),
           "amg_level_layout")
    return padded.value, lanes.value, bool(aligned.value)


def amg_level_transfer(h, level):
    """(form, stored entries) of the restriction from level l (AMG_TRANSFER_*)."""
    form, stored = _I(), _I64()
    _check(lib().amg_level_transfer(h, level, ctypes.byref(form), ctypes.byref(stored)), "amg_level_transfer")
    return form.value, stored.value


def amg_level_patterns(h, level, restriction=False):
    """(entries stored one by one, slices kept as patterns, steps of all patterns) of level l's operator
    or of its restriction product."""
    values, slices, steps = _I64(), _I64(), _I64()
    _check(lib().amg_level_patterns(h, level, int(bool(restriction)), ctypes.byref(values), ctypes.byref(slices),
                                    ctypes.byref(steps)), "amg_level_patterns")
    return values.value, slices.value, steps.value


def amg_level_rows_per_lane(h, level):
    """Rows that a lane of the FP64 kernels serves on level l (1 or 2)."""
    rows = _I()
    _check(lib().amg_level_rows_per_lane(h, level, ctypes.byref(rows)), "amg_level_rows_per_lane")
    return rows.value


def amg_level_export(h, level):
    """(row_ptr, col, val, minv) of level l as new device tensors."""
    import torch
    n, nnz = amg_level_info(h, level)
    dev = torch.device("cuda")
    rp = torch.empty(n + 1, dtype=torch.int32, device=dev)
    cl = torch.empty(nnz, dtype=torch.int32, device=dev)
    vl = torch.empty(nnz, dtype=torch.float64, device=dev)
    mi = torch.empty(n, dtype=torch.float64, device=dev)
    _check(lib().amg_level_export(h, level, _ptr(rp), _ptr(cl), _ptr(vl), _ptr(mi), _stream()), "amg_level_export")
    return rp, cl, vl, mi


def amg_level_aggregates(h, level):
    """Aggregate index (int32, on the device) of every row of level l, l below the coarsest."""
    import torch
    n, _ = amg_level_info(h, level)
    agg = torch.empty(n, dtype=torch.int32, device="cuda")
    _check(lib().amg_level_aggregates(h, level, _ptr(agg), _stream()), "amg_level_aggregates")
    return agg


def amg_default_beta(degree):
    buf = (_D * max(degree, 1))()
    _check(lib().amg_default_beta(degree, buf), "amg_default_beta")
    return [buf[i] for i in range(degree)]


def amg_default_astar(degree):
    v = _D()
    _check(lib().amg_default_astar(degree, ctypes.byref(v)), "amg_default_astar")
    return v.value


def amg_set_beta(h, degree, level, beta):
    buf = (_D * len(beta))(*[float(b) for b in beta])
    if len(beta) != degree:
        raise ValueError("beta must have `degree` entries")
    return _check(lib().amg_set_beta(h, degree, level, buf), "amg_set_beta")


def amg_reset_beta(h):
    return _check(lib().amg_reset_beta(h), "amg_reset_beta")


def amg_spmv(h, level, x, y):
    import torch
    n, _ = amg_level_info(h, level)
    return _check(lib().amg_spmv(h, level, _ptr(x, torch.float64, n, "x"), _ptr(y, torch.float64, n, "y"),
                                 _stream()), "amg_spmv")


def smoother_apply(h, level, kind, degree, b, x, x_is_zero=False):
    import torch
    n, _ = amg_level_info(h, level)
    return _check(lib().smoother_apply(h, level, kind, degree, _ptr(b, torch.float64, n, "b"),
                                       _ptr(x, torch.float64, n, "x"), int(bool(x_is_zero)), _stream()),
                  "smoother_apply")


def smoother_apply_f32(h, level, kind, degree, b, x, x_is_zero=False):
    """The FP32 hierarchy's smoother on float32 device vectors (an AMG_FP32 handle)."""
    import torch
    n, _ = amg_level_info(h, level)
    return _check(lib().smoother_apply_f32(h, level, kind, degree, _ptr(b, torch.float32, n, "b"),
                                           _ptr(x, torch.float32, n, "x"), int(bool(x_is_zero)), _stream()),
                  "smoother_apply_f32")


def amg_restrict_residual(h, level, b, x, bc):
    import torch
    n, _ = amg_level_info(h, level)
    nc, _ = amg_level_info(h, level + 1)
    return _check(lib().amg_restrict_residual(h, level, _ptr(b, torch.float64, n, "b"), _ptr(x, torch.float64, n, "x"),
                                              _ptr(bc, torch.float64, nc, "bc"), _stream()), "amg_restrict_residual")


def amg_prolong_add(h, level, xc, x):
    import torch
    n, _ = amg_level_info(h, level)
    nc, _ = amg_level_info(h, level + 1)
    return _check(lib().amg_prolong_add(h, level, _ptr(xc, torch.float64, nc, "xc"), _ptr(x, torch.float64, n, "x"),
                                        _stream()), "amg_prolong_add")


def amg_coarse_solve(h, b, x):
    import torch
    L = amg_num_levels(h) - 1
    n, _ = amg_level_info(h, L)
    return _check(lib().amg_coarse_solve(h, _ptr(b, torch.float64, n, "b"), _ptr(x, torch.float64, n, "x"),
                                         _stream()), "amg_coarse_solve")


def vcycle_apply(h, kind, degree, r, z):
    import torch
    n, _ = amg_level_info(h, 0)
    return _check(lib().vcycle_apply(h, kind, degree, _ptr(r, torch.float64, n, "r"), _ptr(z, torch.float64, n, "z"),
                                     _stream()), "vcycle_apply")


def _pcg(name, h, kind, degree, b, x, x_is_zero, rtol, maxit, flexible, history):
    import torch
    n, _ = amg_level_info(h, 0)
    it, rel = _I(), _D()
    hist = (_D * (maxit + 1))() if history else None
    rc = getattr(lib(), name)(h, kind, degree, _ptr(b, torch.float64, n, "b"), _ptr(x, torch.float64, n, "x"),
                              int(bool(x_is_zero)), float(rtol), int(maxit), int(bool(flexible)), ctypes.byref(it),
                              ctypes.byref(rel), hist, _stream())
    _check(rc, name, allow=(AMG_OK, AMG_NOT_CONVERGED))
    return rc, it.value, rel.value, ([hist[i] for i in range(it.value + 1)] if history else None)


def pcg_solve(h, kind, degree, b, x, x_is_zero=True, rtol=1e-8, maxit=1000, flexible=False, history=False):
    """V-cycle-preconditioned CG.  Returns (rc, iters, relres, hist list or None); rc is AMG_OK or
    AMG_NOT_CONVERGED (errors raise)."""
    return _pcg("pcg_solve", h, kind, degree, b, x, x_is_zero, rtol, maxit, flexible, history)


def pcg_solve_smoother(h, kind, degree, b, x, x_is_zero=True, rtol=1e-8, maxit=1000, flexible=False,
                       history=False):
    """CG preconditioned by the level-0 polynomial smoother alone; same returns as pcg_solve."""
    return _pcg("pcg_solve_smoother", h, kind, degree, b, x, x_is_zero, rtol, maxit, flexible, history)


# ---------------------------------------------------------------------------
# differentiable V-cycle and learned weights
# ---------------------------------------------------------------------------
def amg_ckpt_bytes(h) -> int:
    v = _I64()
    _check(lib().amg_ckpt_bytes(h, ctypes.byref(v)), "amg_ckpt_bytes")
    return v.value


def vcycle_fwd_ckpt(h, degree, beta, r, z, ckpt):
    """z = B(beta) r saving checkpoints; beta: float64 device [nbatch * nlevels * degree]."""
    import torch
    n, _ = amg_level_info(h, 0)
    return _check(lib().vcycle_fwd_ckpt(h, degree, _ptr(beta, torch.float64, name="beta"),
                                        _ptr(r, torch.float64, n, "r"), _ptr(z, torch.float64, n, "z"),
                                        _ptr(ckpt, name="ckpt"), _stream()), "vcycle_fwd_ckpt")


def vcycle_bwd(h, degree, beta, ckpt, gz, gr, gbeta):
    import torch
    n, _ = amg_level_info(h, 0)
    return _check(lib().vcycle_bwd(h, degree, _ptr(beta, torch.float64, name="beta"), _ptr(ckpt, name="ckpt"),
                                   _ptr(gz, torch.float64, n, "gz"), _ptr(gr, torch.float64, n, "gr"),
                                   _ptr(gbeta, torch.float64, beta.numel(), "gbeta"), _stream()), "vcycle_bwd")


def amg_train_loss_grad(h, degree, beta, b, gbeta, nbatch):
    """Returns (loss, per-problem ratios); gbeta (device float64, layout of beta) is overwritten."""
    import torch
    n, _ = amg_level_info(h, 0)
    out = (_D * (nbatch + 1))()
    _check(lib().amg_train_loss_grad(h, degree, _ptr(beta, torch.float64, name="beta"), _ptr(b, torch.float64, n, "b"),
                                     out, _ptr(gbeta, torch.float64, beta.numel(), "gbeta"), _stream()),
           "amg_train_loss_grad")
    return out[0], [out[1 + p] for p in range(nbatch)]


def amg_level_features(h, degree, sigma):
    """float32 device tensor [nbatch * (nlevels - 1), 8] of per-level features."""
    import torch
    L = amg_num_levels(h)
    sig = (_D * len(sigma))(*[float(s) for s in sigma])
    feat = torch.empty((len(sigma) * (L - 1), 8), dtype=torch.float32, device="cuda")
    _check(lib().amg_level_features(h, degree, sig, _ptr(feat), _stream()), "amg_level_features")
    return feat


def mlp_num_params() -> int:
    return lib().mlp_num_params()


def mlp_fwd(params, x, y, cache):
    import torch
    B = x.shape[0]
    return _check(lib().mlp_fwd(_ptr(params, torch.float32), _ptr(x, torch.float32), B, _ptr(y, torch.float32),
                                _ptr(cache, torch.float32), _stream()), "mlp_fwd")


def mlp_bwd(params, x, cache, gy, gparams, work):
    import torch
    B = x.shape[0]
    return _check(lib().mlp_bwd(_ptr(params, torch.float32), _ptr(x, torch.float32), B, _ptr(cache, torch.float32),
                                _ptr(gy, torch.float32), _ptr(gparams, torch.float32), _ptr(work, torch.float32),
                                _stream()), "mlp_bwd")


def mlp_bwd_noalloc(params, x, cache, gy, gparams):
    """mlp_bwd with the library's own static scratch (no workspace argument, batch <= 256)."""
    import torch
    B = x.shape[0]
    return _check(lib().mlp_bwd_noalloc(_ptr(params, torch.float32), _ptr(x, torch.float32), B,
                                        _ptr(cache, torch.float32), _ptr(gy, torch.float32),
                                        _ptr(gparams, torch.float32), _stream()), "mlp_bwd_noalloc")


def mlp_adam(params, g, m, v, step, lr=1e-3, b1=0.9, b2=0.999, eps=1e-8):
    import torch
    n = params.numel()
    return _check(lib().mlp_adam(_ptr(params, torch.float32, n), _ptr(g, torch.float32, n), _ptr(m, torch.float32, n),
                                 _ptr(v, torch.float32, n), n, int(step), lr, b1, b2, eps, _stream()), "mlp_adam")


def amg_beta_valid(beta, degree, ngrid=4096):
    """int32 device tensor: 1 where row q of beta ([count, degree] float64) keeps |p| < 1 on (0, 1]."""
    import torch
    count = beta.numel() // degree
    valid = torch.empty(count, dtype=torch.int32, device="cuda")
    _check(lib().amg_beta_valid(_ptr(beta, torch.float64), count, degree, ngrid, _ptr(valid), _stream()),
           "amg_beta_valid")
    return valid


def amg_learned_beta(h, degree, y, nbatch, ngrid=4096):
    """(beta float64 [nbatch, nlevels, degree], valid int32 [nbatch * (nlevels - 1)]) on the device:
    the optimal table plus the network output y ([nbatch * (nlevels - 1), 6] float32) on the
    smoothing levels, rows outside Pi_k falling back to the table.  y = None: the plain table."""
    import torch
    L = amg_num_levels(h)
    beta = torch.empty((nbatch, L, degree), dtype=torch.float64, device="cuda")
    valid = torch.empty(nbatch * (L - 1), dtype=torch.int32, device="cuda")
    yp = None if y is None else _ptr(y, torch.float32, nbatch * (L - 1) * 6, "y")
    _check(lib().amg_learned_beta(h, degree, yp, ngrid, _ptr(beta), _ptr(valid), _stream()), "amg_learned_beta")
    return beta, valid


def amg_learned_beta_grad(h, degree, gbeta, valid, gy):
    """gy ([nbatch * (nlevels - 1), 6] float32) = dL/dbeta on the kept rows, 0 elsewhere."""
    import torch
    _check(lib().amg_learned_beta_grad(h, degree, _ptr(gbeta, torch.float64, name="gbeta"),
                                       _ptr(valid, torch.int32, name="valid"),
                                       _ptr(gy, torch.float32, valid.numel() * 6, "gy"), _stream()),
           "amg_learned_beta_grad")


def amg_hbm_read(x, partial):
    """Reads x (float64) once; partial (float64, AMG_HBM_PARTIALS entries) receives block sums."""
    import torch
    return _check(lib().amg_hbm_read(_ptr(x, torch.float64, name="x"), x.numel(),
                                     _ptr(partial, torch.float64, AMG_HBM_PARTIALS, "partial"), _stream()),
                  "amg_hbm_read")


def amg_hbm_copy(x, y):
    """y = x (float64, same length, not overlapping)."""
    import torch
    return _check(lib().amg_hbm_copy(_ptr(x, torch.float64, name="x"), _ptr(y, torch.float64, x.numel(), "y"),
                                     x.numel(), _stream()), "amg_hbm_copy")


def _vcycle_function():
    import torch

    class VCycleFunction(torch.autograd.Function):
        """z = B(beta) r as an autograd function: forward runs vcycle_fwd_ckpt (checkpoints kept
        on the context), backward runs the hand-written adjoint vcycle_bwd."""

        @staticmethod
        def forward(ctx, beta, r, handle, degree):
            ck = torch.empty(amg_ckpt_bytes(handle), dtype=torch.uint8, device="cuda")
            z = torch.empty_like(r)
            vcycle_fwd_ckpt(handle, degree, beta.contiguous(), r.contiguous(), z, ck)
            ctx.save_for_backward(beta)
            ctx.ck = ck
            ctx.handle, ctx.degree = handle, degree
            return z

        @staticmethod
        def backward(ctx, gz):
            (beta,) = ctx.saved_tensors
            gbeta = torch.zeros_like(beta)
            gr = torch.empty_like(gz)
            vcycle_bwd(ctx.handle, ctx.degree, beta.contiguous(), ctx.ck, gz.contiguous(), gr, gbeta)
            ctx.ck = None
            return gbeta, gr, None, None

    return VCycleFunction


class _LazyVCycle:
    _cls = None

    def apply(self, *args):
        if _LazyVCycle._cls is None:
            _LazyVCycle._cls = _vcycle_function()
        return _LazyVCycle._cls.apply(*args)


VCycleFunction = _LazyVCycle()
