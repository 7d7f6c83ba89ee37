"""Python binding of libndgp.so (the C ABI of include/ndgp.h).

Argument marshalling only: torch supplies device memory and the stream, every
step of the solve runs in the library's HIP kernels.  There is no CPU path: if
the library is not built, or no GPU is present, the calls raise.

Units: lengths in c/H0 (``cell_size`` converts from Mpc/h), phi in c^2.
Arrays: float64, natural layout [z][y][x]; patch solutions are padded with a
one-cell ghost shell, shape (m+2, m+2, m+2).
"""
from __future__ import annotations

import contextlib
import ctypes
import math
import dataclasses
import os
from typing import Optional, Sequence

import torch

HERE = os.path.dirname(os.path.abspath(__file__))
LIB_PATH = os.path.join(HERE, "libndgp.so")
C_OVER_H0_MPC_H = 2997.92458  # c / H0 in Mpc/h

NDGP_OK, NDGP_EINVAL, NDGP_ENOMEM, NDGP_ENOCONV, NDGP_EDEVICE = 0, -1, -2, -3, -4
MODE_FULL, MODE_INTERPOLATED, MODE_TRUNCATED = 0, 1, 2
PREC_FP64, PREC_MIXED = 0, 1
WARM_START = 1
PROFILE = 2
TWO_PASS = 4
DAMPED = 8
MAX_PATCHES = 4
ABI_VERSION = 3
HIST_LEN = 64

_STATUS = {NDGP_EINVAL: "EINVAL", NDGP_ENOMEM: "ENOMEM", NDGP_ENOCONV: "ENOCONV",
           NDGP_EDEVICE: "EDEVICE"}


class NdgpError(RuntimeError):
    def __init__(self, status: int, msg: str):
        super().__init__(f"ndgp {_STATUS.get(status, status)}: {msg}")
        self.status = status


class _Grid(ctypes.Structure):
    _fields_ = [("n", ctypes.c_int32), ("h", ctypes.c_double), ("n_patch", ctypes.c_int32),
                ("patch_n", ctypes.c_int32 * MAX_PATCHES),
                ("patch_origin", (ctypes.c_int32 * 3) * MAX_PATCHES)]


class _Params(ctypes.Structure):
    _fields_ = [("rc", ctypes.c_double), ("beta", ctypes.c_double), ("a", ctypes.c_double),
                ("omega_m", ctypes.c_double), ("tol", ctypes.c_double),
                ("max_cycles", ctypes.c_int32), ("nu1", ctypes.c_int32), ("nu2", ctypes.c_int32),
                ("n_levels", ctypes.c_int32), ("mode", ctypes.c_int32),
                ("precision", ctypes.c_int32), ("flags", ctypes.c_uint32),
                ("trunc_level", ctypes.c_int32)]


class _Report(ctypes.Structure):
    _fields_ = [("cycles", ctypes.c_int32 * (1 + MAX_PATCHES)),
                ("rel_res", ctypes.c_double * (1 + MAX_PATCHES)),
                ("removed_mean", ctypes.c_double), ("phi_mean", ctypes.c_double),
                ("fallbacks", ctypes.c_int32), ("hist_len", ctypes.c_int32),
                ("res_hist", ctypes.c_double * HIST_LEN), ("t_total_ms", ctypes.c_double),
                ("t_smooth_ms", ctypes.c_double), ("smooth_launches", ctypes.c_int32),
                ("smooth_cells_per_launch", ctypes.c_int32),
                ("damped_from", ctypes.c_int32 * (1 + MAX_PATCHES)),
                ("iterated_fraction", ctypes.c_double * (1 + MAX_PATCHES)),
                ("holds", ctypes.c_int32)]


class _GeffLevel(ctypes.Structure):
    _fields_ = [("cells", ctypes.c_int64), ("sum", ctypes.c_double), ("sum_sq", ctypes.c_double),
                ("min", ctypes.c_double), ("max", ctypes.c_double)]


GEFF_MAX_EDGES = 255
GEFF_WORKSPACE = 262144

_lib = None


def lib():
    """Load libndgp.so (raises if it has not been built)."""
    global _lib
    if _lib is None:
        if not os.path.exists(LIB_PATH):
            raise RuntimeError(f"{LIB_PATH} is not built: run python -m paper_1511_08200_amd.build")
        L = ctypes.CDLL(LIB_PATH)
        vp = ctypes.c_void_p
        L.ndgp_version.restype = ctypes.c_int32
        if L.ndgp_version() != ABI_VERSION:
            raise RuntimeError(f"{LIB_PATH} has ABI version {L.ndgp_version()}, this binding "
                               f"needs {ABI_VERSION}: rebuild it")
        L.ndgp_last_error.restype = ctypes.c_char_p
        L.ndgp_beta_lcdm.restype = ctypes.c_double
        L.ndgp_beta_lcdm.argtypes = [ctypes.c_double] * 3
        d = ctypes.c_double
        L.ndgp_nfw_r200.restype = d
        L.ndgp_nfw_r200.argtypes = [d, d]
        L.ndgp_nfw_force_ratio.restype = d
        L.ndgp_nfw_force_ratio.argtypes = [d] * 6
        L.ndgp_nfw_screening_radius.restype = d
        L.ndgp_nfw_screening_radius.argtypes = [d] * 6
        L.ndgp_nfw_trunc_level.restype = ctypes.c_int32
        L.ndgp_nfw_trunc_level.argtypes = [d] * 7
        L.ndgp_workspace_bytes.restype = ctypes.c_size_t
        L.ndgp_workspace_bytes.argtypes = [ctypes.POINTER(_Grid), ctypes.POINTER(_Params)]
        arr3 = vp * (1 + MAX_PATCHES)
        L.ndgp_solve.restype = ctypes.c_int
        L.ndgp_solve.argtypes = [ctypes.POINTER(_Grid), ctypes.POINTER(_Params), arr3, arr3, vp,
                                 ctypes.c_size_t, vp, ctypes.POINTER(_Report)]
        L.ndgp_solve_cellwise.restype = ctypes.c_int
        L.ndgp_solve_cellwise.argtypes = [ctypes.POINTER(_Grid), ctypes.POINTER(_Params), arr3,
                                          arr3, ctypes.c_double, arr3, vp, ctypes.c_size_t, vp,
                                          ctypes.POINTER(_Report)]
        L.ndgp_cic_workspace_bytes.restype = ctypes.c_size_t
        L.ndgp_cic_workspace_bytes.argtypes = [ctypes.POINTER(_Grid)]
        L.ndgp_cic_density_workspace_bytes.restype = ctypes.c_size_t
        L.ndgp_cic_density_workspace_bytes.argtypes = [ctypes.POINTER(_Grid), ctypes.c_int64]
        L.ndgp_cic_density.restype = ctypes.c_int
        L.ndgp_cic_density.argtypes = [ctypes.POINTER(_Grid), vp, ctypes.c_int64, arr3, vp,
                                       ctypes.c_size_t, vp]
        L.ndgp_cic_force.restype = ctypes.c_int
        L.ndgp_cic_force.argtypes = [ctypes.POINTER(_Grid), arr3, vp, ctypes.c_int64, vp, vp]
        L.ndgp_cic_force_workspace_bytes.restype = ctypes.c_size_t
        L.ndgp_cic_force_workspace_bytes.argtypes = [ctypes.POINTER(_Grid), ctypes.c_int64]
        L.ndgp_cic_force_in.restype = ctypes.c_int
        L.ndgp_cic_force_in.argtypes = [ctypes.POINTER(_Grid), arr3, vp, ctypes.c_int64, vp, vp,
                                        ctypes.c_size_t, vp]
        L.ndgp_refine_flags.restype = ctypes.c_int
        L.ndgp_refine_flags.argtypes = [ctypes.POINTER(_Grid), arr3, ctypes.c_int64,
                                        ctypes.c_double, arr3, ctypes.POINTER(ctypes.c_int64),
                                        vp, ctypes.c_size_t, vp]
        L.ndgp_total_force.restype = ctypes.c_int
        L.ndgp_total_force.argtypes = [ctypes.POINTER(_Grid), arr3, arr3, arr3, vp]
        L.ndgp_geff_stats.restype = ctypes.c_int
        L.ndgp_geff_stats.argtypes = [ctypes.POINTER(_Grid), arr3, arr3,
                                      ctypes.POINTER(ctypes.c_double), ctypes.c_int32,
                                      ctypes.POINTER(_GeffLevel),
                                      ctypes.POINTER(ctypes.c_int64), vp, ctypes.c_size_t, vp]
        L.ndgp_residual.restype = ctypes.c_int
        L.ndgp_residual.argtypes = [ctypes.POINTER(_Grid), ctypes.POINTER(_Params), ctypes.c_int32,
                                    arr3, vp, vp, ctypes.POINTER(ctypes.c_double), vp,
                                    ctypes.c_size_t, vp]
        L.ndgp_refine_boxes.restype = ctypes.c_int
        L.ndgp_refine_boxes.argtypes = [vp, ctypes.c_int32, ctypes.c_int32, ctypes.c_int32,
                                        ctypes.c_int32, ctypes.c_double, ctypes.c_int32, vp,
                                        ctypes.c_int32, ctypes.POINTER(ctypes.c_int32), vp]
        L.ndgp_amr_workspace_bytes.restype = ctypes.c_size_t
        L.ndgp_amr_workspace_bytes.argtypes = [ctypes.POINTER(_Grid), ctypes.POINTER(_Params),
                                               vp, ctypes.c_int32]
        L.ndgp_solve_amr.restype = ctypes.c_int
        L.ndgp_solve_amr.argtypes = [ctypes.POINTER(_Grid), ctypes.POINTER(_Params), vp,
                                     ctypes.c_int32, vp, vp, vp, ctypes.c_size_t, vp,
                                     ctypes.POINTER(_Report), vp]
        L.ndgp_residual_noalloc.restype = ctypes.c_int
        L.ndgp_residual_noalloc.argtypes = [ctypes.POINTER(_Grid), ctypes.POINTER(_Params),
                                            ctypes.c_int32, arr3, vp, vp, vp, vp]
        L.ndgp_force.restype = ctypes.c_int
        L.ndgp_force.argtypes = [ctypes.POINTER(_Grid), arr3, arr3, vp]
        L.ndgp_plan_create.restype = ctypes.c_int
        L.ndgp_plan_create.argtypes = [ctypes.POINTER(_Grid), ctypes.POINTER(_Params), arr3, arr3,
                                       vp, ctypes.c_size_t, vp, ctypes.POINTER(vp)]
        L.ndgp_plan_poll.restype = ctypes.c_int
        L.ndgp_plan_poll.argtypes = [vp, ctypes.POINTER(ctypes.c_int32), ctypes.POINTER(_Report)]
        L.ndgp_plan_step.restype = ctypes.c_int
        L.ndgp_plan_step.argtypes = [vp]
        L.ndgp_plan_destroy.restype = None
        L.ndgp_plan_destroy.argtypes = [vp]
        L.ndgp_diff_norms.restype = ctypes.c_int
        L.ndgp_diff_norms.argtypes = [vp, vp, ctypes.c_size_t, ctypes.POINTER(ctypes.c_double),
                                      vp, ctypes.c_size_t, vp]
        _lib = L
    return _lib


def _check(status: int):
    if status != NDGP_OK:
        raise NdgpError(status, lib().ndgp_last_error().decode())


# --------------------------------------------------------------------------
# parameters

def cell_size(box_mpc_h: float, n: int) -> float:
    """Cell size in c/H0 of n cells across a box of box_mpc_h Mpc/h."""
    return box_mpc_h / n / C_OVER_H0_MPC_H


def beta_lcdm(a: float, omega_m: float, rc: float) -> float:
    """beta(a) of Eq. (beta) for an LCDM expansion history (library routine)."""
    return float(lib().ndgp_beta_lcdm(a, omega_m, rc))


def _finite_or_raise(v: float) -> float:
    if math.isnan(v):
        raise ValueError(lib().ndgp_last_error().decode())
    return float(v)


def nfw_r200(m200: float, e_z: float = 1.0) -> float:
    """R_200 in Mpc/h of a halo of M_200 M_sun/h (Eq. r200)."""
    return _finite_or_raise(lib().ndgp_nfw_r200(m200, e_z))


def nfw_force_ratio(r: float, m200: float, c200: float, rc: float, beta: float,
                    e_z: float = 1.0) -> float:
    """G_eff - 1 = F_5th / F_GR at radius r (Mpc/h) of an NFW halo."""
    return _finite_or_raise(lib().ndgp_nfw_force_ratio(r, m200, c200, rc, beta, e_z))


def nfw_screening_radius(fraction: float, m200: float, c200: float, rc: float, beta: float,
                         e_z: float = 1.0) -> float:
    """r_t (Mpc/h): where G_eff - 1 has fallen to ``fraction``."""
    return _finite_or_raise(lib().ndgp_nfw_screening_radius(fraction, m200, c200, rc, beta, e_z))


def nfw_trunc_level(h_domain: float, fraction: float, m200: float, c200: float, rc: float,
                    beta: float, e_z: float = 1.0) -> int:
    """First truncated refinement level (Params.trunc_level) for a halo whose
    fifth force must be below ``fraction`` of gravity wherever it is truncated."""
    k = int(lib().ndgp_nfw_trunc_level(h_domain, fraction, m200, c200, rc, beta, e_z))
    if k < 0:
        raise ValueError(lib().ndgp_last_error().decode())
    return k


@dataclasses.dataclass
class Patch:
    n: int                 # cells per side
    origin: tuple          # lower corner (x, y, z) in parent cells


@dataclasses.dataclass
class Grid:
    n: int
    h: float
    patches: list = dataclasses.field(default_factory=list)

    def _c(self) -> _Grid:
        if len(self.patches) > MAX_PATCHES:
            raise ValueError(f"at most {MAX_PATCHES} nested patches")
        g = _Grid()
        g.n, g.h, g.n_patch = self.n, self.h, len(self.patches)
        for q, p in enumerate(self.patches):
            g.patch_n[q] = p.n
            for a in range(3):
                g.patch_origin[q][a] = int(p.origin[a])
        return g

    def level_n(self, level: int) -> int:
        return self.n if level == 0 else self.patches[level - 1].n

    def level_h(self, level: int) -> float:
        return self.h / (1 << level)


@dataclasses.dataclass
class Params:
    rc: float = 1.0
    beta: Optional[float] = None  # None: beta_lcdm(a, omega_m, rc)
    a: float = 1.0
    omega_m: float = 0.3
    tol: float = 1e-10
    max_cycles: int = 50
    nu1: int = 2
    nu2: int = 2
    n_levels: int = 0
    mode: int = MODE_FULL
    trunc_level: int = 0  # MODE_TRUNCATED: first interpolated refinement level
    precision: int = PREC_FP64
    warm_start: bool = False
    profile: bool = False
    two_pass: bool = False
    damped: bool = False

    def _c(self) -> _Params:
        p = _Params()
        p.rc, p.a, p.omega_m, p.tol = self.rc, self.a, self.omega_m, self.tol
        p.beta = self.beta if self.beta is not None else beta_lcdm(self.a, self.omega_m, self.rc)
        p.max_cycles, p.nu1, p.nu2, p.n_levels = self.max_cycles, self.nu1, self.nu2, self.n_levels
        p.mode, p.precision, p.trunc_level = self.mode, self.precision, self.trunc_level
        p.flags = ((WARM_START if self.warm_start else 0) | (PROFILE if self.profile else 0)
                   | (TWO_PASS if self.two_pass else 0) | (DAMPED if self.damped else 0))
        return p


@dataclasses.dataclass
class Report:
    cycles: list
    rel_res: list
    removed_mean: float
    phi_mean: float
    fallbacks: int
    history: list
    t_total_ms: float
    t_smooth_ms: float = 0.0
    smooth_launches: int = 0
    smooth_cells_per_launch: int = 0
    status: int = NDGP_OK
    damped_from: list = dataclasses.field(default_factory=list)
    iterated_fraction: list = dataclasses.field(default_factory=list)
    holds: int = 0


def _report(r: _Report, status: int) -> Report:
    return Report(cycles=list(r.cycles), rel_res=list(r.rel_res), removed_mean=r.removed_mean,
                  phi_mean=r.phi_mean, fallbacks=r.fallbacks,
                  history=[r.res_hist[i] for i in range(r.hist_len)], t_total_ms=r.t_total_ms,
                  t_smooth_ms=r.t_smooth_ms, smooth_launches=r.smooth_launches,
                  smooth_cells_per_launch=r.smooth_cells_per_launch, status=status,
                  damped_from=list(r.damped_from),
                  iterated_fraction=list(r.iterated_fraction), holds=r.holds)


# --------------------------------------------------------------------------
# device buffers

def _dev(t: torch.Tensor, shape=None, name="array") -> int:
    if not isinstance(t, torch.Tensor) or t.dtype != torch.float64 or not t.is_cuda:
        raise TypeError(f"{name} must be a float64 CUDA/HIP tensor")
    if not t.is_contiguous():
        raise ValueError(f"{name} must be contiguous")
    if shape is not None and tuple(t.shape) != tuple(shape):
        raise ValueError(f"{name} has shape {tuple(t.shape)}, expected {tuple(shape)}")
    return t.data_ptr()


def _stream(stream) -> int:
    s = stream if stream is not None else torch.cuda.current_stream()
    return s.cuda_stream


_ws_cache: dict = {}


def workspace_bytes(grid: Grid, params: Params) -> int:
    g, p = grid._c(), params._c()
    nb = lib().ndgp_workspace_bytes(ctypes.byref(g), ctypes.byref(p))
    if nb == 0:
        raise NdgpError(NDGP_EINVAL, lib().ndgp_last_error().decode())
    return int(nb)


def workspace(nbytes: int, device=None, stream=None) -> torch.Tensor:
    """A cached uint8 workspace of at least nbytes for work enqueued on
    `stream` (default: the device's current stream).  One cache entry per
    device and stream, allocated on that stream: calls that enqueue on
    different streams never share a workspace, and a replaced (smaller) one
    is only reused by the allocator after the work queued before it on its
    stream."""
    dev = torch.device(device if device is not None else "cuda")
    idx = dev.index if dev.index is not None else torch.cuda.current_device()
    s = stream if stream is not None else torch.cuda.current_stream(idx)
    key = (dev.type, idx, s.cuda_stream)
    ws = _ws_cache.get(key)
    if ws is None or ws.numel() < nbytes:
        with torch.cuda.stream(s):
            ws = torch.empty(nbytes, dtype=torch.uint8, device=dev)
        _ws_cache[key] = ws
    return ws


def _scratch(nbytes: int, device, stream):
    """Scratch that one call may use: its own buffer, from the allocator's pool of
    the stream the call enqueues on, so that it goes back when the call returns and
    is handed out again only to work behind it (a captured call keeps it with its
    graph).  None for no bytes, or where there is no room."""
    if nbytes == 0:
        return None
    try:
        with torch.cuda.stream(stream) if stream is not None else contextlib.nullcontext():
            return torch.empty(nbytes, dtype=torch.uint8, device=device)
    except torch.OutOfMemoryError:
        return None


def _arr3(ptrs):
    a = (ctypes.c_void_p * (1 + MAX_PATCHES))()
    for i, p in enumerate(ptrs):
        a[i] = p
    return a


def alloc_phi(grid: Grid, device="cuda") -> list:
    out = [torch.zeros((grid.n,) * 3, dtype=torch.float64, device=device)]
    for p in grid.patches:
        out.append(torch.zeros((p.n + 2,) * 3, dtype=torch.float64, device=device))
    return out


def _solve_ptrs(grid: Grid, delta, phi):
    """Device pointers of delta (None where absent) and phi per level."""
    dptr = [_dev(delta[0], (grid.n,) * 3, "delta[0]")]
    pptr = [_dev(phi[0], (grid.n,) * 3, "phi[0]")]
    for q, pt in enumerate(grid.patches):
        d = delta[q + 1] if q + 1 < len(delta) else None
        dptr.append(_dev(d, (pt.n,) * 3, f"delta[{q + 1}]") if d is not None else None)
        pptr.append(_dev(phi[q + 1], (pt.n + 2,) * 3, f"phi[{q + 1}]"))
    return dptr, pptr


def _finish(st: int, rep: _Report, check: bool) -> Report:
    if check or (st != NDGP_OK and st != NDGP_ENOCONV):
        _check(st)
    return _report(rep, st)


def solve(grid: Grid, params: Params, delta: Sequence[torch.Tensor], phi=None, ws=None,
          stream=None, check: bool = True):
    """Run ndgp_solve.  ``delta``: [domain (n^3), patch1 (m^3), ...] device
    float64; returns (phi list, Report).  With check=False a non-OK status is
    reported in Report.status instead of raised."""
    g, p = grid._c(), params._c()
    if phi is None:
        phi = alloc_phi(grid, device=delta[0].device)
    dptr, pptr = _solve_ptrs(grid, delta, phi)
    if ws is None:
        ws = workspace(workspace_bytes(grid, params), delta[0].device, stream)
    rep = _Report()
    st = lib().ndgp_solve(ctypes.byref(g), ctypes.byref(p), _arr3(dptr), _arr3(pptr),
                          ws.data_ptr(), ws.numel(), _stream(stream), ctypes.byref(rep))
    return phi, _finish(st, rep, check)


def solve_cellwise(grid: Grid, params: Params, delta: Sequence[torch.Tensor],
                   psi: Sequence[Optional[torch.Tensor]], threshold: float, phi=None, ws=None,
                   stream=None, check: bool = True):
    """Run ndgp_solve_cellwise: as solve(), but on every relaxed patch only the
    cells whose parent has |F_5th| >= threshold |F_GR| are iterated (Sec.
    III.C).  ``psi``: Newtonian potential per level, laid out like phi
    (domain n^3, patches padded); entries not needed may be None."""
    g, p = grid._c(), params._c()
    if phi is None:
        phi = alloc_phi(grid, device=delta[0].device)
    dptr, pptr = _solve_ptrs(grid, delta, phi)
    sptr = []
    for lvl in range(len(grid.patches) + 1):
        t = psi[lvl] if lvl < len(psi) else None
        shape = (grid.n,) * 3 if lvl == 0 else (grid.patches[lvl - 1].n + 2,) * 3
        sptr.append(_dev(t, shape, f"psi[{lvl}]") if t is not None else None)
    if ws is None:
        ws = workspace(workspace_bytes(grid, params), delta[0].device, stream)
    rep = _Report()
    st = lib().ndgp_solve_cellwise(ctypes.byref(g), ctypes.byref(p), _arr3(dptr), _arr3(sptr),
                                   float(threshold), _arr3(pptr), ws.data_ptr(), ws.numel(),
                                   _stream(stream), ctypes.byref(rep))
    return phi, _finish(st, rep, check)


def residual(grid: Grid, params: Params, delta: Sequence[torch.Tensor], phi: torch.Tensor,
             level: int = 0, want_r: bool = True, ws=None, stream=None):
    """r = S - L_h[phi] (physical units) on one level, and ||r|| / ||S||."""
    g, p = grid._c(), params._c()
    n = grid.level_n(level)
    shape = (n,) * 3 if level == 0 else (n + 2,) * 3
    dptr = [_dev(delta[0], (grid.n,) * 3, "delta[0]")] + [None] * MAX_PATCHES
    if level:
        dptr[level] = _dev(delta[level], (n,) * 3, f"delta[{level}]")
    r = torch.empty((n,) * 3, dtype=torch.float64, device=phi.device) if want_r else None
    nb = workspace_bytes(grid, params)
    if ws is None:
        ws = workspace(nb, phi.device, stream)
    rel = ctypes.c_double()
    _check(lib().ndgp_residual(ctypes.byref(g), ctypes.byref(p), level, _arr3(dptr),
                               _dev(phi, shape, "phi"), r.data_ptr() if r is not None else None,
                               ctypes.byref(rel), ws.data_ptr(), ws.numel(), _stream(stream)))
    return r, rel.value


NOALLOC_MAX_CELLS = 128**3


def residual_noalloc(grid: Grid, params: Params, delta: Sequence[torch.Tensor], phi: torch.Tensor,
                     level: int = 0, r_out: Optional[torch.Tensor] = None,
                     norms: Optional[torch.Tensor] = None, stream=None):
    """As ``residual`` without a workspace and without blocking: the library's
    static device scratch holds the source and the reduction partials.
    ``norms`` (3 float64 on the device) receives sum r^2, sum S^2 (cell units)
    and the relative norm.  Returns (r_out, norms); allocates nothing itself
    when both are given."""
    g, p = grid._c(), params._c()
    n = grid.level_n(level)
    shape = (n,) * 3 if level == 0 else (n + 2,) * 3
    dptr = [_dev(delta[0], (grid.n,) * 3, "delta[0]")] + [None] * MAX_PATCHES
    if level:
        dptr[level] = _dev(delta[level], (n,) * 3, f"delta[{level}]")
    if norms is None:
        norms = torch.empty(3, dtype=torch.float64, device=phi.device)
    _check(lib().ndgp_residual_noalloc(ctypes.byref(g), ctypes.byref(p), level, _arr3(dptr),
                                       _dev(phi, shape, "phi"),
                                       _dev(r_out, (n,) * 3, "r_out") if r_out is not None
                                       else None, _dev(norms, (3,), "norms"), _stream(stream)))
    return r_out, norms


def force(grid: Grid, phi: Sequence[torch.Tensor], stream=None) -> list:
    """F = -grad(phi)/2 on every level: list of (3, m, m, m) tensors."""
    g = grid._c()
    out, pptr = [], []
    for lvl in range(1 + len(grid.patches)):
        n = grid.level_n(lvl)
        shape = (n,) * 3 if lvl == 0 else (n + 2,) * 3
        pptr.append(_dev(phi[lvl], shape, f"phi[{lvl}]"))
        out.append(torch.empty((3, n, n, n), dtype=torch.float64, device=phi[lvl].device))
    _check(lib().ndgp_force(ctypes.byref(g), _arr3(pptr), _arr3([o.data_ptr() for o in out]),
                            _stream(stream)))
    return out


def _level_ptrs(grid: Grid, fields, name):
    out = []
    for lvl in range(1 + len(grid.patches)):
        n = grid.level_n(lvl)
        shape = (n,) * 3 if lvl == 0 else (n + 2,) * 3
        out.append(_dev(fields[lvl], shape, f"{name}[{lvl}]"))
    return out


def total_force(grid: Grid, phi: Sequence[torch.Tensor], psi: Sequence[torch.Tensor],
                stream=None) -> list:
    """F = -grad(psi) - grad(phi)/2 on every level (Eq. modpoisson): list of
    (3, m, m, m) tensors; psi is the Newtonian potential laid out like phi."""
    g = grid._c()
    out = [torch.empty((3,) + (grid.level_n(l),) * 3, dtype=torch.float64, device=phi[0].device)
           for l in range(1 + len(grid.patches))]
    _check(lib().ndgp_total_force(ctypes.byref(g), _arr3(_level_ptrs(grid, phi, "phi")),
                                  _arr3(_level_ptrs(grid, psi, "psi")),
                                  _arr3([o.data_ptr() for o in out]), _stream(stream)))
    return out


def geff_stats(grid: Grid, phi: Sequence[torch.Tensor], psi: Sequence[torch.Tensor], edges,
               stream=None):
    """G_eff - 1 = |F_5th| / |F_GR| per level over the cells no finer patch
    covers: (list of dicts with cells, sum, sum_sq, min, max, mean; int64
    histogram array of shape (levels, len(edges) + 1))."""
    import numpy as np
    g = grid._c()
    e = np.ascontiguousarray(edges, dtype=np.float64)
    nl = 1 + len(grid.patches)
    outs = (_GeffLevel * (1 + MAX_PATCHES))()
    hist = np.zeros((nl, e.size + 1), dtype=np.int64)
    ws = workspace(GEFF_WORKSPACE, phi[0].device, stream)
    _check(lib().ndgp_geff_stats(ctypes.byref(g), _arr3(_level_ptrs(grid, phi, "phi")),
                                 _arr3(_level_ptrs(grid, psi, "psi")),
                                 e.ctypes.data_as(ctypes.POINTER(ctypes.c_double)), e.size, outs,
                                 hist.ctypes.data_as(ctypes.POINTER(ctypes.c_int64)),
                                 ws.data_ptr(), ws.numel(), _stream(stream)))
    levels = []
    for l in range(nl):
        o = outs[l]
        levels.append({"cells": int(o.cells), "sum": o.sum, "sum_sq": o.sum_sq, "min": o.min,
                       "max": o.max, "mean": o.sum / o.cells if o.cells else float("nan")})
    return levels, hist


def cic_density(grid: Grid, pos: torch.Tensor, delta=None, ws=None, stream=None) -> list:
    """Cloud-in-cell density contrast of equal-mass particles on every level
    (ndgp_cic_density).  ``pos``: float64 device tensor (3, N), box units in
    [0, 1).  Returns [domain n^3, patch m^3, ...] (the layout solve() takes)."""
    if pos.dim() != 2 or pos.shape[0] != 3:
        raise ValueError("pos must have shape (3, N)")
    g = grid._c()
    npart = pos.shape[1]
    if delta is None:
        delta = [torch.empty((grid.level_n(l),) * 3, dtype=torch.float64, device=pos.device)
                 for l in range(1 + len(grid.patches))]
    dptr = [_dev(delta[l], (grid.level_n(l),) * 3, f"delta[{l}]")
            for l in range(1 + len(grid.patches))]
    nb = int(lib().ndgp_cic_density_workspace_bytes(ctypes.byref(g), npart))
    if nb == 0:
        _check(NDGP_EINVAL)
    if ws is None:
        ws = workspace(nb, pos.device, stream)
    _check(lib().ndgp_cic_density(ctypes.byref(g), _dev(pos, (3, npart), "pos"), npart,
                                  _arr3(dptr), ws.data_ptr(), ws.numel(), _stream(stream)))
    return delta


def refine_flags(grid: Grid, delta: Sequence[torch.Tensor], n_particles: int,
                 n_ref: float = 4.0, stream=None):
    """Cells with more than n_ref particles (Sec. IV.A), from cic_density's
    output: (list of uint8 device tensors, list of flagged counts)."""
    g = grid._c()
    nl = 1 + len(grid.patches)
    flags = [torch.empty((grid.level_n(l),) * 3, dtype=torch.uint8, device=delta[0].device)
             for l in range(nl)]
    counts = (ctypes.c_int64 * (1 + MAX_PATCHES))()
    ws = workspace(DIFF_NORMS_WORKSPACE, delta[0].device, stream)
    dptr = [_dev(delta[l], (grid.level_n(l),) * 3, f"delta[{l}]") for l in range(nl)]
    _check(lib().ndgp_refine_flags(ctypes.byref(g), _arr3(dptr), int(n_particles), float(n_ref),
                                   _arr3([f.data_ptr() for f in flags]), counts, ws.data_ptr(),
                                   ws.numel(), _stream(stream)))
    return flags, [int(counts[l]) for l in range(nl)]


@dataclasses.dataclass
class Box:
    """One cubic refinement of a tree (ndgp_box): parent -1 is the domain."""
    parent: int
    n: int
    origin: tuple


class _Box(ctypes.Structure):
    _fields_ = [("parent", ctypes.c_int32), ("n", ctypes.c_int32),
                ("origin", ctypes.c_int32 * 3)]


class _BoxReport(ctypes.Structure):
    _fields_ = [("depth", ctypes.c_int32), ("cycles", ctypes.c_int32),
                ("damped_from", ctypes.c_int32), ("rel_res", ctypes.c_double)]


AMR_MAX_BOXES = 4096


def refine_boxes(flags, n: int, periodic: bool, parent_index: int = -1,
                 efficiency: float = 0.7, min_width: int = 4, max_boxes: int = AMR_MAX_BOXES,
                 stream=None) -> list:
    """Cubic refinement boxes covering the flagged cells of one level
    (ndgp_refine_boxes: Berger-Rigoutsos clustering in the library).  ``flags``
    is a uint8 device tensor or a host array (natural n^3)."""
    import numpy as np
    if isinstance(flags, torch.Tensor) and flags.is_cuda:
        if flags.dtype != torch.uint8 or not flags.is_contiguous() or flags.numel() != n**3:
            raise ValueError("flags must be a contiguous uint8 tensor of n^3 cells")
        ptr, on_dev, keep = flags.data_ptr(), 1, flags
    else:
        keep = np.ascontiguousarray(flags, dtype=np.uint8)
        if keep.size != n**3:
            raise ValueError("flags must hold n^3 cells")
        ptr, on_dev = keep.ctypes.data, 0
    out = (_Box * max(max_boxes, 1))()
    nb = ctypes.c_int32()
    st = _stream(stream) if on_dev else None  # host flags need no device
    _check(lib().ndgp_refine_boxes(ptr, on_dev, n, 1 if periodic else 0, parent_index,
                                   float(efficiency), int(min_width), out, max_boxes,
                                   ctypes.byref(nb), st))
    del keep
    return [Box(out[b].parent, out[b].n, tuple(out[b].origin)) for b in range(nb.value)]


def _boxes_c(boxes):
    arr = (_Box * max(len(boxes), 1))()
    for b, x in enumerate(boxes):
        arr[b].parent, arr[b].n = int(x.parent), int(x.n)
        for a in range(3):
            arr[b].origin[a] = int(x.origin[a])
    return arr


def amr_workspace_bytes(grid: Grid, params: Params, boxes) -> int:
    g, p = grid._c(), params._c()
    nb = lib().ndgp_amr_workspace_bytes(ctypes.byref(g), ctypes.byref(p), _boxes_c(boxes),
                                        len(boxes))
    if nb == 0:
        raise NdgpError(NDGP_EINVAL, lib().ndgp_last_error().decode())
    return int(nb)


def solve_amr(grid: Grid, params: Params, boxes, delta: Sequence[Optional[torch.Tensor]],
              phi=None, ws=None, stream=None, check: bool = True):
    """ndgp_solve_amr: the domain, then every box of the tree from its parent.
    ``delta``: [domain (n^3), box 0 (n_b^3), ...]; returns (phi list with the
    padded boxes, Report of the domain level, list of per-box dicts)."""
    if grid.patches:
        raise ValueError("the tree's boxes replace the grid's nested patches")
    g, p = grid._c(), params._c()
    dev = delta[0].device
    if phi is None:
        phi = [torch.zeros((grid.n,) * 3, dtype=torch.float64, device=dev)] + \
              [torch.zeros((b.n + 2,) * 3, dtype=torch.float64, device=dev) for b in boxes]
    nb = len(boxes)
    dptr = (ctypes.c_void_p * (1 + nb))()
    pptr = (ctypes.c_void_p * (1 + nb))()
    dptr[0] = _dev(delta[0], (grid.n,) * 3, "delta[0]")
    pptr[0] = _dev(phi[0], (grid.n,) * 3, "phi[0]")
    for b, x in enumerate(boxes):
        d = delta[1 + b] if 1 + b < len(delta) else None
        dptr[1 + b] = _dev(d, (x.n,) * 3, f"delta[{1 + b}]") if d is not None else None
        pptr[1 + b] = _dev(phi[1 + b], (x.n + 2,) * 3, f"phi[{1 + b}]")
    if ws is None:
        ws = workspace(amr_workspace_bytes(grid, params, boxes), dev, stream)
    rep = _Report()
    brep = (_BoxReport * max(nb, 1))()
    st = lib().ndgp_solve_amr(ctypes.byref(g), ctypes.byref(p), _boxes_c(boxes), nb, dptr, pptr,
                              ws.data_ptr(), ws.numel(), _stream(stream), ctypes.byref(rep), brep)
    report = _finish(st, rep, check)
    per_box = [{"depth": brep[b].depth, "cycles": brep[b].cycles,
                "damped_from": brep[b].damped_from, "rel_res": brep[b].rel_res}
               for b in range(nb)]
    return phi, report, per_box


def cic_force(grid: Grid, force: Sequence[torch.Tensor], pos: torch.Tensor, out=None,
              stream=None) -> torch.Tensor:
    """Cloud-in-cell interpolation of per-level forces (3, m, m, m) to the
    particles (ndgp_cic_force): (3, N)."""
    g = grid._c()
    npart = pos.shape[1]
    if out is None:
        out = torch.empty((3, npart), dtype=torch.float64, device=pos.device)
    fptr = [_dev(force[l], (3,) + (grid.level_n(l),) * 3, f"force[{l}]")
            for l in range(1 + len(grid.patches))]
    # many particles: scratch that lets them read the components side by side
    nb = int(lib().ndgp_cic_force_workspace_bytes(ctypes.byref(g), npart))
    ws = _scratch(nb, pos.device, stream)
    _check(lib().ndgp_cic_force_in(ctypes.byref(g), _arr3(fptr), _dev(pos, (3, npart), "pos"),
                                   npart, _dev(out, (3, npart), "out"),
                                   ws.data_ptr() if ws is not None else None,
                                   ws.numel() if ws is not None else 0, _stream(stream)))
    return out


DIFF_NORMS_WORKSPACE = 131072


def diff_norms(a: torch.Tensor, b: Optional[torch.Tensor] = None, stream=None):
    """(sum (a-b)^2, sum a^2, sum b^2) over all elements, in the library's
    deterministic reduction kernels."""
    if b is not None and b.shape != a.shape:
        raise ValueError("a and b differ in shape")
    out = (ctypes.c_double * 3)()
    ws = workspace(DIFF_NORMS_WORKSPACE, a.device, stream)
    _check(lib().ndgp_diff_norms(_dev(a, None, "a"), _dev(b, None, "b") if b is not None else None,
                                 a.numel(), out, ws.data_ptr(), ws.numel(), _stream(stream)))
    return out[0], out[1], out[2]


class Plan:
    """A non-blocking solve (ndgp_plan_*): create, then alternate poll() and
    step() until poll() reports done.  Keeps its tensors alive."""

    def __init__(self, grid: Grid, params: Params, delta, phi=None, ws=None, stream=None):
        self.grid, self.params = grid, params
        self._g, self._p = grid._c(), params._c()
        dev0 = delta[0].device
        self.phi = phi if phi is not None else alloc_phi(grid, device=dev0)
        self.delta = list(delta)
        dptr = [_dev(delta[0], (grid.n,) * 3, "delta[0]")]
        for q, pt in enumerate(grid.patches):
            d = delta[q + 1] if q + 1 < len(delta) else None
            dptr.append(_dev(d, (pt.n,) * 3, f"delta[{q + 1}]") if d is not None else None)
        pptr = [_dev(self.phi[0], (grid.n,) * 3, "phi[0]")]
        for q, pt in enumerate(grid.patches):
            pptr.append(_dev(self.phi[q + 1], (pt.n + 2,) * 3, f"phi[{q + 1}]"))
        nb = workspace_bytes(grid, params)
        self.ws = ws if ws is not None else torch.empty(nb, dtype=torch.uint8, device=dev0)
        self.stream = stream
        self._h = ctypes.c_void_p()
        _check(lib().ndgp_plan_create(ctypes.byref(self._g), ctypes.byref(self._p), _arr3(dptr),
                                      _arr3(pptr), self.ws.data_ptr(), self.ws.numel(),
                                      _stream(stream), ctypes.byref(self._h)))
        self.report = None

    def poll(self) -> bool:
        done = ctypes.c_int32()
        rep = _Report()
        st = lib().ndgp_plan_poll(self._h, ctypes.byref(done), ctypes.byref(rep))
        if done.value:
            if st not in (NDGP_OK, NDGP_ENOCONV):
                self.report = _report(rep, st)
                _check(st)
            self.report = _report(rep, st)
            return True
        _check(st)
        return False

    def step(self):
        _check(lib().ndgp_plan_step(self._h))

    def close(self):
        if self._h:
            lib().ndgp_plan_destroy(self._h)
            self._h = ctypes.c_void_p()

    def __del__(self):
        try:
            self.close()
        except Exception:
            pass
