"""Thin ctypes binding of libhermite_lf.so (C ABI in include/hl.h).

Argument marshalling only: every step of the method runs in the library's HIP
kernels.  PyTorch provides device memory and streams.  Importing this module
raises if the library has not been built (there is no CPU fallback).
"""

from __future__ import annotations

import ctypes
import os

import numpy as np

_HERE = os.path.dirname(os.path.abspath(__file__))
# HL_LIBRARY overrides the library path (e.g. a differently tuned build).
LIB_PATH = os.environ.get("HL_LIBRARY", os.path.join(_HERE, "libhermite_lf.so"))

HL_OK, HL_ERR_ARG, HL_ERR_CFL, HL_ERR_UNSUPPORTED, HL_ERR_DEVICE, HL_ERR_NOMEM, HL_ERR_NONFINITE = range(7)
HL_FP64, HL_FP32, HL_FP32_COMP = 0, 1, 2
PRECISIONS = {"fp64": HL_FP64, "fp32": HL_FP32, "fp32_comp": HL_FP32_COMP}
HL_PERIODIC, HL_WALLS = 0, 1
BOUNDARIES = {"periodic": HL_PERIODIC, "walls": HL_WALLS}
HL_INIT_STARTUP = 1

STATUS_NAMES = {0: "HL_OK", 1: "HL_ERR_ARG", 2: "HL_ERR_CFL", 3: "HL_ERR_UNSUPPORTED",
                4: "HL_ERR_DEVICE", 5: "HL_ERR_NOMEM", 6: "HL_ERR_NONFINITE"}

# Every symbol include/hl.h declares.
EXPORTS = ("hl_plan", "hl_plan_destroy", "hl_plan_info", "hl_init", "hl_export", "hl_step",
           "hl_p_half", "hl_u_half", "hl_add_source", "hl_set_kappa", "hl_norms", "hl_norms_noalloc",
           "hl_set_tile", "hl_tune",
           "hl_adjoint_step",
           "hl_adjoint_step_var", "hl_kappa_grad", "hl_batch_create", "hl_batch_step", "hl_batch_destroy",
           "hl_batch_set_sources", "hl_last_error")


class HLProblem(ctypes.Structure):
    _fields_ = [("d", ctypes.c_int32), ("m", ctypes.c_int32), ("cells", ctypes.c_int64 * 3),
                ("length", ctypes.c_double * 3), ("dt", ctypes.c_double), ("cfl", ctypes.c_double),
                ("c", ctypes.c_double), ("precision", ctypes.c_int32), ("boundary", ctypes.c_int32),
                ("reserved", ctypes.c_int32 * 2)]


class HLInfo(ctypes.Structure):
    _fields_ = [("dt", ctypes.c_double), ("nu", ctypes.c_double), ("nodes", ctypes.c_int64),
                ("nc", ctypes.c_int32), ("word_bytes", ctypes.c_int32), ("p_words", ctypes.c_int64),
                ("u_words", ctypes.c_int64), ("tile", ctypes.c_int32 * 2), ("ygroup", ctypes.c_int32),
                ("reserved", ctypes.c_int32)]


class HLError(RuntimeError):
    def __init__(self, status, msg):
        super().__init__(f"{STATUS_NAMES.get(status, status)}: {msg}")
        self.status = status


def load_library(path: str = LIB_PATH) -> ctypes.CDLL:
    if not os.path.exists(path):
        raise ImportError(f"{path} is not built; run __graft_entry__.build() "
                          "(python -m paper_1808_10481_amd.build)")
    lib = ctypes.CDLL(path)
    vp, i64, dbl = ctypes.c_void_p, ctypes.c_int64, ctypes.c_double
    sig = {
        "hl_plan": ([ctypes.POINTER(HLProblem), ctypes.POINTER(vp)]),
        "hl_plan_destroy": ([vp]),
        "hl_plan_info": ([vp, ctypes.POINTER(HLInfo)]),
        "hl_init": ([vp, vp, vp, ctypes.c_uint32, vp, vp, vp]),
        "hl_export": ([vp, vp, vp, vp, vp, vp]),
        "hl_step": ([vp, vp, vp, i64, vp]),
        "hl_p_half": ([vp, vp, vp, vp]),
        "hl_u_half": ([vp, vp, vp, dbl, vp]),
        "hl_norms": ([vp, vp, vp, ctypes.POINTER(dbl)]),
        "hl_norms_noalloc": ([vp, vp, vp, ctypes.POINTER(dbl)]),
        "hl_set_kappa": ([vp, vp, vp]),
        "hl_add_source": ([vp, vp, vp, dbl, vp]),
        "hl_batch_create": ([ctypes.POINTER(vp), ctypes.c_int32, ctypes.POINTER(vp)]),
        "hl_batch_step": ([vp, ctypes.POINTER(vp), ctypes.POINTER(vp), i64, vp]),
        "hl_batch_destroy": ([vp]),
        "hl_batch_set_sources": ([vp, vp, vp, vp, vp, i64]),
        "hl_adjoint_step": ([vp, vp, vp, vp, vp, vp, i64, vp]),
        "hl_adjoint_step_var": ([vp, vp, vp, vp, vp, vp]),
        "hl_set_tile": ([vp, ctypes.c_int32, ctypes.c_int32, ctypes.c_int32]),
        "hl_tune": ([vp, vp, vp, ctypes.c_int32, vp]),
        "hl_kappa_grad": ([vp, vp, vp, ctypes.c_int]),
    }
    for name, args in sig.items():
        fn = getattr(lib, name)
        fn.argtypes = args
        fn.restype = ctypes.c_int
    lib.hl_last_error.argtypes = []
    lib.hl_last_error.restype = ctypes.c_char_p
    return lib


_LIB = None


def lib() -> ctypes.CDLL:
    global _LIB
    if _LIB is None:
        _LIB = load_library()
    return _LIB


def _check(status: int):
    if status != HL_OK:
        raise HLError(status, lib().hl_last_error().decode())


def make_problem(d, m, cells, length=None, dt=0.0, cfl=0.5, c=1.0, precision="fp64",
                 boundary="periodic") -> HLProblem:
    cells = tuple(int(k) for k in cells)
    length = tuple(float(v) for v in (length if length is not None else (1.0,) * d))
    pr = HLProblem()
    pr.d, pr.m = int(d), int(m)
    for k in range(3):
        pr.cells[k] = cells[k] if k < len(cells) else 1
        pr.length[k] = length[k] if k < len(length) else 1.0
    pr.dt, pr.cfl, pr.c = float(dt), float(cfl), float(c)
    pr.precision = PRECISIONS[precision]
    pr.boundary = BOUNDARIES[boundary]
    pr.reserved[0] = pr.reserved[1] = 0
    return pr


_TORCH = None


def _torch():
    global _TORCH
    if _TORCH is None:
        import torch
        _TORCH = torch
    return _TORCH


def _stream_ptr(stream):
    """The stream's handle; the current device's current stream without one
    (read without building a Stream object, 0.2 us instead of 1.5, through
    names that a torch version may lack)."""
    if stream is not None:
        return stream.cuda_stream
    torch = _torch()
    try:
        return torch._C._cuda_getCurrentRawStream(torch._C._cuda_getDevice())
    except AttributeError:
        return torch.cuda.current_stream().cuda_stream


class Plan:
    """A plan for one periodic problem; owns the library handle."""

    def __init__(self, d, m, cells, length=None, dt=0.0, cfl=0.5, c=1.0, precision="fp64",
                 boundary="periodic"):
        self.problem = make_problem(d, m, cells, length, dt, cfl, c, precision, boundary)
        self.kappa = float(c) ** 2
        self.d, self.m, self.precision, self.boundary = int(d), int(m), precision, boundary
        self.cells = tuple(int(k) for k in cells)
        self._dtype = None
        h = ctypes.c_void_p()
        _check(lib().hl_plan(ctypes.byref(self.problem), ctypes.byref(h)))
        self._h = h
        info = HLInfo()
        _check(lib().hl_plan_info(self._h, ctypes.byref(info)))
        self.info = info
        self._p_words, self._u_words = int(info.p_words), int(info.u_words)

    @property
    def dt(self):
        return self.info.dt

    def _refresh_info(self):
        info = HLInfo()
        _check(lib().hl_plan_info(self._h, ctypes.byref(info)))
        self.info = info

    def set_tile(self, tx=0, ty=0, ygroup=0):
        """Tile (workgroup) shape of the half-step launches (hl_set_tile); 0s: defaults."""
        _check(lib().hl_set_tile(self._h, int(tx), int(ty), int(ygroup)))
        self._refresh_info()

    def tune(self, p, u, reps=3, stream=None):
        """Pick the fastest tile shape by timing steps on copies of (p, u)
        (hl_tune); returns (tx, ty, ygroup)."""
        self._check_buf(p, u)
        _check(lib().hl_tune(self._h, ctypes.c_void_p(p.data_ptr()), ctypes.c_void_p(u.data_ptr()), int(reps),
                             _stream_ptr(stream)))
        self._refresh_info()
        return (self.info.tile[0], self.info.tile[1], self.info.ygroup)

    def close(self):
        if getattr(self, "_h", None):
            lib().hl_plan_destroy(self._h)
            self._h = None

    def __del__(self):
        try:
            self.close()
        except Exception:
            pass

    # -- device state ------------------------------------------------------
    def torch_dtype(self):
        """Element type of the state buffers: one word per coefficient in FP64
        and FP32; 16-bit words (three per coefficient: FP32 hi, BF16 lo) in
        fp32_comp."""
        if self._dtype is None:
            t = _torch()
            self._dtype = {"fp64": t.float64, "fp32": t.float32, "fp32_comp": t.int16}[self.precision]
        return self._dtype

    def alloc(self, device="cuda"):
        import torch
        p = torch.empty(self.info.p_words, dtype=self.torch_dtype(), device=device)
        u = torch.empty(self.info.u_words, dtype=self.torch_dtype(), device=device)
        return p, u

    def host_shapes(self):
        """Host array shapes of p and u (walls: K+1 primal nodes per dimension)."""
        extra = 1 if self.boundary == "walls" else 0
        coef = (self.m + 1,) * self.d
        return tuple(k + extra for k in self.cells) + coef, (self.d,) + self.cells + coef

    def init(self, p, u, p0, u0=None, startup=False, stream=None):
        """p0, u0: FP64 host arrays in host layout (C order [j..][a..])."""
        ps, us = self.host_shapes()
        p0 = np.ascontiguousarray(p0, dtype=np.float64)
        assert p0.shape == ps, (p0.shape, ps)
        u0p = None
        if u0 is not None:
            u0 = np.ascontiguousarray(u0, dtype=np.float64)
            assert u0.shape == us, (u0.shape, us)
            u0p = u0.ctypes.data_as(ctypes.c_void_p)
        self._check_buf(p, u)
        _check(lib().hl_init(self._h, p0.ctypes.data_as(ctypes.c_void_p), u0p,
                             HL_INIT_STARTUP if startup else 0, ctypes.c_void_p(p.data_ptr()),
                             ctypes.c_void_p(u.data_ptr()), _stream_ptr(stream)))

    def export(self, p, u, stream=None, want_u=True):
        """FP64 host copies (host layout) of p and, unless want_u is False, u."""
        ps, us = self.host_shapes()
        P = np.empty(ps, dtype=np.float64)
        U = np.empty(us, dtype=np.float64) if want_u else None
        self._check_buf(p, u)
        _check(lib().hl_export(self._h, ctypes.c_void_p(p.data_ptr()), ctypes.c_void_p(u.data_ptr()),
                               P.ctypes.data_as(ctypes.c_void_p),
                               U.ctypes.data_as(ctypes.c_void_p) if want_u else None,
                               _stream_ptr(stream)))
        return P, U

    @property
    def coef_bytes(self):
        """Bytes per stored coefficient (8, 4, or 6 for fp32_comp)."""
        return {"fp64": 8, "fp32": 4, "fp32_comp": 6}[self.precision]

    def step(self, p, u, nsteps=1, stream=None):
        self._check_buf(p, u)
        _check(_LIB.hl_step(self._h, p.data_ptr(), u.data_ptr(), int(nsteps), _stream_ptr(stream)))

    def p_half(self, p, u, stream=None):
        self._check_buf(p, u)
        _check(_LIB.hl_p_half(self._h, p.data_ptr(), u.data_ptr(), _stream_ptr(stream)))

    def u_half(self, u, p, weight_scale=1.0, stream=None):
        self._check_buf(p, u)
        _check(_LIB.hl_u_half(self._h, u.data_ptr(), p.data_ptr(), float(weight_scale), _stream_ptr(stream)))

    def adjoint_step(self, p_bar, u_bar, nsteps=1, p=None, u=None, grad_kappa=None, stream=None):
        """nsteps transposed steps on the adjoint state, in place (hl_adjoint_step).
        With grad_kappa (a one-element FP64 device tensor) the kappa-derivative
        of <p_bar, P_n> + <u_bar, U_n> is added to it; p, u are then the forward
        state (P_n, U_n) after the n steps (not modified)."""
        self._check_buf(p_bar, u_bar)
        pp = uu = gg = None
        if grad_kappa is not None:
            self._check_buf(p, u)
            if grad_kappa.dtype.itemsize != 8 or not grad_kappa.is_cuda or grad_kappa.numel() < 1:
                raise ValueError("grad_kappa must be a float64 device tensor")
            pp, uu = ctypes.c_void_p(p.data_ptr()), ctypes.c_void_p(u.data_ptr())
            gg = ctypes.c_void_p(grad_kappa.data_ptr())
        _check(lib().hl_adjoint_step(self._h, ctypes.c_void_p(p_bar.data_ptr()), ctypes.c_void_p(u_bar.data_ptr()),
                                     pp, uu, gg, int(nsteps), _stream_ptr(stream)))

    def adjoint_step_var(self, p_bar, u_bar, p_next, u_prev, stream=None):
        """One transposed variable-kappa step on the adjoint state, in place,
        adding its kappa gradient to the plan's accumulators
        (hl_adjoint_step_var); p_next = P_{t+1}, u_prev = U_t of the step
        being undone."""
        self._check_buf(p_bar, u_bar)
        self._check_buf(p_next, u_prev)
        _check(lib().hl_adjoint_step_var(self._h, ctypes.c_void_p(p_bar.data_ptr()), ctypes.c_void_p(u_bar.data_ptr()),
                                         ctypes.c_void_p(p_next.data_ptr()), ctypes.c_void_p(u_prev.data_ptr()),
                                         _stream_ptr(stream)))

    def kappa_grad(self, reset=False):
        """(grad_p, grad_u): the accumulated gradient with respect to the kappa
        data, FP64 arrays shaped like set_kappa's inputs (hl_kappa_grad)."""
        n2 = (2 * self.m + 2,) * self.d
        gp = np.zeros(self.host_shapes()[0][:self.d] + n2)    # primal nodes (K+1 per dimension with walls)
        gu = np.zeros(self.cells + n2)
        _check(lib().hl_kappa_grad(self._h, gp.ctypes.data_as(ctypes.c_void_p), gu.ctypes.data_as(ctypes.c_void_p),
                                   1 if reset else 0))
        return gp, gu

    def _clear_kappa_grad(self):
        """Zero the accumulated gradient without copying it out."""
        _check(_LIB.hl_kappa_grad(self._h, None, None, 1))

    def source_buffer(self, g, stream=None):
        """Device buffer (p layout) holding the scaled data g (host layout of p)."""
        import torch
        ps, _ = self.host_shapes()
        g = np.ascontiguousarray(g, dtype=np.float64)
        assert g.shape == ps, (g.shape, ps)
        buf = torch.empty(self.info.p_words, dtype=self.torch_dtype(), device="cuda")
        _check(lib().hl_init(self._h, g.ctypes.data_as(ctypes.c_void_p), None, 0, ctypes.c_void_p(buf.data_ptr()),
                             None, _stream_ptr(stream)))
        return buf

    def add_source(self, p, g, a, stream=None):
        """p += a g (hl_add_source): the source's contribution to one step is
        a = dt r(t_n + dt/2), added after the pressure half-step."""
        dtype = self._dtype or self.torch_dtype()
        if not (p.is_cuda and g.is_cuda) or p.dtype != dtype or g.dtype != dtype:
            raise ValueError("p and g must be device buffers of the plan's storage type")
        if p.numel() < self._p_words or g.numel() < self._p_words:
            raise ValueError("buffers are smaller than the plan's pressure state")
        _check(_LIB.hl_add_source(self._h, p.data_ptr(), g.data_ptr(), float(a), _stream_ptr(stream)))

    def set_kappa(self, kappa_p=None, kappa_u=None):
        """Variable kappa: FP64 Taylor data (nodes,) + (2m+2,)*d about the
        primal nodes (K, or K+1 per dimension with walls) and the dual nodes (K)
        (hl_set_kappa); None, None restores the constant kappa."""
        if kappa_p is None and kappa_u is None:
            _check(lib().hl_set_kappa(self._h, None, None))
            return
        n2 = 2 * self.m + 2
        pshape = self.host_shapes()[0][:self.d] + (n2,) * self.d     # primal nodes (K+1 with walls)
        ushape = self.cells + (n2,) * self.d                           # dual nodes
        kp = np.ascontiguousarray(kappa_p, dtype=np.float64)
        ku = np.ascontiguousarray(kappa_u, dtype=np.float64)
        if kp.shape != pshape or ku.shape != ushape:
            raise ValueError(f"kappa data must have shapes {pshape} (primal) and {ushape} (dual)")
        _check(lib().hl_set_kappa(self._h, kp.ctypes.data_as(ctypes.c_void_p), ku.ctypes.data_as(ctypes.c_void_p)))

    def norms(self, p, u):
        out = (ctypes.c_double * 2)()
        self._check_buf(p, u)
        _check(lib().hl_norms(self._h, ctypes.c_void_p(p.data_ptr()), ctypes.c_void_p(u.data_ptr()), out))
        return out[0], out[1]

    def _check_buf(self, p, u):
        if not (p.is_cuda and u.is_cuda):
            raise ValueError("state buffers must be device tensors")
        dtype = self._dtype or self.torch_dtype()
        if p.dtype != dtype or u.dtype != dtype:
            raise ValueError("state dtype does not match the plan precision")
        if p.numel() < self._p_words or u.numel() < self._u_words:
            raise ValueError("state buffers are smaller than the plan's state")
        if not (p.is_contiguous() and u.is_contiguous()):
            raise ValueError("state buffers must be contiguous")


class Batch:
    """Shots (Plans of the same d, m, precision) advanced together, one launch
    per half-step (hl_batch_*).  Keeps the plans alive."""

    def __init__(self, plans):
        self.plans = list(plans)
        arr = (ctypes.c_void_p * len(self.plans))(*[p._h.value for p in self.plans])
        h = ctypes.c_void_p()
        _check(lib().hl_batch_create(arr, len(self.plans), ctypes.byref(h)))
        self._h = h

    def step(self, ps, us, nsteps=1, stream=None):
        if len(ps) != len(self.plans) or len(us) != len(self.plans):
            raise ValueError("one (p, u) pair per plan")
        for plan, p, u in zip(self.plans, ps, us):
            plan._check_buf(p, u)
        pa = (ctypes.c_void_p * len(ps))(*[p.data_ptr() for p in ps])
        ua = (ctypes.c_void_p * len(us))(*[u.data_ptr() for u in us])
        _check(lib().hl_batch_step(self._h, pa, ua, int(nsteps), _stream_ptr(stream)))

    def set_sources(self, sources, amps=None):
        """Sources inside the batched launch (hl_batch_set_sources).
        sources[i]: None, or (nodes, values) with nodes an int array (k, d) of
        primal node tuples and values a float array (k,) + (m+1,)*d of the
        scaled data of g_i there; amps[i]: the amplitudes dt r(t_n + dt/2)
        of shot i for batch steps n = 0, 1, ...  sources=None removes them."""
        if sources is None:
            _check(lib().hl_batch_set_sources(self._h, None, None, None, None, 0))
            return
        n = len(self.plans)
        if len(sources) != n or amps is None or len(amps) != n:
            raise ValueError("one source (or None) and one amplitude array per shot")
        namps = max([len(a) for a in amps if a is not None] + [0])
        keep = []
        counts = (ctypes.c_int64 * n)()
        nodes = (ctypes.c_void_p * n)()
        vals = (ctypes.c_void_p * n)()
        amp = (ctypes.c_void_p * n)()
        for i, (plan, src) in enumerate(zip(self.plans, sources)):
            if src is not None:
                nd = np.asarray(src[0], dtype=np.int64).reshape(-1, plan.d)
                pn = plan.host_shapes()[0][:plan.d]                 # primal nodes (K+1 with walls)
                flat = np.ravel_multi_index(tuple(nd[:, k] for k in range(plan.d)), pn)
                flat = np.ascontiguousarray(flat, dtype=np.int64)
                v = np.ascontiguousarray(src[1], dtype=np.float64).reshape(nd.shape[0], -1)
                if v.shape[1] != plan.info.nc:
                    raise ValueError("values must hold (m+1)^d coefficients per node")
                counts[i] = nd.shape[0]
                nodes[i], vals[i] = flat.ctypes.data, v.ctypes.data
                keep += [flat, v]
            if amps[i] is not None:
                a = np.zeros(namps)
                a[:len(amps[i])] = np.asarray(amps[i], dtype=np.float64)
                amp[i] = a.ctypes.data
                keep.append(a)
        _check(lib().hl_batch_set_sources(self._h, counts, nodes, vals, amp, namps))

    def close(self):
        if getattr(self, "_h", None):
            lib().hl_batch_destroy(self._h)
            self._h = None

    def __del__(self):
        try:
            self.close()
        except Exception:
            pass
