"""Heisenberg spin-glass Monte Carlo on AMD MI355X (gfx950).

Python binding of ``libhsg.so`` (C interface in ``include/hsg.h``).  This module
only marshals arguments: every step of a sweep runs in the HIP kernels of the
library.  PyTorch provides device memory and the current HIP stream.

The model and dynamics are those of Bernaschi, Parisi & Parisi, "The Heisenberg spin
glass model on GPU: myths and actual facts" (arXiv:1006.2566): 3-component unit spins
on an L^3 periodic lattice with Gaussian couplings (§2, eqs. 1-2), checkerboard
updates with over-relaxation (§4), plus the Metropolis / heat-bath moves the paper
names, driven by a Philox counter-based generator.
"""
from __future__ import annotations

import ctypes
import math
import os

import torch

__all__ = ["Lattice", "HsgError", "lib", "lattice_bytes", "LIB_PATH"]

_HERE = os.path.dirname(os.path.abspath(__file__))
LIB_PATH = os.path.join(_HERE, "libhsg.so")

HSG_F32, HSG_F64 = 0, 1
HSG_HEAT_BATH = 1
HSG_SNAKE = 2
HSG_FUSED = 4
HSG_MARCH_PHASE = 16
HSG_PLANE_LAUNCH = 32
HSG_STREAM_LOADS = 64
HSG_PHASE_LAUNCH = 128
HSG_PHASE_MC = 256
HSG_BRICK = 2048
# launch kinds reported by hsg_sweep_timed
LAUNCH_OTHER, LAUNCH_MC_PASS, LAUNCH_OR_PASS, LAUNCH_OR_PHASE, LAUNCH_OR_PHASE_MC, \
    LAUNCH_MARCH = range(6)
LAUNCH_NAMES = ("other", "mc_pass", "or_pass", "or_phase", "or_phase_mc", "march")
FUSED_MIN_L, FUSED_MAX_L = 256, 1024
PHASE_MIN_L, PHASE_MAX_L = 98, 1024
BRICK_MAX_L, BRICK_MAX_L_F64 = 64, 40
FOURIER_VALUES = 65
L_MAX = 1290


def fused_supported(L: int) -> bool:
    """Whether HSG_FUSED takes effect for an L^3 lattice."""
    return FUSED_MIN_L <= L <= FUSED_MAX_L and L % 64 == 0


def phase_supported(L: int) -> bool:
    """Whether HSG_PHASE_LAUNCH takes effect for an L^3 lattice (even L from 98 to 1024,
    whose offsets fit 32 bits, and L = 64)."""
    return L <= PHASE_MAX_L and ((L >= PHASE_MIN_L and L % 2 == 0) or L == 64)


def default_flags(L: int, dtype=None) -> int:
    """Traversal flags by the lattice alone: several colour passes per launch on small
    lattices (L <= 64, in binary64 40); Monte Carlo passes one launch each in alternating z
    order, and for multiples of 64 from 256 up over-relaxation phases as one launch each --
    in binary32 with the next sweep's colour-0 Monte Carlo pass in the same launch.
    Spins are the same either way.  A sweep that names no flags also looks at its hits
    (call_flags).  hsg_sweep_noalloc takes neither HSG_BRICK nor the phase launches; HSG_BRICK
    goes with HSG_HEAT_BATH and HSG_SNAKE alone (Lattice.sweep drops it beside others)."""
    f64 = dtype is not None and str(dtype) in ("torch.float64", "float64")
    if L <= (BRICK_MAX_L_F64 if f64 else BRICK_MAX_L):
        return HSG_SNAKE | HSG_BRICK
    if not (L >= 256 and L % 64 == 0 and phase_supported(L)):
        return HSG_SNAKE
    return HSG_SNAKE | (HSG_PHASE_LAUNCH if f64 else HSG_PHASE_MC)


def _brick_hits(L: int, f64: bool, n_or: int) -> float:
    """Most Metropolis hits with which the small lattices' launches are the faster.

    One workgroup has the hits of a whole lattice to do, and a brick those of its ring again,
    where a pass has the whole chip; every over-relaxation phase saves launches, worth some hits
    more.  us a sweep with one such phase, colour passes / HSG_BRICK: one workgroup, L = 10 k =
    64 36.7 / 32.8, 256 104 / 126; 12 and 16 18.2 / 18.1, 64 36.6 / 64.5; 14 and 8 16.0 / 14.2,
    16 18.3 / 24.8; binary64 10 and 16 22.1 / 19.9, 32 31.9 / 36.8.  Bricks: 24 and 256 130 / 102;
    44 and 16 19.7 / 18.1, 32 24.9 / 26.2; 48 and 8 17.2 / 16.6, 16 19.1 / 21.6; 64 and 8 20.1 /
    19.2, 16 23.3 / 25.4, 64 47.2 / 61.8; binary64 14 and 16 23.3 / 21.7, 32 33.2 / 36.7; 36 and 8
    20.0 / 18.3, 16 24.7 / 24.9, 64 53.9 / 64.6."""
    if f64:
        a, b = ((12, 10) if L == 10 else (14, 3) if L == 14 else (10, 3) if L >= 34 else
                (float("inf"), 0))
    else:
        a, b = ((56, 40) if L == 10 else (11, 6) if L == 12 else (5, 4.5) if L == 14 else
                (12, 0) if L == 46 else (8, 0) if L >= 48 else (28, 6) if L >= 34 else
                (float("inf"), 0))
    return a + b * n_or


# Bytes of spins and couplings, 6 L^3 values, that colour passes in place find in the 256 MB
# memory-side cache, but launches that also read or write a second spin array (9 L^3) do not.
PHASE_CACHE_BYTES = (204_000_000, 272_000_000)


def call_flags(L: int, dtype=None, k: int = 1, heat_bath: bool = False, n_or: int = 1) -> int:
    """Traversal flags of a sweep that names none, by its hits and over-relaxation phases.
    Small lattices run pass by pass where the hits are many (_brick_hits).  Over
    default_flags, every even L from 98 to 1024 runs its over-relaxation phases in launches
    of one or two, the last of a sweep with the next sweep's colour-0 Monte Carlo pass where
    that pays.  us a sweep on MI355X with one over-relaxation phase, colour passes / a launch
    per phase / with the Monte Carlo pass:

      binary32  L = 98 k = 1  28.4 / 26.5 / 25.3     98 k = 2  29.4 / 27.3 / 27.6
                   122 k = 2  42.6 / 40.6 / 39.9    178 k = 1   101 / 89.4 / 79.2
                   146 k = 3  65.4 / 61.9 / 59.9    178 k = 4   108 / 98.2 /  102
                   146 heat bath 64.6 / 61.9 / 59.6 194 heat bath 132 / 121 / 123
                   210 k = 1   161 /  167 /  143    218 k = 1   177 /  189 /  175
                   218 k = 4   186 /  194 /  198    242 k = 4   330 /  294 /  275
                   242 k = 8   377 /  340 /  367    258 k = 8   462 /  414 /  398
                   512 k = 4  3281 / 2753 / 2412    512 k = 8  3701 / 3224 / 2994
      binary64  L =122 k = 1  74.0 / 67.7 / 68.2    130 k = 1  86.0 / 81.1 / 78.1
                   146 k = 2   117 /  108 /  119    178 k = 1   211 /  229 /  214
                   182 k = 4   269 /  260 /  256    320 k = 8  2111 / 1845 / 1923
                   448 k = 8  5891 / 5165 / 5153    512 k = 8  9040 / 7930 / 8050
                   512 k = 4  7170 / 6090 / 5660    320 heat bath 1656 / 1386 / 1689

    so binary32 takes the pass along with one hit, from L = 114 with two, from 128 with three
    or a heat bath, from 226 with four and from 256 always; binary64 with one hit from 126,
    with up to four from 180, never with more or a heat bath.  Where only the passes'
    footprint fits the memory-side cache (206 <= L <= 224, in binary64 162 to 178) they stay,
    but for one hit in binary32.

    With an even number of phases the Monte Carlo pass would break up a pair of them.  Two
    phases, passes / pairs / with the Monte Carlo pass: binary32 L = 130 k = 4 73.2 / 61.1 /
    67.3, 162 k = 1 119 / 99.0 / 95.5, 210 k = 4 245 / 227 / 236, 258 k = 1 602 / 448 / 471,
    320 k = 4 1139 / 906 / 827, 512 k = 8 5338 / 4004 / 4036; binary64 130 k = 1 128 / 110 /
    115, 258 k = 1 1251 / 971 / 975, 384 k = 4 4292 / 3257 / 3489: it goes along from L = 310
    with up to four hits or a heat bath, in binary32 only.  An odd number is as one phase,
    without the exception for the cache (218 k = 4, three phases: 362 / 343 / 340)."""
    f64 = dtype is not None and str(dtype) in ("torch.float64", "float64")
    f = default_flags(L, dtype)
    if f & HSG_BRICK and k > 5 and not heat_bath and k > _brick_hits(L, f64, n_or):
        return f & ~HSG_BRICK
    if L < PHASE_MIN_L or not phase_supported(L):
        return f
    if n_or > 0 and n_or % 2 == 0:
        carry = not f64 and L >= 310 and (heat_bath or k <= 4)
    elif f64:
        carry = not heat_bath and ((L >= 126 and k <= 1) or (L >= 180 and k <= 4))
    else:
        carry = (L >= (128 if heat_bath or k == 3 else 226 if k == 4 else 256) or
                 (not heat_bath and (k <= 1 or (k == 2 and L >= 114))))
    lo, hi = PHASE_CACHE_BYTES
    if (lo < 6 * L ** 3 * (8 if f64 else 4) < hi and n_or <= 1 and k > 0 and
            (f64 or heat_bath or k != 1)):
        return f
    return f & ~HSG_PHASE_MC | (HSG_PHASE_MC if carry and k > 0 else HSG_PHASE_LAUNCH)


class HsgError(RuntimeError):
    """A libhsg call returned an error status."""

    def __init__(self, code: int, message: str):
        super().__init__(f"libhsg error {code}: {message}")
        self.code = code


class _Lattice(ctypes.Structure):
    _fields_ = [("L", ctypes.c_int32), ("dtype", ctypes.c_int32), ("seed", ctypes.c_uint64),
                ("sweep", ctypes.c_uint64), ("spins", ctypes.c_void_p), ("J", ctypes.c_void_p),
                ("E", ctypes.c_void_p), ("work", ctypes.c_void_p), ("work_bytes", ctypes.c_size_t)]


class _SweepParams(ctypes.Structure):
    _fields_ = [("T", ctypes.c_double), ("k_hits", ctypes.c_int32), ("n_or", ctypes.c_int32),
                ("renorm_every", ctypes.c_int32), ("flags", ctypes.c_int32)]


_lib = None


def lib() -> ctypes.CDLL:
    """The loaded HIP library.  Raises if it has not been built: there is no fallback."""
    global _lib
    if _lib is None:
        if not os.path.exists(LIB_PATH):
            raise ImportError(f"{LIB_PATH} is missing; build it with "
                              "`python -c 'import __graft_entry__ as g; g.build()'`")
        L = ctypes.CDLL(LIB_PATH)
        P, I32, SZ = ctypes.c_void_p, ctypes.c_int32, ctypes.POINTER(ctypes.c_size_t)
        LP = ctypes.POINTER(_Lattice)
        L.hsg_lattice_bytes.argtypes = [I32, I32, SZ, SZ, SZ]
        L.hsg_init_lattice.argtypes = [LP, P]
        L.hsg_import.argtypes = [LP, P, P, P]
        L.hsg_export.argtypes = [LP, P, P, P]
        L.hsg_sweep.argtypes = [LP, ctypes.POINTER(_SweepParams), I32, P]
        L.hsg_sweep_timed.argtypes = [LP, ctypes.POINTER(_SweepParams), I32, P, I32, P, P,
                                      ctypes.POINTER(I32)]
        L.hsg_sweep_noalloc.argtypes = [LP, ctypes.POINTER(_SweepParams), I32, P]
        L.hsg_energy.argtypes = [LP, I32, P, P]
        L.hsg_overlap.argtypes = [LP, LP, P, P]
        L.hsg_overlap_fourier.argtypes = [LP, LP, P, P]
        L.hsg_last_error.restype = ctypes.c_char_p
        for name in ("hsg_lattice_bytes", "hsg_init_lattice", "hsg_import", "hsg_export",
                     "hsg_sweep", "hsg_sweep_timed", "hsg_sweep_noalloc", "hsg_energy",
                     "hsg_overlap",
                     "hsg_overlap_fourier"):
            getattr(L, name).restype = ctypes.c_int
        _lib = L
    return _lib


def check(rc: int) -> None:
    if rc != 0:
        raise HsgError(rc, lib().hsg_last_error().decode())


def _dtype_code(dtype: torch.dtype) -> int:
    if dtype == torch.float32:
        return HSG_F32
    if dtype == torch.float64:
        return HSG_F64
    raise TypeError(f"spins are float32 or float64, not {dtype}")


def lattice_bytes(L: int, dtype: torch.dtype = torch.float32) -> tuple[int, int, int]:
    """(spin_bytes, J_bytes, work_bytes) of an L^3 lattice."""
    s, j, w = ctypes.c_size_t(), ctypes.c_size_t(), ctypes.c_size_t()
    check(lib().hsg_lattice_bytes(L, _dtype_code(dtype), ctypes.byref(s), ctypes.byref(j),
                                  ctypes.byref(w)))
    return s.value, j.value, w.value


def _stream(stream=None) -> ctypes.c_void_p:
    s = stream if stream is not None else torch.cuda.current_stream()
    return ctypes.c_void_p(s.cuda_stream)


def _ptr(t: torch.Tensor) -> ctypes.c_void_p:
    return ctypes.c_void_p(t.data_ptr())


class Lattice:
    """One L^3 lattice resident on the GPU (colour-split layout, see include/hsg.h).

    ``init="random"`` draws the Philox initial state from ``seed``; ``init=None``
    leaves the buffers for :meth:`load`.
    """

    def __init__(self, L: int, dtype: torch.dtype = torch.float32, seed: int = 1,
                 device: str | torch.device = "cuda", init: str | None = "random",
                 stream=None):
        spin_b, j_b, work_b = lattice_bytes(L, dtype)
        self.L, self.dtype, self.device = L, dtype, torch.device(device)
        n = 3 * L ** 3
        self.spins = torch.empty(n, dtype=dtype, device=self.device)
        self.J = torch.empty(n, dtype=dtype, device=self.device)
        self.E = torch.zeros(1, dtype=torch.float64, device=self.device)
        self.work = torch.empty(work_b, dtype=torch.uint8, device=self.device)
        # partial sums, zero between calls; a second spin array behind them (from L = 64 up the
        # larger of the two) is written before it is read, and takes 1.3 GB at L = 382 binary64
        spare = work_b - spin_b
        self.work[:spare if L >= 64 and spare > 0 else work_b].zero_()
        self._d = _Lattice(L, _dtype_code(dtype), seed & (2 ** 64 - 1), 0, self.spins.data_ptr(),
                           self.J.data_ptr(), self.E.data_ptr(), self.work.data_ptr(), work_b)
        if init == "random":
            self.init_random(stream)

    # ------------------------------------------------------------------ state
    @property
    def N(self) -> int:
        return self.L ** 3

    @property
    def seed(self) -> int:
        return self._d.seed

    @property
    def sweep_index(self) -> int:
        return self._d.sweep

    @sweep_index.setter
    def sweep_index(self, value: int) -> None:
        self._d.sweep = int(value)

    def init_random(self, stream=None) -> None:
        check(lib().hsg_init_lattice(ctypes.byref(self._d), _stream(stream)))

    def load(self, spins, J=None, stream=None) -> None:
        """Load canonical-layout spins (and couplings), shape (3, N), any device."""
        s = torch.as_tensor(spins).to(device=self.device, dtype=self.dtype).contiguous()
        assert s.numel() == 3 * self.N
        j = None
        if J is not None:
            j = torch.as_tensor(J).to(device=self.device, dtype=self.dtype).contiguous()
            assert j.numel() == 3 * self.N
        check(lib().hsg_import(ctypes.byref(self._d), _ptr(s), _ptr(j) if j is not None else None,
                               _stream(stream)))
        torch.cuda.current_stream().synchronize() if stream is None else stream.synchronize()

    def export(self, stream=None) -> tuple[torch.Tensor, torch.Tensor]:
        """Canonical-layout (spins, J), each of shape (3, N), on the device."""
        s = torch.empty((3, self.N), dtype=self.dtype, device=self.device)
        j = torch.empty((3, self.N), dtype=self.dtype, device=self.device)
        check(lib().hsg_export(ctypes.byref(self._d), _ptr(s), _ptr(j), _stream(stream)))
        return s, j

    # --------------------------------------------------------------- dynamics
    def _flags(self, flags: int | None, k: int, heat_bath: bool, n_or: int) -> int:
        if flags is None:
            return call_flags(self.L, self.dtype, k, heat_bath, n_or)
        f = int(flags)
        # default_flags() with a traversal flag added: the traversal that was asked for
        return f if f & ~(HSG_HEAT_BATH | HSG_SNAKE | HSG_BRICK) == 0 else f & ~HSG_BRICK

    def sweep(self, T: float, k: int = 1, n_or: int = 0, renorm_every: int = 0,
              n_sweeps: int = 1, heat_bath: bool = False, flags: int | None = None,
              stream=None) -> None:
        """n_sweeps sweeps; flags None = call_flags(L, dtype, k, heat_bath, n_or)."""
        f = self._flags(flags, k, heat_bath, n_or)
        p = _SweepParams(float(T), int(k), int(n_or), int(renorm_every),
                         (HSG_HEAT_BATH if heat_bath else 0) | f)
        check(lib().hsg_sweep(ctypes.byref(self._d), ctypes.byref(p), int(n_sweeps),
                              _stream(stream)))

    def sweep_timed(self, T: float, k: int = 1, n_or: int = 0, renorm_every: int = 0,
                    n_sweeps: int = 1, heat_bath: bool = False, flags: int | None = None,
                    capacity: int = 4096, stream=None) -> list[tuple[int, float]]:
        """As sweep(), with every launch timed by HIP events on the launch stream:
        [(launch kind, ms)] in launch order (hsg_sweep_timed; waits for the stream)."""
        import numpy as np
        f = self._flags(flags, k, heat_bath, n_or)
        p = _SweepParams(float(T), int(k), int(n_or), int(renorm_every),
                         (HSG_HEAT_BATH if heat_bath else 0) | f)
        kinds = np.zeros(capacity, dtype=np.int32)
        ms = np.zeros(capacity, dtype=np.float32)
        n = ctypes.c_int32()
        check(lib().hsg_sweep_timed(ctypes.byref(self._d), ctypes.byref(p), int(n_sweeps),
                                    _stream(stream), capacity, kinds.ctypes.data_as(ctypes.c_void_p),
                                    ms.ctypes.data_as(ctypes.c_void_p), ctypes.byref(n)))
        return [(int(kinds[i]), float(ms[i])) for i in range(n.value)]

    # ---------------------------------------------------------- observables
    def energy(self, recompute: bool = False, stream=None) -> torch.Tensor:
        """Energy H as a 1-element float64 device tensor (tracked or recomputed)."""
        out = torch.empty(1, dtype=torch.float64, device=self.device)
        check(lib().hsg_energy(ctypes.byref(self._d), int(bool(recompute)), _ptr(out),
                               _stream(stream)))
        return out

    def overlap(self, other: "Lattice", stream=None) -> torch.Tensor:
        """15 float64 values: Q[3x3] row-major, then m_self[3], m_other[3]."""
        out = torch.empty(15, dtype=torch.float64, device=self.device)
        check(lib().hsg_overlap(ctypes.byref(self._d), ctypes.byref(other._d), _ptr(out),
                                _stream(stream)))
        return out

    def overlap_fourier(self, other: "Lattice", out: torch.Tensor | None = None,
                        stream=None) -> torch.Tensor:
        """The 65-value record of hsg_overlap_fourier: Q(0) (9), Re/Im Q(k_d) for
        d = x, y, z (18 each), q2(0), q2(k_min)."""
        if out is None:
            out = torch.empty(FOURIER_VALUES, dtype=torch.float64, device=self.device)
        check(lib().hsg_overlap_fourier(ctypes.byref(self._d), ctypes.byref(other._d),
                                        _ptr(out), _stream(stream)))
        return out


def beta(T: float) -> float:
    return 0.0 if math.isinf(T) else 1.0 / T
