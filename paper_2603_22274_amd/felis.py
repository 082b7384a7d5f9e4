"""Thin ctypes binding of libfelis.so (include/felis.h).

Argument marshalling only: PyTorch provides device memory and the stream;
every step of the computation runs in the library's HIP kernels.  Functions
carry the C names without the ``felis_`` prefix.  Importing this module
never falls back to another implementation: if the shared library is missing
or cannot be loaded, ``lib()`` raises.
"""
from __future__ import annotations

import ctypes as C
import os

import numpy as np
import torch

_HERE = os.path.dirname(os.path.abspath(__file__))
LIB_PATH = os.path.join(_HERE, 'libfelis.so')

OK, E_INVAL, E_DEVICE, E_BOX, E_CAPACITY, E_OVERFLOW, E_NOCONV, E_UNSUPPORTED = 0, -1, -2, -3, -4, -5, -6, -7
FORCE_SCALE = 4294967296.0
NE = 8
COMPONENTS = ('coul_real', 'lj', 'excl', 'self', 'recip', 'bond', 'restraint', 'total')
ENERGY = 1
PROF_PAIRS, PROF_PME, PROF_NLIST, PROF_INTEGRATE, PROF_UKN, PROF_BARO = 0, 1, 2, 3, 4, 5
BARO_NS = 10                 # values per window from barostat_stats

vp = C.c_void_p


class FelisLeg(C.Structure):
    _fields_ = [
        ('n_atoms', C.c_int32), ('box', C.c_double * 3), ('r_cut', C.c_double), ('skin', C.c_double),
        ('ewald_alpha', C.c_double), ('sc_alpha', C.c_double), ('sc_p', C.c_int32),
        ('grid', C.c_int32 * 3), ('spline_order', C.c_int32),
        ('charge', vp), ('sigma', vp), ('epsilon', vp), ('mass', vp), ('is_ligand', vp),
        ('n_excl', C.c_int32), ('excl_ij', vp), ('excl_ptr', vp), ('excl_idx', vp),
        ('n_bonds', C.c_int32), ('bond_ij', vp), ('bond_k', vp), ('bond_r0', vp),
        ('n_waters', C.c_int32), ('water_ohh', vp), ('d_oh', C.c_double), ('d_hh', C.c_double),
        ('has_restraint', C.c_int32), ('restraint_atoms', C.c_int32 * 6),
        ('restraint_g0', C.c_double * 6), ('restraint_k', C.c_double * 6),
        ('n_windows', C.c_int32), ('lambdas', vp),
        ('x', vp), ('y', vp), ('z', vp), ('vx', vp), ('vy', vp), ('vz', vp),
        ('fx', vp), ('fy', vp), ('fz', vp), ('energy', vp),
        ('seed', C.c_uint64), ('step', C.c_int64), ('list_cap', C.c_int32),
        ('pressure_bar', C.c_double), ('barostat_every', C.c_int32),
        ('n_torsions', C.c_int32), ('torsion_ijkl', vp), ('torsion_k', vp), ('torsion_n', vp),
        ('torsion_phase', vp), ('alch_offset', vp), ('plain_fp64', C.c_int32),
        ('work', vp), ('work_bytes', C.c_size_t),
    ]


_LIB = None


class FelisError(RuntimeError):
    def __init__(self, code, msg):
        super().__init__(f"felis error {code}: {msg}")
        self.code = code


def lib():
    """Load libfelis.so (raises if it has not been built)."""
    global _LIB
    if _LIB is not None:
        return _LIB
    if not os.path.exists(LIB_PATH):
        raise RuntimeError(f"{LIB_PATH} is missing: build it with __graft_entry__.build()")
    L = C.CDLL(LIB_PATH)
    P = C.POINTER
    sig = {
        'felis_create': (C.c_int, [P(vp), C.c_int, vp]),
        'felis_destroy': (None, [vp]),
        'felis_last_error': (C.c_char_p, [vp]),
        'felis_check': (C.c_int, [vp, P(C.c_int32)]),
        'felis_check_detail': (C.c_int, [vp, P(C.c_int32), P(C.c_int32), P(C.c_int32), P(C.c_int32)]),
        'felis_leg_work_size': (C.c_int, [P(FelisLeg), P(C.c_size_t)]),
        'felis_leg_init': (C.c_int, [vp, P(FelisLeg)]),
        'felis_build_nlist': (C.c_int, [vp, P(FelisLeg), C.c_int, C.c_int]),
        'felis_leg_rebuilds': (C.c_int, [vp, P(FelisLeg), vp]),
        'felis_leg_states': (C.c_int, [vp, P(FelisLeg), vp]),
        'felis_restraint_dg': (C.c_int, [vp, vp, C.c_double, P(C.c_double)]),
        'felis_delta_g': (C.c_int, [vp, C.c_int, C.c_double, P(C.c_double)]),
        'felis_segment_bounds': (C.c_int, [C.c_int, C.c_int, vp]),
        'felis_binding_dg': (C.c_int, [vp, C.c_int, vp, C.c_int, vp, vp, C.c_double, P(C.c_double)]),
        'felis_hrex': (C.c_int, [vp, P(FelisLeg), vp, C.c_int64, C.c_int64, C.c_uint64, vp]),
        'felis_barostat': (C.c_int, [vp, P(FelisLeg), C.c_int, C.c_double, C.c_int64]),
        'felis_leg_boxes': (C.c_int, [vp, P(FelisLeg), vp]),
        'felis_leg_boxes_async': (C.c_int, [vp, P(FelisLeg), vp]),
        'felis_barostat_stats': (C.c_int, [vp, P(FelisLeg), vp]),
        'felis_nlist_export_pairs': (C.c_int, [vp, P(FelisLeg), C.c_int, C.c_double, vp, C.c_int64, P(C.c_int64)]),
        'felis_nonbonded': (C.c_int, [vp, P(FelisLeg), C.c_int, C.c_int]),
        'felis_pme': (C.c_int, [vp, P(FelisLeg), C.c_int, C.c_int]),
        'felis_bonded': (C.c_int, [vp, P(FelisLeg), C.c_int, C.c_int]),
        'felis_forces_energy': (C.c_int, [vp, P(FelisLeg), C.c_int, C.c_int]),
        'felis_step': (C.c_int, [vp, P(FelisLeg), C.c_int, C.c_int, C.c_double, C.c_double, C.c_double]),
        'felis_ukn': (C.c_int, [vp, P(FelisLeg), vp, C.c_int, vp, vp, vp, C.c_int64, C.c_int64, vp,
                                C.c_double, vp, C.c_int64]),
        'felis_profile': (C.c_int, [vp, C.c_int]),
        'felis_profile_every': (C.c_int, [vp, C.c_int]),
        'felis_profile_read': (C.c_int, [vp, C.c_int, P(C.c_double), P(C.c_int64)]),
        'felis_mbar_work_size': (C.c_int, [C.c_int, C.c_int64, P(C.c_size_t)]),
        'felis_mbar': (C.c_int, [vp, vp, vp, C.c_int, C.c_int64, C.c_double, C.c_int, vp, P(C.c_int), vp,
                                 C.c_size_t]),
        'felis_mbar_noalloc': (C.c_int, [vp, vp, vp, C.c_int, C.c_int64, C.c_double, C.c_int, vp, P(C.c_int)]),
    }
    for name, (res, args) in sig.items():
        f = getattr(L, name)
        f.restype = res
        f.argtypes = args
    _LIB = L
    return L


def _ptr(t):
    return C.c_void_p(t.data_ptr()) if t is not None else None


class Context:
    """A felis context bound to a device and the current torch stream."""

    def __init__(self, device=0, stream=None):
        self.device = device
        self.stream = stream or torch.cuda.current_stream(device)
        h = vp()
        rc = lib().felis_create(C.byref(h), device, C.c_void_p(self.stream.cuda_stream))
        if rc:
            raise FelisError(rc, "felis_create failed")
        self.h = h

    def check(self, rc):
        if rc:
            raise FelisError(rc, lib().felis_last_error(self.h).decode())

    def device_check(self):
        need, leg, win, atom = C.c_int32(0), C.c_int32(-1), C.c_int32(-1), C.c_int32(-1)
        rc = lib().felis_check_detail(self.h, C.byref(need), C.byref(leg), C.byref(win), C.byref(atom))
        if rc:
            e = FelisError(rc, lib().felis_last_error(self.h).decode() + f" (longest list {need.value})")
            e.needed_cap, e.leg, e.window, e.atom = need.value, leg.value, win.value, atom.value
            raise e

    def close(self):
        if self.h:
            lib().felis_destroy(self.h)
            self.h = None

    def __del__(self):
        try:
            self.close()
        except Exception:
            pass


class Leg:
    """Device-resident leg: topology, per-window state and library scratch for
    a synthetic system (``paper_2603_22274_amd.gen.System``)."""

    def __init__(self, ctx: Context, sysd, windows=None, seed=1234, device='cuda', list_cap=0, positions=None,
                 pressure_bar=0.0, barostat_every=25, plain_fp64=False):
        self.sys = sysd
        self.ctx = ctx
        lam = sysd.lambdas if windows is None else sysd.lambdas[windows]
        self.lambdas = np.ascontiguousarray(lam, np.float64)
        W, N = len(self.lambdas), sysd.n_atoms
        dev = torch.device(device)
        t = lambda a, dt: torch.as_tensor(np.ascontiguousarray(a), dtype=dt, device=dev)
        self.charge = t(sysd.charge, torch.float32)
        self.sigma = t(sysd.sigma, torch.float32)
        self.epsilon = t(sysd.epsilon, torch.float32)
        self.mass = t(sysd.mass, torch.float32)
        self.is_ligand = t(sysd.is_ligand, torch.uint8)
        self.excl_ij = t(sysd.excl.reshape(-1, 2), torch.int32)
        ptr, idx = sysd.excl_csr()
        self.excl_ptr = t(ptr, torch.int32)
        self.excl_idx = t(idx if len(idx) else np.zeros(1, np.int32), torch.int32)
        nb = len(sysd.bonds)
        self.bond_ij = t(sysd.bonds.reshape(-1, 2) if nb else np.zeros((1, 2), np.int32), torch.int32)
        self.bond_k = t(sysd.bond_k if nb else np.zeros(1, np.float32), torch.float32)
        self.bond_r0 = t(sysd.bond_r0 if nb else np.zeros(1, np.float32), torch.float32)
        nw = len(sysd.waters)
        self.water = t(sysd.waters.reshape(-1, 3) if nw else np.zeros((1, 3), np.int32), torch.int32)
        nt = 0 if getattr(sysd, 'torsions', None) is None else len(sysd.torsions)
        self.tors = t(sysd.torsions.reshape(-1, 4) if nt else np.zeros((1, 4), np.int32), torch.int32)
        self.tors_k = t(sysd.torsion_k if nt else np.zeros(1, np.float32), torch.float32)
        self.tors_n = t(sysd.torsion_n if nt else np.ones(1, np.int32), torch.int32)
        self.tors_phase = t(sysd.torsion_phase if nt else np.zeros(1, np.float32), torch.float32)
        off = getattr(sysd, 'alch_offset', None)
        self.alch_offset = t(off, torch.float32) if off is not None and np.any(off) else None
        pos = sysd.pos if positions is None else positions
        pos = np.asarray(pos, np.float32)
        if pos.ndim == 2:
            pos = np.broadcast_to(pos, (W, N, 3))
        self.x = t(pos[..., 0], torch.float32)
        self.y = t(pos[..., 1], torch.float32)
        self.z = t(pos[..., 2], torch.float32)
        self.vx = torch.zeros((W, N), dtype=torch.float32, device=dev)
        self.vy = torch.zeros_like(self.vx)
        self.vz = torch.zeros_like(self.vx)
        self.fx = torch.zeros((W, N), dtype=torch.int64, device=dev)
        self.fy = torch.zeros_like(self.fx)
        self.fz = torch.zeros_like(self.fx)
        self.energy = torch.zeros((W, NE), dtype=torch.float64, device=dev)
        s = FelisLeg()
        s.n_atoms = N
        s.box = (C.c_double * 3)(*[float(v) for v in sysd.box])
        s.r_cut, s.skin, s.ewald_alpha = sysd.r_cut, sysd.skin, sysd.ewald_alpha
        s.sc_alpha, s.sc_p = sysd.sc_alpha, sysd.sc_p
        s.grid = (C.c_int32 * 3)(*sysd.grid)
        s.spline_order = sysd.spline_order
        s.charge, s.sigma, s.epsilon, s.mass = _ptr(self.charge), _ptr(self.sigma), _ptr(self.epsilon), _ptr(self.mass)
        s.is_ligand = _ptr(self.is_ligand)
        s.n_excl = len(sysd.excl)
        s.excl_ij, s.excl_ptr, s.excl_idx = _ptr(self.excl_ij), _ptr(self.excl_ptr), _ptr(self.excl_idx)
        s.n_bonds = nb
        s.bond_ij, s.bond_k, s.bond_r0 = _ptr(self.bond_ij), _ptr(self.bond_k), _ptr(self.bond_r0)
        s.n_waters = nw
        s.water_ohh = _ptr(self.water)
        s.d_oh, s.d_hh = sysd.d_oh, sysd.d_hh
        if sysd.restraint_atoms is not None:
            s.has_restraint = 1
            s.restraint_atoms = (C.c_int32 * 6)(*[int(a) for a in sysd.restraint_atoms])
            s.restraint_g0 = (C.c_double * 6)(*[float(v) for v in sysd.restraint_g0])
            s.restraint_k = (C.c_double * 6)(*[float(v) for v in sysd.restraint_k])
        s.n_windows = W
        s.lambdas = self.lambdas.ctypes.data_as(C.c_void_p)
        s.x, s.y, s.z = _ptr(self.x), _ptr(self.y), _ptr(self.z)
        s.vx, s.vy, s.vz = _ptr(self.vx), _ptr(self.vy), _ptr(self.vz)
        s.fx, s.fy, s.fz = _ptr(self.fx), _ptr(self.fy), _ptr(self.fz)
        s.energy = _ptr(self.energy)
        s.seed = seed
        s.step = 0
        s.list_cap = list_cap
        s.pressure_bar, s.barostat_every = float(pressure_bar), int(barostat_every)
        s.n_torsions = nt
        s.torsion_ijkl, s.torsion_k = _ptr(self.tors), _ptr(self.tors_k)
        s.torsion_n, s.torsion_phase = _ptr(self.tors_n), _ptr(self.tors_phase)
        s.alch_offset = _ptr(self.alch_offset)
        s.plain_fp64 = 1 if plain_fp64 else 0
        nbytes = C.c_size_t(0)
        ctx.check(lib().felis_leg_work_size(C.byref(s), C.byref(nbytes)))
        self.work = torch.empty(int(nbytes.value), dtype=torch.uint8, device=dev)
        s.work, s.work_bytes = _ptr(self.work), nbytes.value
        self.s = s
        ctx.check(lib().felis_leg_init(ctx.h, C.byref(s)))

    @property
    def n_windows(self):
        return self.s.n_windows

    @property
    def n_atoms(self):
        return self.s.n_atoms

    def positions(self):
        return torch.stack([self.x, self.y, self.z], -1)

    def set_positions(self, pos):
        pos = torch.as_tensor(pos, dtype=torch.float32, device=self.x.device)
        if pos.dim() == 2:
            pos = pos.expand(self.n_windows, -1, -1)
        self.x.copy_(pos[..., 0]); self.y.copy_(pos[..., 1]); self.z.copy_(pos[..., 2])
        self.ctx.check(lib().felis_leg_init(self.ctx.h, C.byref(self.s)))

    def forces(self):
        """(W, N, 3) float64 kcal/mol/A."""
        return torch.stack([self.fx, self.fy, self.fz], -1).to(torch.float64) / FORCE_SCALE

    def state_bytes(self):
        tens = [self.x, self.y, self.z, self.vx, self.vy, self.vz, self.fx, self.fy, self.fz, self.energy, self.work]
        return sum(t.numel() * t.element_size() for t in tens)


def leg_footprint(sysd, n_windows=None, list_cap=0, pressure_bar=0.0):
    """Device bytes a ``Leg`` of ``sysd`` holds (library scratch + state and
    topology tensors), computed without allocating anything."""
    W, N = (sysd.n_windows if n_windows is None else n_windows), sysd.n_atoms
    s = FelisLeg()
    s.n_atoms, s.n_windows = N, W
    s.box = (C.c_double * 3)(*[float(v) for v in sysd.box])
    s.r_cut, s.skin, s.ewald_alpha = sysd.r_cut, sysd.skin, sysd.ewald_alpha
    s.sc_alpha, s.sc_p = sysd.sc_alpha, sysd.sc_p
    s.grid = (C.c_int32 * 3)(*sysd.grid)
    s.spline_order = sysd.spline_order
    s.list_cap = list_cap
    s.pressure_bar, s.barostat_every = float(pressure_bar), 25
    s.n_excl, s.n_bonds, s.n_waters = len(sysd.excl), len(sysd.bonds), len(sysd.waters)
    s.n_torsions = 0 if getattr(sysd, 'torsions', None) is None else len(sysd.torsions)
    # felis_leg_work_size validates but never dereferences the arrays
    fake = C.c_void_p(256)
    for k in ('charge', 'sigma', 'epsilon', 'mass', 'is_ligand', 'excl_ij', 'excl_ptr', 'excl_idx', 'bond_ij',
              'bond_k', 'bond_r0', 'water_ohh', 'lambdas', 'x', 'y', 'z', 'vx', 'vy', 'vz', 'fx', 'fy', 'fz',
              'energy', 'torsion_ijkl', 'torsion_k', 'torsion_n', 'torsion_phase'):
        setattr(s, k, fake)
    nbytes = C.c_size_t(0)
    rc = lib().felis_leg_work_size(C.byref(s), C.byref(nbytes))
    if rc:
        raise FelisError(rc, "leg configuration rejected")
    state = W * N * (6 * 4 + 3 * 8) + W * NE * 8
    topo = (N * 17 + (N + 1) * 4 + len(sysd.excl) * 12 + len(sysd.bonds) * 16 + len(sysd.waters) * 12
            + s.n_torsions * 28)
    return int(nbytes.value) + state + topo


def _batch(legs):
    arr = (FelisLeg * len(legs))()
    for i, l in enumerate(legs):
        arr[i] = l.s
    return arr


def _sync_back(legs, arr):
    for i, l in enumerate(legs):
        l.s.step = arr[i].step


def build_nlist(ctx, legs, force=False):
    arr = _batch(legs)
    ctx.check(lib().felis_build_nlist(ctx.h, arr, len(legs), 1 if force else 0))


def leg_rebuilds(ctx, leg):
    """List builds per window since the leg was initialised (numpy int64)."""
    out = np.zeros(leg.n_windows, np.int64)
    ctx.check(lib().felis_leg_rebuilds(ctx.h, C.byref(leg.s), out.ctypes.data_as(C.c_void_p)))
    return out


def leg_states(ctx, leg):
    """State (index into the leg's lambda table) held by each replica (numpy int32)."""
    out = np.zeros(leg.n_windows, np.int32)
    ctx.check(lib().felis_leg_states(ctx.h, C.byref(leg.s), out.ctypes.data_as(C.c_void_p)))
    return out


def restraint_dg(g0, k, temperature=300.0):
    """Free energy (kcal/mol) of imposing the Boresch restraints on the decoupled
    ligand from the 1 mol/L standard state (host computation in the library)."""
    g = np.ascontiguousarray(g0, np.float64)
    kk = np.ascontiguousarray(k, np.float64)
    if g.shape != (6,) or kk.shape != (6,):
        raise ValueError('six restraint geometries and force constants')
    out = C.c_double(0.0)
    rc = lib().felis_restraint_dg(g.ctypes.data_as(C.c_void_p), kk.ctypes.data_as(C.c_void_p), float(temperature),
                                  C.byref(out))
    if rc:
        raise FelisError(rc, 'restraint term: invalid geometry, force constants or temperature')
    return out.value


def delta_g(f, temperature=300.0):
    """kT (f[-1] - f[0]) in kcal/mol from MBAR's free energies (library arithmetic)."""
    ff = np.ascontiguousarray(f, np.float64)
    out = C.c_double(0.0)
    rc = lib().felis_delta_g(ff.ctypes.data_as(C.c_void_p), len(ff), float(temperature), C.byref(out))
    if rc:
        raise FelisError(rc, 'delta_g: at least two finite free energies and a positive temperature')
    return out.value


def segment_bounds(n_windows, n_segments):
    """First window of each segment and the last window of the leg (numpy int32, n_segments + 1)."""
    out = np.zeros(n_segments + 1, np.int32)
    rc = lib().felis_segment_bounds(int(n_windows), int(n_segments), out.ctypes.data_as(C.c_void_p))
    if rc:
        raise FelisError(rc, 'every segment needs at least two windows')
    return out


def binding_dg(dg_solvent_segments, dg_complex_segments, g0, k, temperature=300.0):
    """dG_bind = sum(solvent segments) - sum(complex segments) + dG_restrain (library arithmetic)."""
    a = np.ascontiguousarray(np.atleast_1d(dg_solvent_segments), np.float64)
    b = np.ascontiguousarray(np.atleast_1d(dg_complex_segments), np.float64)
    g = np.ascontiguousarray(g0, np.float64)
    kk = np.ascontiguousarray(k, np.float64)
    if g.shape != (6,) or kk.shape != (6,):
        raise ValueError('six restraint geometries and force constants')
    out = C.c_double(0.0)
    rc = lib().felis_binding_dg(a.ctypes.data_as(C.c_void_p), len(a), b.ctypes.data_as(C.c_void_p), len(b),
                                g.ctypes.data_as(C.c_void_p), kk.ctypes.data_as(C.c_void_p), float(temperature),
                                C.byref(out))
    if rc:
        raise FelisError(rc, 'binding_dg: invalid segment values, restraint geometry or temperature')
    return out.value


def barostat(ctx, legs, temperature, attempt):
    """One Monte Carlo volume move now for every leg of ``legs`` that has a
    pressure (the others are evaluated but unchanged)."""
    legs = legs if isinstance(legs, (list, tuple)) else [legs]
    arr = _batch(legs)
    ctx.check(lib().felis_barostat(ctx.h, arr, len(legs), float(temperature), int(attempt)))
    _sync_back(legs, arr)


def leg_boxes(ctx, leg):
    """(W, 3) numpy float64: each window's current box edges (synchronises)."""
    out = np.zeros((leg.n_windows, 3), np.float64)
    ctx.check(lib().felis_leg_boxes(ctx.h, C.byref(leg.s), out.ctypes.data_as(C.c_void_p)))
    return out


def leg_boxes_device(ctx, leg, out=None):
    """(W, 3) device float64 tensor of each window's box edges, enqueued on
    the context's stream (no host synchronisation)."""
    out = out if out is not None else torch.empty((leg.n_windows, 3), dtype=torch.float64, device=leg.x.device)
    ctx.check(lib().felis_leg_boxes_async(ctx.h, C.byref(leg.s), _ptr(out)))
    return out


def barostat_stats(ctx, leg):
    """(W, 10) numpy float64 per window after the last volume move: U before,
    U after the trial move, w, V, V', s, accepted, dV_max, attempts,
    acceptances (synchronises)."""
    out = np.zeros((leg.n_windows, BARO_NS), np.float64)
    ctx.check(lib().felis_barostat_stats(ctx.h, C.byref(leg.s), out.ctypes.data_as(C.c_void_p)))
    return out


def hrex(ctx, leg, u, attempt, seed, count=True):
    """One replica-exchange attempt among the leg's windows from u[state][replica]
    (device float64, at least n_windows columns).  Returns the number of swaps
    taken (synchronises) when ``count``, else None."""
    n = C.c_int32(0)
    ctx.check(lib().felis_hrex(ctx.h, C.byref(leg.s), _ptr(u), u.stride(0), int(attempt), int(seed) & (2**64 - 1),
                               C.byref(n) if count else None))
    return n.value if count else None


def nlist_export_pairs(ctx, leg, window, r=None, cap=None):
    """Listed pairs (i < j) with FP64 distance < r; returns an (n, 2) int64 numpy array, sorted."""
    r = leg.sys.r_list if r is None else r
    cap = cap or max(1024, leg.n_atoms * 700)
    buf = torch.empty((cap, 2), dtype=torch.int32, device=leg.x.device)
    n = C.c_int64(0)
    ctx.check(lib().felis_nlist_export_pairs(ctx.h, C.byref(leg.s), window, r, _ptr(buf), cap, C.byref(n)))
    p = buf[: n.value].cpu().numpy().astype(np.int64)
    order = np.lexsort((p[:, 1], p[:, 0]))
    return p[order]


def nlist_count_pairs(ctx, leg, window, r=None):
    """Number of listed pairs (i < j) with FP64 distance < r (nothing is copied)."""
    r = leg.sys.r_list if r is None else r
    n = C.c_int64(0)
    rc = lib().felis_nlist_export_pairs(ctx.h, C.byref(leg.s), window, r, None, 0, C.byref(n))
    if rc not in (OK, E_CAPACITY):
        ctx.check(rc)
    return int(n.value)


def nonbonded(ctx, legs, energy=True):
    arr = _batch(legs)
    ctx.check(lib().felis_nonbonded(ctx.h, arr, len(legs), ENERGY if energy else 0))


def pme(ctx, legs, energy=True):
    arr = _batch(legs)
    ctx.check(lib().felis_pme(ctx.h, arr, len(legs), ENERGY if energy else 0))


def bonded(ctx, legs, energy=True):
    arr = _batch(legs)
    ctx.check(lib().felis_bonded(ctx.h, arr, len(legs), ENERGY if energy else 0))


def forces_and_energy(ctx, legs, energy=True):
    """Full force evaluation (list check, real space, PME, bonded)."""
    arr = _batch(legs)
    ctx.check(lib().felis_forces_energy(ctx.h, arr, len(legs), ENERGY if energy else 0))


def step(ctx, legs, n_steps, dt=0.002, temperature=300.0, gamma=0.5):
    arr = _batch(legs)
    ctx.check(lib().felis_step(ctx.h, arr, len(legs), n_steps, dt, temperature, gamma))
    _sync_back(legs, arr)


def ukn(ctx, leg, lambdas, x, y, z, beta, out=None, boxes=None):
    """Reduced potentials [K, n_frames] (device float64) of frames given as
    (n_frames, N) float32 device tensors; ``boxes``: (n_frames, 3) float64
    device tensor of each frame's box edges (None: the leg's box)."""
    lam = np.ascontiguousarray(lambdas, np.float64)
    K = len(lam)
    nf = x.shape[0]
    stride = x.stride(0)
    u = out if out is not None else torch.empty((K, nf), dtype=torch.float64, device=x.device)
    fb = None
    if boxes is not None:
        fb = torch.as_tensor(boxes, dtype=torch.float64, device=x.device).contiguous()
        if fb.shape != (nf, 3):
            raise ValueError('boxes must be (n_frames, 3)')
    ctx.check(lib().felis_ukn(ctx.h, C.byref(leg.s), lam.ctypes.data_as(C.c_void_p), K, _ptr(x), _ptr(y), _ptr(z),
                              stride, nf, _ptr(fb) if fb is not None else None, beta, _ptr(u), u.stride(0)))
    return u


def mbar(ctx, u, N_k, tol=1e-10, max_iter=100000):
    """Dimensionless free energies (numpy, gauge f_0 = 0) and iterations."""
    u = u.contiguous()
    K, N = u.shape
    nk = np.ascontiguousarray(N_k, np.int32)
    nbytes = C.c_size_t(0)
    ctx.check(lib().felis_mbar_work_size(K, N, C.byref(nbytes)))
    work = torch.empty(int(nbytes.value), dtype=torch.uint8, device=u.device)
    f = np.zeros(K, np.float64)
    it = C.c_int(0)
    ctx.check(lib().felis_mbar(ctx.h, _ptr(u), nk.ctypes.data_as(C.c_void_p), K, N, tol, max_iter,
                               f.ctypes.data_as(C.c_void_p), C.byref(it), _ptr(work), nbytes.value))
    return f, it.value


def mbar_noalloc(ctx, u, N_k, tol=1e-10, max_iter=100000):
    """As ``mbar`` through the allocation-free entry point (scratch in the
    library's static device array; ``u`` must already be contiguous)."""
    if not u.is_contiguous():
        raise ValueError('u must be contiguous (no copy is made here)')
    K, N = u.shape
    nk = np.ascontiguousarray(N_k, np.int32)
    f = np.zeros(K, np.float64)
    it = C.c_int(0)
    ctx.check(lib().felis_mbar_noalloc(ctx.h, _ptr(u), nk.ctypes.data_as(C.c_void_p), K, N, tol, max_iter,
                                       f.ctypes.data_as(C.c_void_p), C.byref(it)))
    return f, it.value


def profile(ctx, enable=True, stages=None, every=1):
    """Record HIP events around every stage (``stages`` None) or only around
    the given PROF_* stages, bracketing every ``every``-th occurrence of each;
    ``enable`` False stops recording."""
    ctx.check(lib().felis_profile_every(ctx.h, int(every)))
    if not enable:
        v = 0
    elif stages is None:
        v = 1
    else:
        v = 0x40000000 | sum(1 << int(t) for t in stages)
    ctx.check(lib().felis_profile(ctx.h, v))


def profile_read(ctx, which):
    """(total milliseconds, launches) bracketed for stage ``which`` since the last read."""
    ms = C.c_double(0)
    n = C.c_int64(0)
    ctx.check(lib().felis_profile_read(ctx.h, which, C.byref(ms), C.byref(n)))
    return ms.value, n.value
