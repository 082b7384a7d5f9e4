"""MD steps repeat to the last bit, from a process's first launch on, on legs
whose bonded chains span many waves of the integrator, however the steps are
divided into calls; and every free atom's velocity after a step is the one that
the forces at the step's start and the documented noise give."""
import math

import numpy as np
import pytest
import torch

from oracle.integrate import normals
from paper_2603_22274_amd import gen

pytestmark = pytest.mark.gpu
KB, ACCEL, DT, T, GAMMA, SEED = 0.0019872043, 418.4, 0.002, 300.0, 0.5, 9


def _state(leg):
    return [t.clone() for t in (leg.x, leg.y, leg.z, leg.vx, leg.vy, leg.vz, leg.fx, leg.fy, leg.fz)]


def _leg(felis, ctx, s):
    leg = felis.Leg(ctx, s, seed=SEED)
    g = torch.Generator(device='cuda')
    g.manual_seed(3)
    for v in (leg.vx, leg.vy, leg.vz):
        v.copy_(4.0 * torch.randn(v.shape, generator=g, device='cuda'))
    return leg


@pytest.mark.parametrize('make', [gen.config2, gen.small_complex, gen.torsion_leg])
def test_steps_repeat_and_follow_the_starting_forces(make):
    from paper_2603_22274_amd import felis
    s = make()
    free = np.setdiff1d(np.arange(s.n_atoms), s.waters.reshape(-1))
    ctx = felis.Context(0)
    leg = _leg(felis, ctx, s)
    felis.step(ctx, [leg], 4, DT, T, GAMMA)
    first = _state(leg)
    for _ in range(2):
        leg = _leg(felis, ctx, s)
        felis.step(ctx, [leg], 4, DT, T, GAMMA)
        assert all(torch.equal(a, b) for a, b in zip(first, _state(leg)))
    leg = _leg(felis, ctx, s)
    m = s.mass[free].astype(np.float64)[:, None]
    a = math.exp(-GAMMA * DT)
    sd = np.sqrt((1.0 - a * a) * KB * T * ACCEL / m)
    for k in range(4):
        felis.forces_and_energy(ctx, [leg], energy=False)
        F = leg.forces()[:, free].cpu().numpy()
        v = torch.stack([leg.vx, leg.vy, leg.vz], -1)[:, free].double().cpu().numpy()
        felis.step(ctx, [leg], 1, DT, T, GAMMA)
        got = torch.stack([leg.vx, leg.vy, leg.vz], -1)[:, free].double().cpu().numpy()
        for w in sorted({0, 1, s.n_windows // 2, s.n_windows - 1}):
            want = a * (v[w] + DT * ACCEL * F[w] / m) + sd * normals(SEED, w, k, s.n_atoms)[free]
            # bonded forces agree to 2e-3 kcal/mol/A (summed per atom in FP32 here, per term there); the rest
            # is FP32: some 16 roundings of the speed, the kick and the noise
            bound = DT * ACCEL * 2e-3 / m + 16 * 2.0 ** -24 * (np.abs(v[w]) + DT * ACCEL * np.abs(F[w]) / m + 6 * sd)
            err = np.abs(got[w] - want)
            assert (err <= bound).all(), (k, w, float(err.max()), int(free[(err - bound).max(1).argmax()]))
    assert all(torch.equal(a, b) for a, b in zip(first, _state(leg)))
    ctx.device_check()
    ctx.close()
