"""u_kn where its kernels change: ligands at and across the box faces and
whole boxes away (the bounding sphere, the touched rows of the transform), odd
and single frames, passes that follow each other on one leg with the ligand
elsewhere, one and many lambda_vdw values (the lanes of the softcore sums), an
alchemical-water set, grids of one and several row chunks."""
import numpy as np
import pytest
import torch

from oracle import ukn as oukn
from paper_2603_22274_amd import gen

pytestmark = pytest.mark.gpu
BETA = 1.0 / (0.0019872043 * 300.0)


def _lam(kv):
    lv = np.linspace(0.0, 1.0, kv)
    return np.stack([np.where(lv == 1.0, 0.5, 0.0), lv, np.zeros(kv)], 1)


def _check(felis, ctx, leg, s, frames, lam):
    x, y, z = (torch.as_tensor(np.ascontiguousarray(frames[..., d])).cuda() for d in range(3))
    u = felis.ukn(ctx, leg, lam, x, y, z, BETA).cpu().numpy()
    ctx.device_check()
    ref = oukn.ukn(s, frames.astype(np.float64), lam, BETA)
    # FP32 transform and erfc (1e-6 of the terms), as the parity tests hold u_kn
    assert np.max(np.abs(u - ref)) <= 1e-6 * np.abs(ref).max() + 2e-4, np.max(np.abs(u - ref))


@pytest.mark.parametrize('shift', [(0.0, 0.0, 0.0), (9.3, 9.3, 9.3), (-9.0, 0.4, 27.9)])
@pytest.mark.parametrize('nf,kv', [(1, 1), (3, 12), (5, 33), (2, 64)])
def test_frames_states_and_places(shift, nf, kv):
    from paper_2603_22274_amd import felis
    s = gen.config0()
    rng = np.random.default_rng([nf, kv])
    frames = (s.pos + np.float32(shift) + rng.normal(0, 0.03, (nf, s.n_atoms, 3))).astype(np.float32)
    ctx = felis.Context(0)
    leg = felis.Leg(ctx, s, windows=[0, 5, 11], seed=1)          # two complex grids: up to four frames a pass
    _check(felis, ctx, leg, s, frames, _lam(kv))
    _check(felis, ctx, leg, s, np.roll(frames, 1, 2), _lam(kv)[:1])       # the ligand elsewhere, the same scratch
    ctx.close()


@pytest.mark.parametrize('q', [1.0, -1.0])
def test_alchemical_waters(q):
    from paper_2603_22274_amd import felis
    s = gen.charged_leg(q_ligand=q)
    frames = np.stack([s.pos, s.pos + np.float32(5.5)]).astype(np.float32)
    ctx = felis.Context(0)
    leg = felis.Leg(ctx, s, seed=1)
    _check(felis, ctx, leg, s, frames, s.lambdas)
    ctx.close()


def test_ragged_leg_of_a_few_atoms():
    from paper_2603_22274_amd import felis
    s = gen.solvent_leg(config=77, n_waters=21, lattice_n=4, box_edge=13.5, n_lig=4, r_cut=6.0,
                        grid=(15, 15, 15), skin=0.25, sched='cfg0')
    ctx = felis.Context(0)
    leg = felis.Leg(ctx, s, windows=[3], seed=1)
    _check(felis, ctx, leg, s, np.stack([s.pos, s.pos - np.float32(6.7), s.pos + np.float32(13.4)]), s.lambdas)
    ctx.close()
