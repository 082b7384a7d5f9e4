"""Pair forces where the pair kernel's special cases meet: clusters at the
faces of the box (an image on some axes, or one per pair in small boxes),
entries that lack an excluded pair or the atom itself, partly filled clusters,
lists that end inside a step, and half-clusters with and without LJ or ligand
atoms.  Against the FP64 oracle, to the force tolerance of the parity tests:
FP32 terms of a few roundings each, 1e-5 of the RMS force."""
import numpy as np
import pytest

from oracle import pairs as opairs
from tests._systems import point_charges

pytestmark = pytest.mark.gpu


def _system(n, box):
    rng = np.random.default_rng(n)
    box = np.asarray(box, np.float64)
    side = np.ceil((n / box.prod()) ** (1 / 3) * box).astype(int)
    while side.prod() < n:
        side += 1
    cell = np.stack(np.meshgrid(*[np.arange(k) for k in side], indexing='ij'), -1).reshape(-1, 3)
    cell = cell[rng.permutation(len(cell))[:n]]
    pos = (cell + 0.5) * box / side + rng.uniform(-0.25, 0.25, (n, 3)) + rng.integers(-1, 2, (n, 3)) * box
    lig = np.zeros(n, np.uint8)
    lig[: max(1, n // 40)] = 1
    eps = np.where(rng.uniform(size=n) < 0.5, 0.1, 0.0)
    s = point_charges(pos, rng.normal(0, 0.4, n), box, 9.0, 0.35, sigma=rng.uniform(2.2, 2.8, n), eps=eps, lig=lig)
    s.skin = 0.5
    s.lambdas = np.array([[1.0, 1.0, 0.0], [0.5, 0.4, 0.0], [0.0, 0.0, 0.0]])
    ex = [(i, i + k) for k in (1, 2) for i in range(n - k) if rng.uniform() < 0.5]
    s.excl = np.unique(np.asarray(ex, np.int32).reshape(-1, 2), axis=0)
    return s


@pytest.mark.parametrize('n,box', [(9, (20.0, 20.0, 20.0)), (61, (20.0, 22.0, 31.0)), (500, (24.0, 24.0, 24.0)),
                                   (1003, (33.0, 30.0, 46.0)), (2600, (48.0, 50.0, 47.0))])
def test_forces_against_the_oracle(n, box):
    from paper_2603_22274_amd import felis
    s = _system(n, box)
    ctx = felis.Context(0)
    leg = felis.Leg(ctx, s)
    felis.build_nlist(ctx, [leg], force=True)
    felis.nonbonded(ctx, [leg], energy=False)
    got = leg.forces().cpu().numpy()
    ctx.device_check()
    x = s.pos.astype(np.float64)
    for w, lam in enumerate(s.lambdas):
        ref = opairs.real_space(x, s, lam)[2] + opairs.exclusion_correction(x, s, lam)[1]
        err = np.sqrt(((got[w] - ref) ** 2).sum() / (ref ** 2).sum())
        assert err <= 1e-5, (w, err)
    ctx.close()
