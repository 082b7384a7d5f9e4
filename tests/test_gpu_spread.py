"""Charge spreading by wide bricks (launches with many of them) on grids whose
edges leave partial bricks, with atoms whose stencils wrap at every face:
reciprocal energy and forces of single windows against the FP64 PME, to the
tolerances of the parity tests."""
import numpy as np
import pytest

from oracle import pairs as opairs
from oracle.ewald import PME
from tests._systems import point_charges

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize('n,box,grid,windows', [
    (300, (21.0, 20.0, 20.0), (20, 18, 16), 520), (900, (31.0, 20.0, 45.0), (36, 20, 50), 90),
    (41, (20.0, 20.0, 40.0), (15, 32, 48), 345), (1500, (33.0, 34.0, 32.0), (32, 32, 32), 257)])
def test_reciprocal_terms(n, box, grid, windows):
    from paper_2603_22274_amd import felis
    rng = np.random.default_rng(n)
    s = point_charges(rng.uniform(-0.5, 1.5, (n, 3)) * np.asarray(box), rng.normal(0, 0.4, n), box, 9.0, 0.35,
                      grid=grid, lig=(np.arange(n) < n // 10).astype(np.uint8))
    s.skin = 0.5
    bricks = windows * int(np.prod([-(-k // 16) for k in grid]))
    assert bricks >= 2048
    s.lambdas = np.stack([np.linspace(1, 0, windows), np.ones(windows), np.zeros(windows)], 1)
    ctx = felis.Context(0)
    leg = felis.Leg(ctx, s, list_cap=n + 8)
    felis.build_nlist(ctx, [leg], force=True)
    felis.nonbonded(ctx, [leg])
    before = leg.forces().cpu().numpy()
    felis.pme(ctx, [leg])
    f = leg.forces().cpu().numpy() - before
    E = leg.energy.cpu().numpy()
    ctx.device_check()
    pme = PME(s.box, s.grid, s.ewald_alpha)
    x = s.pos.astype(np.float64)
    for w in (0, 1, windows // 2, windows - 1):
        er, fr = pme.energy_forces(x, opairs.scaled_charges(s, s.lambdas[w][0]))
        assert abs(E[w, 4] - er) <= 1e-6 * abs(er), (w, E[w, 4], er)
        err = np.sqrt(((f[w] - fr) ** 2).sum() / (fr ** 2).sum())
        assert err <= 1e-5, (w, err)
    ctx.close()
