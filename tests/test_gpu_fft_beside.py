"""The transform that runs beside a large pair kernel (smaller workgroups in
fewer registers) gives an MD step the forces that the plain one gives a force
evaluation: whole planes in LDS and one pass per axis, ragged grids."""
import numpy as np
import pytest

from tests._systems import point_charges

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize('n,box,grid,windows', [(500, (24.0, 23.0, 25.0), (20, 18, 24), 200),
                                                (1003, (33.0, 34.0, 30.0), (96, 72, 20), 101),
                                                (777, (30.0, 30.0, 30.0), (75, 128, 15), 127)])
def test_step_forces_equal_a_force_evaluation(n, box, grid, windows):
    from paper_2603_22274_amd import felis
    rng = np.random.default_rng(n)
    box = np.asarray(box)
    side = int(np.ceil(n ** (1 / 3)))
    cell = np.stack(np.meshgrid(*[np.arange(side)] * 3, indexing='ij'), -1).reshape(-1, 3)[:n]
    pos = (cell + 0.5) * box / side + rng.uniform(-0.3, 0.3, (n, 3))
    s = point_charges(pos, rng.normal(0, 0.4, n), box, 9.0, 0.35, grid=grid, lig=(np.arange(n) < 40).astype(np.uint8))
    s.skin = 0.5
    s.lambdas = np.stack([np.linspace(1, 0, windows), np.ones(windows), np.zeros(windows)], 1)
    assert windows * -(-n // 8) >= 4 * 3072            # pair workgroups of four clusters
    ctx = felis.Context(0)
    leg = felis.Leg(ctx, s, seed=5)
    felis.forces_and_energy(ctx, [leg], energy=False)
    want = leg.forces().cpu().numpy()
    felis.step(ctx, [leg], 1)
    got = leg.forces().cpu().numpy()
    ctx.device_check()
    # a trajectory does not depend on the batch it runs in, so not on the launch's size either
    assert np.array_equal(got, want), np.abs(got - want).max()
    ctx.close()
