"""The forms of the reciprocal part that only differ in how a launch is divided
agree to the last bit: 32 lines a workgroup beside a large pair kernel and by
themselves, wide and small spreading bricks, a window in a large batch and with
its partner alone; grids with partial bricks, windows with a grid of their own."""
import numpy as np
import pytest
import torch

from tests._systems import point_charges

pytestmark = pytest.mark.gpu


def _system(n, box, grid, windows):
    rng = np.random.default_rng(n)
    box = np.asarray(box)
    side = int(np.ceil(n ** (1 / 3)))
    cell = np.stack(np.meshgrid(*[np.arange(side)] * 3, indexing='ij'), -1).reshape(-1, 3)[:n]
    pos = (cell + 0.5) * box / side + rng.uniform(-0.3, 0.3, (n, 3)) - 0.2 * box      # beyond the faces
    s = point_charges(pos, rng.normal(0, 0.4, n), box, 9.0, 0.35, grid=grid, lig=(np.arange(n) < 40).astype(np.uint8))
    s.skin = 0.5
    s.lambdas = np.stack([np.linspace(1, 0, windows), np.ones(windows), np.zeros(windows)], 1)
    return s


@pytest.mark.parametrize('n,box,grid,windows', [(1003, (33.0, 34.0, 30.0), (96, 72, 20), 141),
                                                (777, (30.0, 30.0, 30.0), (75, 128, 15), 185)])
def test_step_and_force_evaluation_at_32_lines(n, box, grid, windows):
    from paper_2603_22274_amd import felis
    s = _system(n, box, grid, windows)
    npair, chunks = (windows + 1) // 2, [-(-k // 32) for k in grid]
    # x, y and z passes at 32 lines, beside a pair kernel of 3,072 workgroups or more
    assert min(npair * grid[2] * chunks[1], npair * grid[2] * chunks[0], npair * grid[1] * chunks[0]) >= 4096
    assert windows * -(-n // 8) >= 4 * 3072
    ctx = felis.Context(0)
    leg = felis.Leg(ctx, s, seed=5)
    felis.forces_and_energy(ctx, [leg], energy=False)
    want = leg.forces().cpu().numpy()
    felis.step(ctx, [leg], 1)
    got = leg.forces().cpu().numpy()
    ctx.device_check()
    assert np.array_equal(got, want), np.abs(got - want).max()
    ctx.close()


@pytest.mark.parametrize('n,box,grid,windows', [
    (1003, (33.0, 34.0, 30.0), (96, 72, 20), 141), (300, (21.0, 20.0, 20.0), (20, 18, 16), 521),
    (900, (31.0, 20.0, 45.0), (36, 20, 50), 91), (1500, (33.0, 34.0, 32.0), (32, 32, 32), 257)])
@pytest.mark.parametrize('npt', [False, True])
def test_a_window_alone_and_in_a_large_batch(n, box, grid, windows, npt):
    from paper_2603_22274_amd import felis
    s = _system(n, box, grid, windows)
    bricks = int(np.prod([-(-k // 16) for k in grid]))
    assert windows * bricks >= 2048 > 2 * bricks
    ctx = felis.Context(0)

    def reciprocal(which):
        leg = felis.Leg(ctx, s, windows=which, pressure_bar=1.0 if npt else 0.0)
        felis.build_nlist(ctx, [leg], force=True)
        felis.pme(ctx, [leg])
        return torch.stack([leg.fx, leg.fy, leg.fz]), leg.energy[:, 4].clone()

    f, e = reciprocal(list(range(windows)))
    # windows 2p and 2p + 1 share a complex grid, so a pair is taken alone; the last one has a grid to itself
    for which in ([0, 1], [windows // 4 * 2, windows // 4 * 2 + 1], [windows - 1]):
        g, d = reciprocal(which)
        assert torch.equal(f[:, which], g) and torch.equal(e[which], d), which
    ctx.device_check()
    ctx.close()
