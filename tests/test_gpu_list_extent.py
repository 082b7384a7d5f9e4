"""Lists of sparse systems in large boxes, where the 16 atoms of a cluster pair
lie hundreds of Angstrom apart: every pair just inside r_list is listed, however
far from the pair's first atom it lies."""
import numpy as np
import pytest

from oracle import pairs as opairs
from tests._systems import point_charges

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize('n,edge,windows', [(240, 700.0, 1), (1000, 2000.0, 1), (4000, 4000.0, 1), (1000, 3000.0, 300),
                                            (2000, 8000.0, 1)])
def test_pairs_just_inside_the_list_radius(n, edge, windows):
    from paper_2603_22274_amd import felis
    rng = np.random.default_rng(n)
    box = np.full(3, edge)
    a = rng.uniform(0.0, 1.0, (n // 2, 3)) * box
    d = rng.normal(size=(n // 2, 3))
    d /= np.linalg.norm(d, axis=1, keepdims=True)
    # a partner each, from just inside r_list (by more than FP32 positions are apart) to well inside
    b = a + d * (10.0 - np.geomspace(2e-3, 1.0, n // 2))[:, None]
    s = point_charges(np.concatenate([a, b])[rng.permutation(n)], rng.normal(0, 0.3, n), box, 9.0, 0.35)
    s.skin = 1.0
    s.lambdas = np.tile(s.lambdas, (windows, 1))
    ctx = felis.Context(0)
    leg = felis.Leg(ctx, s, list_cap=64)
    felis.build_nlist(ctx, [leg], force=True)
    ctx.device_check()
    for w in sorted({0, windows - 1}):
        ref = opairs.neighbor_pairs(s.pos, s.box, s, s.r_list)
        got = felis.nlist_export_pairs(ctx, leg, w)
        assert len(ref) >= n // 4
        assert got.shape == ref.shape and np.array_equal(got, ref), (w, got.shape, ref.shape)
    ctx.close()
