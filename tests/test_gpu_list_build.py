"""List build at the edges of its tiles: the exported pairs equal the canonical
list for odd numbers of clusters, partly filled clusters, one atom, dense
clumps (more candidates than one table window), boxes where each pair takes its
own image, and exclusions that reach far along the sorted order; with one and
with four waves a cluster pair (few and many pairs in the launch)."""
import numpy as np
import pytest
import torch

from oracle import pairs as opairs
from tests._systems import point_charges

pytestmark = pytest.mark.gpu


def _system(n, box, kind, r_cut=9.0, skin=1.0, windows=1):
    rng = np.random.default_rng(n)
    box = np.asarray(box, np.float64)
    if kind == 'clump':
        pos = np.mod(0.97 * box + rng.normal(0, 2.0, (n, 3)), box)         # across the faces
    else:
        pos = rng.uniform(-0.2, 1.2, (n, 3)) * box                         # beyond the box on either side
    s = point_charges(pos, rng.normal(0, 0.3, n), box, r_cut, 0.35)
    s.skin = skin
    s.lambdas = np.tile(s.lambdas, (windows, 1))
    # up to 8 exclusions an atom: three neighbours either side along the index, one anywhere
    ex = [(i, i + k) for k in (1, 2, 3) for i in range(n - k) if rng.uniform() < 0.7]
    far = rng.permutation(n)[: 2 * (n // 2)].reshape(-1, 2)
    ex += [tuple(sorted(p)) for p in far.tolist()]
    s.excl = np.unique(np.asarray(ex, np.int32).reshape(-1, 2), axis=0)
    return s


@pytest.mark.parametrize('n,box,kind,windows', [
    (1, (24.0, 24.0, 24.0), 'even', 2), (8, (24.0, 24.0, 24.0), 'even', 1), (9, (24.0, 24.0, 24.0), 'even', 3),
    (17, (24.0, 28.0, 41.0), 'clump', 1), (333, (20.5, 21.0, 30.0), 'even', 2), (1001, (31.0, 30.0, 45.0), 'even', 2),
    (4500, (40.0, 40.0, 40.0), 'clump', 1), (5005, (42.0, 37.0, 90.0), 'even', 60)])
def test_pairs_equal_the_canonical_list(n, box, kind, windows):
    from paper_2603_22274_amd import felis
    s = _system(n, box, kind, windows=windows)
    ctx = felis.Context(0)
    rng = np.random.default_rng(5)
    pos = (s.pos[None] + rng.normal(0, 0.05, (windows, n, 3))).astype(np.float32)
    leg = felis.Leg(ctx, s, positions=pos, list_cap=n + 8)
    felis.build_nlist(ctx, [leg], force=True)
    ctx.device_check()
    for w in sorted({0, windows - 1}):
        ref = opairs.neighbor_pairs(pos[w], s.box, s, s.r_list)
        got = felis.nlist_export_pairs(ctx, leg, w, cap=max(1024, len(ref) + 1024))
        assert got.shape == ref.shape and np.array_equal(got, ref), (w, got.shape, ref.shape)
    torch.cuda.synchronize()
    ctx.close()


@pytest.mark.parametrize('n,box', [(1200, (30.0, 30.0, 30.0)), (900, (90.0, 80.0, 85.0)), (8192, (90.0, 80.0, 85.0)),
                                   (12289, (44.0, 60.0, 52.0)), (10241, (95.0, 80.0, 85.0))])
def test_one_atom_beyond_half_the_skin_rebuilds_its_window(n, box):
    """The check of a call's first positions, for sizes on either side of its forms: the last atom, the first
    and one in the middle, each in a window of its own."""
    from paper_2603_22274_amd import felis
    s = _system(n, box, 'even', windows=4)
    ctx = felis.Context(0)
    leg = felis.Leg(ctx, s, list_cap=4096)
    felis.build_nlist(ctx, [leg], force=True)
    ctx.device_check()
    built = felis.leg_rebuilds(ctx, leg)
    x = leg.x.view(4, n)
    for w, a in enumerate((n - 1, 0, n // 2)):
        x[w, a] += 0.499 * s.skin
    felis.build_nlist(ctx, [leg])
    assert np.array_equal(felis.leg_rebuilds(ctx, leg), built)
    for w, a in enumerate((n - 1, 0, n // 2)):
        x[w, a] += 0.002 * s.skin
    felis.build_nlist(ctx, [leg])
    assert np.array_equal(felis.leg_rebuilds(ctx, leg) - built, [1, 1, 1, 0])
    felis.build_nlist(ctx, [leg])
    assert np.array_equal(felis.leg_rebuilds(ctx, leg) - built, [1, 1, 1, 0])
    pos = torch.stack([leg.x.view(4, n), leg.y.view(4, n), leg.z.view(4, n)], -1).cpu().numpy()
    ref = opairs.neighbor_pairs_tree(pos[0], s.box, s, s.r_list)
    assert np.array_equal(felis.nlist_export_pairs(ctx, leg, 0), ref)
    ctx.device_check()
    ctx.close()
