"""Reduced potentials that no free energy can be computed from are reported,
never answered: a NaN, or a sample that no sampled state can hold (+inf at all
of them), in the fused form, at its limit and in the general form, with and
without a workspace.  +inf at some of the states is an ordinary weight of zero."""
import numpy as np
import pytest
import torch

from oracle import mbar as ombar
from tests.test_gpu_mbar_sizes import _harmonic

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize('K,N,unsampled', [(2, 64, ()), (12, 96, ()), (17, 641, (16,)), (80, 2003, ()), (81, 2003, ()),
                                           (81, 2003, (7,)), (3, 65, (1, 2))])
@pytest.mark.parametrize('kind', ['nan', 'inf'])
@pytest.mark.parametrize('form', ['mbar', 'mbar_noalloc'])
def test_not_answered(K, N, unsampled, kind, form):
    from paper_2603_22274_amd import felis
    u, nk = _harmonic(K, N, set(unsampled), 1)
    if kind == 'nan':
        u[int(np.flatnonzero(nk)[-1]), N // 2] = np.nan
    else:
        u[nk > 0, N // 2] = np.inf
    ctx = felis.Context(0)
    with pytest.raises(felis.FelisError) as e:
        getattr(felis, form)(ctx, torch.as_tensor(u).cuda(), nk)
    ctx.close()
    assert e.value.code == felis.E_NOCONV


@pytest.mark.parametrize('K', [12, 80, 81])
def test_infinite_at_some_states_is_a_weight_of_zero(K):
    from paper_2603_22274_amd import felis
    u, nk = _harmonic(K, 25 * K, set(), 3)
    of = np.repeat(np.arange(K), nk)
    u[np.abs(np.arange(K)[:, None] - of[None]) > 6] = np.inf
    ctx = felis.Context(0)
    f, _ = felis.mbar(ctx, torch.as_tensor(u).cuda(), nk, tol=1e-12)
    ctx.close()
    W = ombar.weights(u, nk, f).sum(1)
    # as in the sizes' test: the last accepted change of f is at most tol x max|f|
    assert np.max(np.abs(W - 1.0)) <= 1e-11 * max(1.0, np.abs(f).max()) + 1e-13 * u.shape[1]


@pytest.mark.parametrize('K', [12, 81])
def test_a_gauge_state_without_weight_is_not_convergence(K):
    """The states' free energies lie so far from the first one's that it holds no weight at f = 0 and the
    Newton system vanishes: there is no step to take, which is not a step of zero."""
    from paper_2603_22274_amd import felis
    u, nk = _harmonic(K, 25 * K, set(), 4)
    u = u - 5000.0 * np.arange(K)[:, None]
    ctx = felis.Context(0)
    with pytest.raises(felis.FelisError) as e:
        felis.mbar(ctx, torch.as_tensor(u).cuda(), nk)
    ctx.close()
    assert e.value.code == felis.E_NOCONV
