"""The Boresch restraint of a step is the one that the leg's descriptor names
when felis_step is called, as in a force evaluation: switched on, moved to other
anchors and switched off after the leg was set up, on anchors with and without
bonds."""
import ctypes as C

import numpy as np
import pytest

from tests._systems import point_charges

pytestmark = pytest.mark.gpu


def _system():
    rng = np.random.default_rng(11)
    box = np.array([24.0, 25.0, 26.0])
    cell = np.stack(np.meshgrid(*[np.arange(6)] * 3, indexing='ij'), -1).reshape(-1, 3)
    pos = (cell + 0.5) * box / 6 + rng.uniform(-0.4, 0.4, (216, 3))
    s = point_charges(pos, rng.normal(0, 0.3, 216), box, 9.0, 0.35, lig=(np.arange(216) < 20).astype(np.uint8))
    s.skin = 1.0
    s.lambdas = np.array([[1.0, 1.0, 1.0], [0.5, 1.0, 0.25], [0.0, 0.5, 1.0]])
    s.bonds = np.array([[0, 1], [1, 2], [100, 101]], np.int32)
    s.bond_k, s.bond_r0 = np.full(3, 200.0, np.float32), np.full(3, 4.0, np.float32)
    return s


def _restrain(leg, atoms):
    leg.s.has_restraint = int(atoms is not None)
    if atoms is not None:
        leg.s.restraint_atoms = (C.c_int32 * 6)(*atoms)
        leg.s.restraint_g0 = (C.c_double * 6)(8.0, 1.2, 1.4, 0.3, -0.7, 1.1)
        leg.s.restraint_k = (C.c_double * 6)(5.0, 40.0, 40.0, 20.0, 20.0, 20.0)


ANCHORS = {'free': (150, 163, 171, 8, 13, 17), 'bonded': (100, 101, 163, 0, 1, 2), 'one': (101, 163, 171, 8, 0, 17)}


@pytest.mark.parametrize('first', [None, 'free', 'bonded', 'one'])
@pytest.mark.parametrize('then', [None, 'free', 'bonded', 'one'])
def test_step_takes_the_descriptors_restraint(first, then):
    from paper_2603_22274_amd import felis
    s = _system()
    ctx = felis.Context(0)
    leg = felis.Leg(ctx, s, seed=5)
    _restrain(leg, ANCHORS.get(first))
    leg.set_positions(s.pos)                             # sets the leg up again
    _restrain(leg, ANCHORS.get(then))
    felis.forces_and_energy(ctx, [leg], energy=False)
    want = leg.forces().cpu().numpy()
    felis.step(ctx, [leg], 1)
    got = leg.forces().cpu().numpy()
    ctx.device_check()
    # the same FP32 terms, summed per atom in FP32 here and per term in fixed point there: a few
    # roundings of 2^-24 of an atom's bonded forces (at most some 1e3 kcal/mol/A)
    assert np.abs(got - want).max() <= 5e-4, np.abs(got - want).max()
    ctx.close()
