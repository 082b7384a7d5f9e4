"""The bonded forces of an MD step are those of the positions it starts from:
after one step fx/fy/fz equal the forces evaluated beforehand, on legs whose
chains span many waves of the integrator."""
import numpy as np
import pytest
import torch

from paper_2603_22274_amd import gen

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize('make', [gen.config2, gen.small_complex, gen.torsion_leg])
def test_step_forces_are_the_starting_positions_forces(make):
    from paper_2603_22274_amd import felis
    s = make()
    ctx = felis.Context(0)
    leg = felis.Leg(ctx, s, seed=5)
    for v in (leg.vx, leg.vy, leg.vz):
        v.normal_(0.0, 5.0)
    felis.forces_and_energy(ctx, [leg], energy=False)
    want = [t.clone() for t in (leg.fx, leg.fy, leg.fz)]
    felis.step(ctx, [leg], 1)
    ctx.device_check()
    for got, ref in zip((leg.fx, leg.fy, leg.fz), want):
        g, r = got.double() / felis.FORCE_SCALE, ref.double() / felis.FORCE_SCALE
        # the same FP32 terms, added per atom in FP32 here and per term in fixed point there:
        # a few roundings of 2^-24 of the atom's bonded forces (at most some 1e4 kcal/mol/A)
        err = float(((g - r).abs() - 1e-6 * r.abs()).max())
        assert err <= 2e-3, err
    ctx.close()
