"""One call for a force evaluation gives what its four parts give one after the
other, to the last bit: integer force sums and energy sums in fixed point."""
import pytest
import torch

from paper_2603_22274_amd import gen

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize('make,windows', [(gen.config0, None), (gen.torsion_leg, None), (gen.small_complex, [0, 20, 41]),
                                          (gen.config1, None), (gen.config2, [3])])
@pytest.mark.parametrize('energy', [False, True])
def test_equals_its_parts(make, windows, energy):
    from paper_2603_22274_amd import felis
    s = make()
    ctx = felis.Context(0)
    legs = [felis.Leg(ctx, s, windows=windows, seed=5) for _ in range(2)]
    for k, v in enumerate((legs[0].x, legs[0].y, legs[0].z)):
        g = torch.Generator(device='cuda')
        g.manual_seed(k)
        v += 0.7 + 0.03 * torch.randn(v.shape, generator=g, device='cuda')
    for a, b in zip((legs[1].x, legs[1].y, legs[1].z), (legs[0].x, legs[0].y, legs[0].z)):
        a.copy_(b)
    for _ in range(2):                                   # a first call, which builds the lists, and another
        felis.forces_and_energy(ctx, legs[:1], energy=energy)
        felis.build_nlist(ctx, legs[1:])
        felis.nonbonded(ctx, legs[1:], energy)
        felis.pme(ctx, legs[1:], energy)
        felis.bonded(ctx, legs[1:], energy)
        for a, b in zip((legs[0].fx, legs[0].fy, legs[0].fz), (legs[1].fx, legs[1].fy, legs[1].fz)):
            assert torch.equal(a, b)
        if energy:
            assert torch.equal(legs[0].energy, legs[1].energy)
    ctx.device_check()
    ctx.close()
