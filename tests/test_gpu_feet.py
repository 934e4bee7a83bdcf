"""The feet of one kernel per velocity against their steps taken one by one:
predictor displacement, velocity interpolated there (cl_interp), corrector.
The steps round the same operations in FP32, so the results are equal."""
import math

import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


# (16, 16, 16): no tiles; voxels: the largest displacement of a time step.
# rough: independent nodes, so that no tile's stencils fit its box; mixed: a
# single rough node per tile column in a smooth field.
@pytest.mark.parametrize("interp", ["cubic", "linear"])
@pytest.mark.parametrize("kind", ["smooth", "rough", "mixed"])
@pytest.mark.parametrize("shape", [(16, 16, 16), (16, 16, 32), (64, 16, 32), (32, 64, 128)])
def test_feet_are_predictor_interpolation_corrector(shape, kind, interp):
    from paper_2209_08189_amd import claire
    nt = 4
    r = claire.Registration(shape, nt=nt, interp=interp)
    g = torch.Generator().manual_seed(7 + sum(shape))
    h = [torch.tensor(2.0 * math.pi / n, dtype=torch.float32).cuda() for n in shape]
    if kind == "rough":
        v = torch.rand((3,) + shape, generator=g) * 2 - 1
    else:
        x = [2 * math.pi * torch.arange(n, dtype=torch.float32) / n for n in shape]
        w = torch.sin(x[0])[:, None, None] * torch.cos(x[1])[None, :, None] * torch.cos(x[2])[None, None, :]
        v = torch.stack([w, torch.roll(w, 3, 1), torch.roll(w, 5, 2)])
    v = (v * (1.4 * nt * float(max(h)))).cuda()
    if kind == "mixed":
        v[:, 5, 9, ::64] += 40.0 * nt * float(max(h))
    v = v.contiguous()
    r.set_images(torch.rand(shape, generator=g).cuda(), torch.rand(shape, generator=g).cuda())
    r.set_velocity(v)
    r.gradient(want_g=False)
    dt = 1.0 / nt
    for which, a in ((claire.FIELD_FEET_F, -dt), (claire.FIELD_FEET_B, dt)):
        pred = torch.stack([(a * v[c]) / h[c] for c in range(3)])
        vi = torch.stack([r.interp(v[c].contiguous(), pred) for c in range(3)])
        ref = torch.stack([(0.5 * a * (v[c] + vi[c])) / h[c] for c in range(3)])
        assert torch.equal(r.field(which), ref)
    # the tile boxes that come with the feet: a step with them equals an
    # interpolation that finds its own
    m1 = r.interp(r.field(claire.FIELD_STATE, 0), r.field(claire.FIELD_FEET_F))
    assert torch.equal(r.field(claire.FIELD_STATE, 1), m1)
