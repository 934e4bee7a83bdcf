"""det grad y with one, odd and even numbers of time steps (its two buffers take
turns, one step has no interpolation of its own), against the FP64 oracle with the
bounds of the four-step test: 1e-5 relative, 1e-4 of J - 1."""
import numpy as np
import pytest

import oracle
from paper_2209_08189_amd import synth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


# tiles of 8 x 8 x 32 nodes, and a grid too small for them
@pytest.mark.parametrize("interp", ["cubic", "linear"])
@pytest.mark.parametrize("nt", [1, 2, 3, 5])
@pytest.mark.parametrize("shape", [(32, 16, 64), (32, 32, 16)])
def test_jacobian_of_any_number_of_steps(shape, nt, interp):
    from paper_2209_08189_amd.claire import Registration
    v = np.stack([0.4 * synth.smooth_random_field(shape, 80 + a, kmax=3.0) for a in range(3)]).astype(np.float32)
    o = oracle.Oracle(shape, nt=nt, interp=3 if interp == "cubic" else 1)
    o.set_images(np.zeros(shape), np.zeros(shape))
    o.set_velocity(v.astype(np.float64))
    want = o.jacobian_det()
    r = Registration(shape, nt=nt, interp=interp)
    r.set_velocity(torch.from_numpy(v).cuda())
    got, lo, hi = r.jacobian_det(want_field=True)
    r.close()
    got = got.double().cpu().numpy()
    assert (lo, hi) == (got.min(), got.max())
    assert np.linalg.norm(got - want) < 1e-5 * np.linalg.norm(want)
    assert np.linalg.norm(got - want) < 1e-4 * np.linalg.norm(want - 1.0)
