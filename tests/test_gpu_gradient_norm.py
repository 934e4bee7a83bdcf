"""||g|| summed by the quadrature that produces g: stored gradients, FD8 per node,
marching, more levels than one launch takes.  The products of FP32 values are
exact in FP64, so 3 n additions round to 3 n 2^-53 at most."""
import math

import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.mark.parametrize("shape,nt,lean,storage", [((32, 32, 32), 4, False, "f32"), ((16, 16, 32), 2, True, "f32"),
                                                   ((16, 32, 128), 4, False, "f32"), ((32, 16, 64), 8, False, "f16"),
                                                   ((16, 16, 64), 4, True, "f32")])
def test_norm_of_the_gradient(shape, nt, lean, storage):
    from paper_2209_08189_amd import synth
    from paper_2209_08189_amd.claire import Registration, query_workspace
    kw = dict(nt=nt, storage_state=storage, storage_adjoint=storage)
    if lean:
        kw["workspace_cap"] = query_workspace(shape, workspace_cap=1, **kw)
    n = shape[0] * shape[1] * shape[2]
    hv = (2 * math.pi) ** 3 / n
    gen = torch.Generator().manual_seed(sum(shape))
    v = np.float32(synth.trig_velocity(shape, 0.4)) + 0.01 * torch.randn((3,) + shape, generator=gen).numpy()
    m0 = torch.from_numpy(np.float32(synth.trig_template(shape))).cuda()
    r = Registration(shape, beta_v=1e-3, **kw)
    r.set_images(m0, (0.9 * m0 + 0.02).contiguous())
    r.set_velocity(torch.from_numpy(v).cuda())
    g, gn, J = r.gradient()
    g = g.cpu().numpy().astype(np.float64)
    want = math.sqrt(hv * (g ** 2).sum())
    print("%s: ||g|| %.1e" % (shape, gn / want - 1))
    assert abs(gn - want) <= 3 * n * 2.0 ** -53 * want
    r.close()
