"""<r, P r> of the inner CG as the transform's x1 pass forms it (Parseval over the
half spectrum).  On a constant template the zero-velocity Hessian is L_0, and one
inner step gives z = (<r, P r> / <P r, L_0 P r>) P r with L_0 P r = r: the
denominator is summed over the nodes, so z / P r is the ratio of the two sums, 1
but for rounding.  White noise fills every mode (a wrong weight on the planes k3 =
0 or n3 / 2, or a column past the last one, moves the ratio by over 1e-3); three
transforms of relative error <= 4 log2(N) eps enter, the first one squared."""
import math

import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.mark.parametrize("shape", [(16, 16, 16), (64, 32, 128), (128, 16, 32), (256, 32, 16), (512, 16, 32),
                                   (1024, 16, 16)])
def test_parseval_sum_is_that_over_the_nodes(shape):
    from paper_2209_08189_amd.claire import Registration
    g = torch.Generator().manual_seed(sum(shape))
    x = torch.randn((3,) + shape, generator=g).cuda()
    flat = torch.full(shape, 0.5, device="cuda")
    z = []
    for kw in ({"precond": "h0", "precond_inner": 1}, {}):
        r = Registration(shape, **kw)
        r.set_images(flat, flat)
        r.set_velocity(torch.zeros((3,) + shape, device="cuda"))
        z.append(r.precond(x).double().cpu())
        r.close()
    ratio = float((z[0] * z[1]).sum() / (z[1] * z[1]).sum())
    print("%s: ratio - 1 = %.2e" % (shape, ratio - 1))
    assert abs(ratio - 1) <= 16 * 2.0 ** -24 * math.log2(shape[0] * shape[1] * shape[2])


@pytest.mark.parametrize("shape", [(16, 32, 128), (32, 16, 256), (16, 16, 512), (16, 16, 1024)])
def test_residual_formed_by_the_row_pass(shape):
    """Inner steps whose residual the row pass forms while it reads (n3 >= 128),
    against the FP64 oracle: 1e-4 relative L2, as the applications at n3 <= 64; and
    r itself stays as it was."""
    import oracle
    from paper_2209_08189_amd import synth
    from paper_2209_08189_amd.claire import Registration
    m0 = np.float32(synth.trig_template(shape))
    x = np.float32(synth.random_field((3,) + shape, 95))
    o = oracle.Oracle(shape, nt=4, beta=5e-4)
    o.set_images(np.float64(m0), np.float64(m0))
    o.set_velocity(np.zeros((3,) + shape))
    o.set_precond(1, 4)
    want = np.asarray(o.precond(np.float64(x)))
    r = Registration(shape, precond="h0", precond_inner=4)
    m, xd = torch.from_numpy(m0).cuda(), torch.from_numpy(x).cuda()
    r.set_images(m, m)
    r.set_velocity(torch.zeros((3,) + shape, device="cuda"))
    got = r.precond(xd).double().cpu().numpy()
    r.close()
    e = np.linalg.norm(got - want) / np.linalg.norm(want)
    print("%s: rel %.2e" % (shape, e))
    assert e < 1e-4
    assert torch.equal(xd.cpu(), torch.from_numpy(x))


@pytest.mark.parametrize("shape", [(16, 16, 32), (16, 16, 128)])
def test_residual_at_any_alignment(shape):
    """A residual that starts at an odd element gives what an aligned copy gives."""
    from paper_2209_08189_amd import synth
    from paper_2209_08189_amd.claire import Registration
    m = torch.from_numpy(np.float32(synth.trig_template(shape))).cuda()
    n = 3 * shape[0] * shape[1] * shape[2]
    buf = torch.randn(n + 1, generator=torch.Generator().manual_seed(3)).cuda()
    x = buf[1:].view((3,) + shape)
    r = Registration(shape, precond="h0", precond_inner=3)
    r.set_images(m, m)
    r.set_velocity(torch.zeros((3,) + shape, device="cuda"))
    assert torch.equal(r.precond(x), r.precond(x.clone()))
    r.close()
