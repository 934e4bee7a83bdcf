"""Sources of later groups of time levels: one to five levels past the first five, in
every storage, against one level at a time (lean layout).  The operations of a node are
the same: results are equal."""
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.mark.parametrize("state,adjoint", [("f32", "f32"), ("f16", "f16"), ("f16", "bf16"), ("bf16", "bf16")])
@pytest.mark.parametrize("nt", [5, 6, 7, 8, 9, 10])
def test_groups_equal_single_levels(nt, state, adjoint):
    from paper_2209_08189_amd.claire import Registration, query_workspace
    shape, kw = (32, 16, 64), dict(nt=nt, storage_state=state, storage_adjoint=adjoint)
    g = torch.Generator().manual_seed(nt)
    m0, m1 = (torch.rand(shape, generator=g).cuda() for _ in range(2))
    v, vt = (0.1 * torch.randn((3,) + shape, generator=g).cuda() for _ in range(2))
    out = []
    for cap in (0, query_workspace(shape, workspace_cap=1, **kw)):
        r = Registration(shape, workspace_cap=cap, **kw)
        assert r.layout() == (1 if cap else 0)
        r.set_images(m0, m1)
        r.set_velocity(v)
        out.append((r.gradient()[0], r.hessian_matvec(vt)))
        r.close()
    assert torch.equal(out[0][0], out[1][0])
    assert torch.equal(out[0][1], out[1][1])
