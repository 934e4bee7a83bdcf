"""A convolution's values do not depend on the brick that its grid takes: the sum of
an output runs over input chunks, then taps, in every variant.  Each plane of a grid
that takes one brick is bitwise that of the three planes around it taken as a grid of
their own, which takes another."""
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


# bricks of 2 x 2, 4 x 1, 2 x 1 and 1 x 1 (planes x output tiles) of 8 rows, then 4 x 1,
# 2 x 2, 2 x 1 and 1 x 1 of 4 rows for the whole grid; three planes take 1 x 1 of 8
@pytest.mark.parametrize("f32,transpose", [(True, False), (False, False), (False, True)])
@pytest.mark.parametrize("shape,ci,co", [((22, 50, 100), 32, 32), ((36, 70, 130), 16, 16), ((30, 30, 30), 64, 64),
                                         ((5, 33, 90), 64, 64), ((17, 23, 30), 64, 64),
                                         ((45, 17, 130), 16, 16), ((41, 9, 119), 32, 32), ((39, 25, 17), 64, 64),
                                         ((49, 25, 35), 16, 16), ((44, 11, 17), 64, 64), ((41, 3, 18), 64, 64)])
def test_planes_alone(shape, ci, co, f32, transpose):
    from paper_2209_08189_amd.claire import nn_conv3
    g = torch.Generator().manual_seed(sum(shape))
    x = torch.randn(shape + (co if transpose else ci,), generator=g).cuda().to(torch.bfloat16)
    w, b = torch.randn((27, ci, co), generator=g).cuda(), torch.randn(co, generator=g).cuda()
    kw = dict(out_f32=f32, transpose=transpose, act=0 if transpose else 1)
    bias = None if transpose else b
    whole = nn_conv3(x, w, bias, **kw)
    for z in sorted({0, shape[0] // 2, shape[0] - 2, shape[0] - 1} & set(range(shape[0]))):
        lo = max(z - 1, 0)
        assert torch.equal(nn_conv3(x[lo:z + 2].contiguous(), w, bias, **kw)[z - lo], whole[z])
