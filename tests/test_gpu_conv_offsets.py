"""A convolution whose brick spans 4 GiB of its input, beyond 32-bit offsets: pieces of
the grid, which take 32-bit offsets, hold bitwise the same values away from the cuts."""
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def test_convolution_past_32_bit_offsets():
    from paper_2209_08189_amd.claire import nn_conv3
    D, H, W, ci, co = 3, 610, 600, 1024, 16
    assert (6 * H + 10) * W * ci * 2 >= 2 ** 32
    g = torch.Generator(device="cuda").manual_seed(1)
    x = torch.randn((D, H, W, ci), generator=g, device="cuda", dtype=torch.bfloat16)
    w = torch.randn((27, ci, co), generator=g, device="cuda") / (27 * ci) ** 0.5
    b = torch.randn(co, generator=g, device="cuda")
    whole = nn_conv3(x, w, b)
    for y0, y1 in ((0, 9), (300, 317), (601, 610)):
        lo, hi = max(y0 - 1, 0), min(y1 + 1, H)
        assert (10 * (hi - lo) + 10) * W * ci * 2 < 2 ** 32
        part = nn_conv3(x[:, lo:hi].contiguous(), w, b)
        assert torch.equal(part[:, y0 - lo:y1 - lo], whole[:, y0:y1])
