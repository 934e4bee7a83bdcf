"""The convolution's tilings (brick depth, output tiles per workgroup, walked
tiles beyond the resident workgroups) at sizes that no brick divides, against
the FP64 layer oracle fed the same BF16 operands: products of BF16 values are
exact in FP32, so only the accumulation order differs (1e-5, as for every other
layer size).  An output that starts at any element holds the same values."""
import ctypes

import numpy as np
import pytest

import oracle
from oracle.net_oracle import bf16_round

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _bf16(a):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).cuda().to(torch.bfloat16)


def _rel(t, ref):
    a = t.detach().float().cpu().numpy().astype(np.float64)
    return float(np.linalg.norm(np.ravel(a - ref)) / np.linalg.norm(np.ravel(ref)))


# (36, 70, 130): 729 tiles of depth 4; (33, 60, 70): 680 of depth 2; (22, 50,
# 100) to 32 channels: 539 of two output tiles; (9, 17, 33) to 48 and 64: depth
# 1 with output groups; (1, 1, 1), (2, 9, 17): less than a brick
@pytest.mark.parametrize("shape,ci,co", [((36, 70, 130), 16, 16), ((33, 60, 70), 32, 16), ((22, 50, 100), 16, 32),
                                         ((9, 17, 33), 16, 48), ((9, 17, 33), 48, 64), ((1, 1, 1), 16, 16),
                                         ((2, 9, 17), 32, 32)])
def test_conv3_tilings_against_oracle(shape, ci, co):
    from paper_2209_08189_amd.claire import nn_conv3
    r = np.random.default_rng(sum(shape) + ci + co)
    x = bf16_round(r.standard_normal(shape + (ci,)))
    w = r.standard_normal((27, ci, co)) / np.sqrt(27 * ci)
    b = r.standard_normal(co)
    wt = torch.from_numpy(w.astype(np.float32)).cuda()
    out = nn_conv3(_bf16(x), wt, torch.from_numpy(b.astype(np.float32)).cuda(), act=0)
    assert _rel(out, oracle.conv3(x, bf16_round(w), b.astype(np.float32).astype(np.float64))) < 1e-5


@pytest.mark.parametrize("f32", [True, False])
def test_conv3_output_at_any_element(f32):
    from paper_2209_08189_amd import claire
    shape, ci, co = (3, 9, 20), 16, 32
    g = torch.Generator().manual_seed(3)
    x = torch.randn(shape + (ci,), generator=g).cuda().to(torch.bfloat16)
    w, b = torch.randn((27, ci, co), generator=g).cuda(), torch.randn(co, generator=g).cuda()
    ref = claire.nn_conv3(x, w, b, out_f32=f32)
    n = ref.numel()
    buf = torch.zeros(n + 8, dtype=ref.dtype, device="cuda")
    wpack = torch.empty(28 * ci * co * 2, dtype=torch.uint8, device="cuda")
    for off in (1, 2, 3):
        buf.zero_()
        at = ctypes.c_void_p(buf.data_ptr() + off * buf.element_size())
        st = claire.lib().cl_nn_conv3(claire._ptr(x), claire._ptr(w), claire._ptr(b), at, int(f32), *shape, ci, co, 1,
                                      0.2, 0, claire._ptr(wpack),
                                      ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
        assert st == 0
        assert torch.equal(buf[off:off + n], ref.reshape(-1))
        assert not buf[:off].any() and not buf[off + n:].any()


# less than a voxel tile of 16 x 4 x 4; ragged in every direction; several tiles
# per run with a short last run (1458 tiles over 512 workgroups, 96 over 28)
@pytest.mark.parametrize("shape,ci,co", [((1, 1, 1), 16, 16), ((5, 9, 17), 32, 48), ((2, 3, 40), 16, 64),
                                         ((36, 70, 130), 16, 16), ((23, 29, 30), 48, 96)])
def test_conv3_weight_gradient_tilings_against_oracle(shape, ci, co):
    from paper_2209_08189_amd.claire import nn_conv3_dw
    r = np.random.default_rng(sum(shape) + ci + co)
    x, dz = bf16_round(r.standard_normal(shape + (ci,))), bf16_round(r.standard_normal(shape + (co,)))
    gw, gb = nn_conv3_dw(_bf16(x), _bf16(dz))
    rw, rb = oracle.conv3_dw(x, dz)
    assert _rel(gw, rw) < 1e-5
    assert _rel(gb, rb) < 1e-5


@pytest.mark.parametrize("shift", [(1, 0), (0, 4), (3, 5)])
def test_conv3_weight_gradient_at_any_element(shift):
    from paper_2209_08189_amd.claire import nn_conv3_dw
    shape, ci, co = (7, 9, 40), 16, 32
    g = torch.Generator().manual_seed(4)
    t, s = [], []
    for c, off in zip((ci, co), shift):
        buf = torch.randn(shape[0] * shape[1] * shape[2] * c + 8, generator=g).cuda().to(torch.bfloat16)
        s.append(buf[off:off + buf.numel() - 8].view(shape + (c,)))
        t.append(s[-1].clone())
    for a, b in zip(nn_conv3_dw(*s), nn_conv3_dw(*t)):
        assert torch.equal(a, b)
