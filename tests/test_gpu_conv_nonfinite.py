"""Weight gradient of operands with a value that is not finite: it reaches the taps
whose products it takes part in and no others (a voxel next to a face is outside the
grid for some taps).  The other sums are those of the FP64 oracle to the rounding of
n FP32 additions, n 2^-24 of the sum of magnitudes."""
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


# corners, faces, edges and the inside; whole tiles of 16 x 4 x 4 voxels and ragged
# ones in every direction; several tiles per run
@pytest.mark.parametrize("operand", ["x", "dz"])
@pytest.mark.parametrize("shape", [(4, 4, 16), (8, 8, 32), (6, 8, 32), (5, 7, 19), (1, 2, 1), (2, 1, 33)])
@pytest.mark.parametrize("at", [(0, 0, 0), (-1, -1, -1), (0, -1, 0), (-1, 0, -1), (0.5, 0.5, 0), (0.5, 0.5, -1),
                                (0.5, 0, 0.5), (0.5, -1, 0.5), (0, 0.5, 0.5), (-1, 0.5, 0.5), (0.5, 0.5, 0.5)])
def test_weight_gradient_of_an_infinite_voxel(shape, at, operand):
    check(shape, at, operand, 16, 32)


@pytest.mark.parametrize("operand", ["x", "dz"])
def test_weight_gradient_of_an_infinite_voxel_in_a_long_run(operand):
    check((20, 30, 90), (-1, -1, -1), operand, 96, 48)


def check(shape, at, operand, ci, co):
    from paper_2209_08189_amd.claire import nn_conv3_dw
    r = np.random.default_rng(sum(shape))
    x = bf16_round(r.standard_normal(shape + (ci,)))
    dz = bf16_round(r.standard_normal(shape + (co,)))
    p = tuple(n // 2 if a == 0.5 else a % n for a, n in zip(at, shape))
    (x if operand == "x" else dz)[p + (3,)] = np.inf
    t = [torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).cuda().to(torch.bfloat16) for a in (x, dz)]
    n = shape[0] * shape[1] * shape[2]
    with np.errstate(invalid="ignore"):
        want, size = oracle.conv3_dw(x, dz), oracle.conv3_dw(np.abs(x), np.abs(dz))
    for got, w, s in zip(nn_conv3_dw(*t), want, size):
        got, w, s = got.cpu().numpy().ravel(), w.ravel(), s.ravel()
        ok = np.isfinite(w)
        assert np.array_equal(np.isfinite(got), ok)
        assert np.all(np.abs(got[ok] - w[ok]) <= n * 2.0 ** -24 * s[ok])
