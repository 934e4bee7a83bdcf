"""The sum of a weight gradient's partials over 1 ... 129 runs of voxel tiles: below,
at and above the loads a wavefront has in flight and the run count from which 16
wavefronts share them.  Against the FP64 layer oracle fed the same BF16 operands,
1e-5 as for every other layer size (products of BF16 values are exact in FP32)."""
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


# tiles of 16 x 4 x 4 voxels along z, one per run (16 -> 16 has one channel pair)
@pytest.mark.parametrize("runs", [1, 3, 4, 5, 28, 29, 32, 33, 48, 127, 128, 129])
def test_sum_of_runs(runs):
    from paper_2209_08189_amd.claire import nn_conv3_dw
    shape, c = (4 * runs - 1, 3, 15), 16
    r = np.random.default_rng(runs)
    x, dz = (bf16_round(r.standard_normal(shape + (c,))) for _ in range(2))
    t = [torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).cuda().to(torch.bfloat16) for a in (x, dz)]
    for got, want in zip(nn_conv3_dw(*t), oracle.conv3_dw(x, dz)):
        got = got.cpu().numpy().astype(np.float64)
        assert np.linalg.norm(got.ravel() - want.ravel()) < 1e-5 * np.linalg.norm(want)
