"""The staged convolution keeps the last plan it worked out.  A call must get what belongs to its own
matrix and geometry, whatever the call before it left there.  Small integers: every result is exact."""
import numpy as np
import pytest

from oracle import c_oracle
from paper_2203_05016_amd import binding, synth
from gpu_util import announce, to_device, to_host

pytestmark = pytest.mark.gpu


def _with_kept(p, kept):
    """Mask of p with kept[g] columns in group g, spread over the reduction."""
    K = p.mask.shape[1]
    mask = np.zeros_like(p.mask)
    for g, n in enumerate(kept):
        rows = p.perm[g * p.V:(g + 1) * p.V]
        mask[np.ix_(rows, np.linspace(0, K - 1, n).astype(int))] = 1
    return mask


@pytest.mark.parametrize("V,evenly,unevenly", [
    (32, (144, 144, 144, 144), (96, 192, 144, 144)),   # 9 steps of 16 in every group, then 6 / 12 / 9 / 9
    (16, (128, 128, 128, 128), (32, 224, 64, 192)),
])
def test_plan_of_another_matrix_of_the_same_size(V, evenly, unevenly):
    """Same shape and number of kept weights, other step counts per group; the handle of the first matrix
    is gone before the second is made, and usually its address is used again."""
    import torch
    announce("conv plan, other matrix", V)
    p = synth.make_conv(2, 64, 8, 9, 4 * V, 3, 3, V, 0.75, seed=901 + V, pad=(1, 1), integer=True)
    assert sum(evenly) == sum(unevenly)
    x = to_device(p.conv["input"])
    for kept in (evenly, unevenly, evenly):
        mask = _with_kept(p, kept)
        want, _ = c_oracle.conv2d(p.W, mask, p.conv["input"], 3, 3, (1, 1), (1, 1))
        A = binding.compress(p.W, mask, p.perm, V)
        A.set_tuning(2, 0)
        A.bind_device("cuda:0")
        got = A.conv2d(x, 3, 3, (1, 1), (1, 1), out_dtype=torch.float32)
        torch.cuda.synchronize()
        assert "shflbw_conv_kernel" in binding.last_kernel()
        assert np.array_equal(to_host(got).astype(np.float64), want), kept
        del A


@pytest.mark.parametrize("layout", ["NCHW", "CHWN"])
def test_plan_of_another_stride(layout):
    """Strides longer than the image are taken, and are not mistaken for others (1, 65537 for 2, 1)."""
    import torch
    announce("conv plan, other stride", layout)
    p = synth.make_conv(3, 16, 8, 9, 64, 3, 3, 32, 0.5, seed=931, pad=(1, 1), layout=layout, integer=True)
    x = to_device(p.conv["input"])
    A = binding.compress(p.W, p.mask, p.perm, 32)
    A.set_tuning(2, 0)
    A.bind_device("cuda:0")
    for stride in ((2, 1), (1, 65537), (2, 1), (65537, 1)):
        want, _ = c_oracle.conv2d(p.W, p.mask, p.conv["input"], 3, 3, stride, (1, 1), layout)
        got = A.conv2d(x, 3, 3, stride, (1, 1), layout, out_dtype=torch.float32)
        torch.cuda.synchronize()
        assert np.array_equal(to_host(got).astype(np.float64), want), stride
