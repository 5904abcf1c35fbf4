"""NCHW convolutions with a stride of two along x, gathered in pairs of runs or held resident: runs that begin before the image and
end one or two columns after it, the narrowest image, images whose last run holds one column, every group size.  Small integers: the
comparison with the oracle is bit for bit."""
import numpy as np
import pytest

from oracle import c_oracle
from paper_2203_05016_amd import binding, synth
from gpu_util import announce, to_device, to_host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("fmt", ["f16", "bf16"])
@pytest.mark.parametrize("V,batch,C,H,W,M,R,S,stride_h,pad,sparsity,kernel", [
    (16, 3, 64, 15, 16, 64, 3, 3, 2, 1, 0.6, "gather"),      # the narrowest image, 8 columns of results
    (32, 2, 70, 17, 17, 64, 3, 3, 2, 1, 0.6, "gather"),      # one column in the last run
    (32, 2, 70, 20, 18, 64, 3, 3, 1, 0, 0.5, "gather"),      # no padding, another stride along y
    (64, 2, 80, 21, 24, 128, 3, 3, 2, 1, 0.7, "gather"),
    (64, 5, 256, 16, 31, 512, 1, 1, 2, 0, 0.5, "gather"),    # 1x1
    (128, 2, 48, 19, 33, 256, 3, 3, 2, 1, 0.5, "gather"),
    (128, 9, 40, 30, 29, 256, 1, 1, 2, 1, 0.3, "gather"),    # 1x1 with padding: a column of zeros on either side
    (32, 1, 33, 16, 40, 64, 5, 5, 2, 1, 0.5, "gather"),      # padding smaller than the kernel's half
    (16, 2, 40, 16, 19, 96, 3, 2, 2, 1, 0.8, "gather"),      # an even kernel: two columns after the image
    (32, 48, 64, 20, 130, 64, 3, 3, 2, 1, 0.5, "gather"),    # thousands of tiles
    (16, 24, 128, 32, 30, 512, 3, 3, 2, 1, 0.6, "resident"),
    (32, 32, 400, 33, 34, 2048, 1, 1, 2, 0, 0.3, "resident"),
    (16, 32, 64, 40, 17, 1024, 3, 3, 2, 1, 0.3, "resident"),
    (32, 16, 256, 28, 28, 512, 3, 3, 2, 1, 0.5, "conv"),     # too long to be resident, many groups that fetch much: staged
    (64, 6, 120, 39, 39, 512, 3, 3, 2, 1, 0.3, "conv"),      # the same for groups of 64
    (16, 6, 220, 34, 33, 64, 3, 3, 2, 1, 0.3, "conv"),       # few groups of 16 that keep most of a row
    (32, 12, 512, 33, 33, 160, 1, 1, 2, 0, 0.0, "conv"),      # 1x1, unpruned
    (16, 1, 1700, 17, 17, 64, 3, 3, 2, 1, 0.0, "gather"),    # would be staged, if a box of 1700 channels fitted the LDS
])
def test_stride_two_exact(V, batch, C, H, W, M, R, S, stride_h, pad, sparsity, kernel, fmt):
    import torch
    announce("strided runs", V, batch, C, H, W, M, R, S, stride_h, pad, fmt)
    p = synth.make_conv(batch, C, H, W, M, R, S, V, sparsity, seed=1801 + V + W, pad=(pad, pad), stride=(stride_h, 2), integer=True, fmt=fmt)
    want, _ = c_oracle.conv2d(p.W, p.mask, p.conv["input"], R, S, (stride_h, 2), (pad, pad))
    A = binding.compress(p.W, p.mask, p.perm, V).bind_device("cuda:0")
    x = to_device(p.conv["input"])
    flat = torch.full((x.numel() + 16,), float("nan"), dtype=x.dtype, device="cuda:0")
    flat[5:-11] = x.flatten()                               # no particular alignment, NaN right before and after
    guard = torch.full((want.size + 16,), float("nan"), dtype=x.dtype, device="cuda:0")
    out = guard[3:-13].view(want.shape)
    A.conv2d(flat[5:-11].view(x.shape), R, S, (stride_h, 2), (pad, pad), out=out)
    torch.cuda.synchronize()
    assert kernel in binding.last_kernel(), binding.last_kernel()
    rounded = torch.from_numpy(want).to(x.dtype).double().numpy()
    assert np.array_equal(to_host(out).astype(np.float64), rounded)
    assert bool(torch.isnan(guard[:3]).all()) and bool(torch.isnan(guard[-13:]).all())


def test_stride_two_of_more_groups_than_a_grid_has_rows():
    """65 536 groups, one more than the gather kernel takes, of a size that is never resident: staged."""
    import torch
    announce("strided runs, 65536 groups")
    p = synth.make_conv(1, 8, 1, 16, 65536 * 64, 1, 1, 64, 0.5, seed=1861, stride=(2, 2), integer=True)
    want, _ = c_oracle.conv2d(p.W, p.mask, p.conv["input"], 1, 1, (2, 2), (0, 0))
    A = binding.compress(p.W, p.mask, p.perm, 64).bind_device("cuda:0")
    got = A.conv2d(to_device(p.conv["input"]), 1, 1, (2, 2), (0, 0))
    torch.cuda.synchronize()
    assert "conv" in binding.last_kernel(), binding.last_kernel()
    assert np.array_equal(to_host(got).astype(np.float64), want)
