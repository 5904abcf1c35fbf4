"""Convolutions gathered in runs of 8 along the innermost dimension, and products split over the
wavefronts of a workgroup.  Small integers: every sum is exact, so the comparison with the oracle is
bit for bit."""
import numpy as np
import pytest

from oracle import c_oracle
from paper_2203_05016_amd import binding, synth
from gpu_util import announce, run_spmm, to_device, to_host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kernel", [0, 1, 3])
@pytest.mark.parametrize("layout,batch,C,H,W,R,S,stride,pad,V", [
    ("NCHW", 2, 24, 8, 8, 3, 3, (1, 1), (1, 1), 32),     # one slot per row: shifted at both ends
    ("NCHW", 3, 20, 9, 9, 3, 3, (1, 1), (1, 1), 64),     # the second slot overlaps all but one column
    ("NCHW", 2, 20, 5, 15, 3, 3, (2, 1), (1, 1), 16),    # rows strided, columns not
    ("NCHW", 2, 20, 11, 10, 3, 3, (1, 1), (2, 0), 128),  # no column padding, 8 output columns, more row padding
    ("NCHW", 1, 20, 9, 16, 1, 5, (1, 1), (0, 1), 32),    # kernel wider than the slot's overlap
    ("NCHW", 2, 20, 9, 12, 5, 1, (1, 1), (2, 0), 32),
    ("NCHW", 5, 140, 6, 17, 1, 1, (1, 1), (1, 1), 32),   # 1x1 with padding: output rows and columns of zeros
    ("CHWN", 8, 24, 6, 5, 3, 3, (1, 1), (1, 1), 32),     # one slot of images
    ("CHWN", 9, 20, 7, 6, 3, 3, (2, 2), (1, 1), 64),     # the second slot overlaps all but one image
    ("CHWN", 23, 20, 5, 5, 5, 5, (1, 2), (2, 2), 16),
    ("CHWN", 16, 20, 4, 4, 1, 1, (2, 2), (0, 0), 128),
])
def test_convolution_in_runs_exact(kernel, layout, batch, C, H, W, R, S, stride, pad, V):
    import torch
    announce("conv runs", kernel, layout, batch, C, H, W, R, S, stride, pad, V)
    p = synth.make_conv(batch, C, H, W, 2 * V, R, S, V, 0.6, seed=501 + C + W + V, stride=stride, pad=pad,
                        layout=layout, integer=True)
    g = p.conv
    want, _ = c_oracle.conv2d(p.W, p.mask, g["input"], R, S, stride, pad, layout)
    A = binding.compress(p.W, p.mask, p.perm, V)
    A.set_tuning(kernel, 0)
    A.bind_device("cuda:0")
    flat = torch.full((g["input"].size + 1,), float("nan"), dtype=torch.float16, device="cuda:0")
    for base in (0, 1):   # NaN right before or right after the tensor; two bytes off alignment
        x = flat[base:base + g["input"].size].view(g["input"].shape)
        flat.fill_(float("nan"))
        x.copy_(to_device(g["input"]))
        for dt in (torch.float16, torch.float32):
            out = A.conv2d(x, R, S, stride, pad, layout, out_dtype=dt)
            torch.cuda.synchronize()
            if V != 16 or kernel:
                assert "shflbw_gather_kernel" in binding.last_kernel(), binding.last_kernel()
            assert np.array_equal(to_host(out).astype(np.float64), want)


def test_runs_and_staged_convolution_agree_on_bfloat16():
    """Both kernels on the same bfloat16 convolution, integers: the same bits; the shape's reduction is
    long enough for several batches of the gather list and for an uneven split of the k-steps."""
    import torch
    announce("conv runs, bf16")
    p = synth.make_conv(3, 70, 12, 14, 96, 3, 3, 32, 0.55, seed=601, pad=(1, 1), integer=True, fmt="bf16")
    A = binding.compress(p.W, p.mask, p.perm, 32).bind_device("cuda:0")
    x = to_device(p.conv["input"])
    got = {}
    for kernel in (0, 1, 2, 3):
        A.set_tuning(kernel, 0)
        got[kernel] = to_host(A.conv2d(x, 3, 3, (1, 1), (1, 1), out_dtype=torch.float32))
    for kernel in (0, 1, 3):
        assert np.array_equal(got[kernel], got[2])


@pytest.mark.parametrize("V,M,K,N", [
    (32, 64, 2048, 64),      # 2 tiles of 32 k-steps and more: split by 8
    (16, 48, 4096, 72),
    (64, 128, 600, 200),     # split by 4, fewer k-steps than wavefronts share evenly
    (128, 256, 400, 64),
    (32, 1024, 500, 1024),   # 512 tiles: split by 2
    (16, 640, 700, 1032),    # odd number of steps, ragged last tile
    (128, 1280, 300, 3000),
])
@pytest.mark.parametrize("out_dtype", ["float16", "float32"])
def test_split_products_exact(V, M, K, N, out_dtype):
    announce("split", V, M, K, N, out_dtype)
    p = synth.make_spmm(M, K, N, V, 0.45, seed=701 + N, integer=True, ragged=(V == 16))
    got = run_spmm(p, out_dtype=out_dtype)
    assert "split k-steps by" in binding.last_kernel(), binding.last_kernel()
    want, _ = c_oracle.spmm(p.W, p.mask, p.X)
    if out_dtype == "float16":
        want = want.astype(np.float16).astype(np.float64)   # sums of more than 2048 round
    assert np.array_equal(got.astype(np.float64), want)


@pytest.mark.parametrize("V", [16, 32, 64, 128])
@pytest.mark.parametrize("N,K", [(1, 1024), (2, 33), (3, 64), (5, 100), (7, 8), (7, 2), (1, 8), (1, 7)])
def test_few_columns_exact(V, N, K):
    """Rows of fewer than 8 columns: the last row's load would reach past X (K*N down to 8 and below)."""
    announce("few columns", V, N, K)
    p = synth.make_spmm(2 * V, K, N, V, 0.3, seed=801 + N + K, integer=True)
    want, _ = c_oracle.spmm(p.W, p.mask, p.X)
    for pad_ld, offset in ((0, 0), (3, 1)):
        for dt in ("float16", "float32"):
            assert np.array_equal(run_spmm(p, out_dtype=dt, pad_ld=pad_ld, offset=offset).astype(np.float64), want)
