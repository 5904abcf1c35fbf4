"""Rows of no particular alignment (linear layers whose token count, leading dimension or base is
not a multiple of 16 bytes; 1x1 convolutions on images of any size): slots of 8 columns, the last
one of a row overlapping the one before it.  Small integers, so that every result is exact and the
comparison with the oracle is bit for bit."""
import numpy as np
import pytest

from oracle import c_oracle
from paper_2203_05016_amd import binding, synth
from gpu_util import announce, run_spmm, to_device, to_host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("V", [16, 32, 64, 128])
@pytest.mark.parametrize("N,pad_ld,offset", [
    (8, 1, 0), (9, 0, 0), (15, 0, 1), (63, 0, 0), (64, 3, 0), (65, 0, 0), (71, 5, 3), (127, 0, 0), (513, 0, 1), (1023, 1, 0),
])
def test_ragged_columns_exact(V, N, pad_ld, offset):
    """One slot, a slot and one column, tiles of 64 columns one short / exact / one over, misaligned
    leading dimensions and bases; nothing outside the window is written (run_spmm checks it)."""
    announce("rows", V, N, pad_ld, offset)
    fmt = "bf16" if N % 3 == 0 else "f16"
    p = synth.make_spmm(3 * V, 200, N, V, 0.6, seed=301 + N + V, integer=True, ragged=(V == 32), fmt=fmt)
    want, _ = c_oracle.spmm(p.W, p.mask, p.X)
    for out in ("float32", "float16" if fmt == "f16" else "bfloat16"):
        got = run_spmm(p, out_dtype=out, pad_ld=pad_ld, offset=offset).astype(np.float64)
        exact = want if out != "bfloat16" else synth.bfloat16_bits_to_float32(synth.float32_to_bfloat16_bits(want.astype(np.float32)))
        assert np.array_equal(got, exact), (out, np.argwhere(got != exact)[:4])


@pytest.mark.parametrize("H,W", [(1, 8), (3, 3), (2, 5), (7, 7), (5, 13), (8, 8)])
@pytest.mark.parametrize("V,batch", [(16, 1), (32, 9), (64, 3), (128, 2)])
def test_1x1_convolution_of_odd_images_exact(H, W, V, batch):
    import torch
    announce("rows, 1x1", H, W, V, batch)
    p = synth.make_conv(batch, 72, H, W, 2 * V, 1, 1, V, 0.6, seed=401 + H * W + V, integer=True)
    want, _ = c_oracle.conv2d(p.W, p.mask, p.conv["input"], 1, 1, (1, 1), (0, 0))
    A = binding.compress(p.W, p.mask, p.perm, V).bind_device("cuda:0")
    flat = torch.full((p.conv["input"].size + 1,), float("nan"), dtype=torch.float16, device="cuda:0")
    for base in (0, 1):   # a tensor that starts two bytes off as well
        x = flat[base:base + p.conv["input"].size].view(p.conv["input"].shape)
        x.copy_(to_device(p.conv["input"]))
        for dt in (torch.float16, torch.float32):
            out = A.conv2d(x, 1, 1, out_dtype=dt)
            torch.cuda.synchronize()
            assert "shflbw_gather_kernel" in binding.last_kernel()
            assert np.array_equal(to_host(out).astype(np.float64), want)


@pytest.mark.parametrize("batch,H,W,V,C", [(136, 8, 8, 32, 40), (160, 7, 7, 64, 72), (1100, 3, 3, 16, 64)])
def test_1x1_convolution_of_many_images_exact(batch, H, W, V, C):
    """More than 128 blocks of column tiles, with and without a number that eight divides: each XCD takes a
    range of them."""
    import torch
    announce("rows, 1x1, many images", batch, H, W, V)
    p = synth.make_conv(batch, C, H, W, 2 * V, 1, 1, V, 0.5, seed=451 + V, integer=True)
    want, _ = c_oracle.conv2d(p.W, p.mask, p.conv["input"], 1, 1, (1, 1), (0, 0))
    A = binding.compress(p.W, p.mask, p.perm, V).bind_device("cuda:0")
    out = torch.full((batch, 2 * V, H, W), float("nan"), dtype=torch.float32, device="cuda:0")
    A.conv2d(to_device(p.conv["input"]), 1, 1, out=out)
    torch.cuda.synchronize()
    assert "split k-steps by 2" in binding.last_kernel() or batch == 1100
    assert np.array_equal(to_host(out).astype(np.float64), want)
