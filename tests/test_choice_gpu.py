"""What the automatic choice launches where the measured alternatives differ most: many column tiles whose
k-steps are not worth sharing between wavefronts, convolutions whose rows fill their slots badly.  The
results are exact whichever kernel runs (small integers)."""
import numpy as np
import pytest

from oracle import c_oracle
from paper_2203_05016_amd import binding, synth
from gpu_util import announce, run_spmm, to_device, to_host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("V,M,K,N,sparsity,shares", [
    (128, 256, 160, 64 * 512, 0.4, 2),      # 1024 tiles: shared
    (128, 256, 160, 64 * 560, 0.4, 1),      # 1120 tiles, V = 128: whole
    (64, 128, 256, 64 * 640, 0.5, 2),       # 1280 tiles of 8 k-steps
    (64, 128, 256, 64 * 704, 0.5, 1),       # 1408 tiles of 8
    (32, 64, 512, 64 * 704, 0.5, 2),        # 1408 tiles of 16
    (32, 64, 1024, 64 * 896 + 8, 0.5, 2),   # 1794 tiles of 32
    (64, 128, 1024, 64 * 896, 0.5, 1),      # 1792 tiles of 32, V = 64
    (16, 64, 512, 64 + 8, 0.9, 2),          # 8 tiles of 2
    (32, 64, 256, 64 + 8, 0.5, 4),          # 4 tiles of 4
    (16, 64, 512, 64 * 160, 0.9, 1),        # 640 tiles of 2, V = 16
    (32, 64, 512, 64 * 320, 0.9, 2),        # 640 tiles of 2
])
def test_k_steps_are_shared_where_that_pays(V, M, K, N, sparsity, shares):
    import torch
    announce("choice, splits", V, M, K, N)
    p = synth.make_spmm(M, K, N, V, sparsity, seed=951 + V, integer=True)
    A = binding.compress(p.W, p.mask, p.perm, V).bind_device("cuda:0")
    out = torch.empty((M, N), dtype=torch.float32, device="cuda:0")
    X = to_device(p.X)
    # rows of no particular alignment: the slab kernel is not in the choice
    flat = torch.empty(K * (N + 1), dtype=X.dtype, device="cuda:0").view(K, N + 1)[:, :N]
    flat.copy_(X)
    A.spmm(flat, out)
    torch.cuda.synchronize()
    name = binding.last_kernel()
    assert ("split k-steps by %d" % shares if shares > 1 else "whole tiles") in name, name
    want, _ = c_oracle.spmm(p.W, p.mask, p.X)
    assert np.array_equal(to_host(out).astype(np.float64), want)


@pytest.mark.parametrize("batch,H,W", [(1, 2, 4), (7, 3, 3), (5, 8, 1), (3, 1, 9), (70, 4, 5), (2, 61, 67), (513, 3, 3)])
def test_images_of_any_number_of_slots(batch, H, W):
    """One slot per image (8 positions), two (9), an exact number, and many images: the quotient that finds a
    slot's image, with streaming and with plain stores."""
    import torch
    announce("choice, slots", batch, H, W)
    p = synth.make_conv(batch, 24, H, W, 64, 1, 1, 32, 0.5, seed=971 + H * W, integer=True)
    want, _ = c_oracle.conv2d(p.W, p.mask, p.conv["input"], 1, 1, (1, 1), (0, 0))
    A = binding.compress(p.W, p.mask, p.perm, 32).bind_device("cuda:0")
    x = to_device(p.conv["input"])
    for dt in (torch.float16, torch.float32):
        out = torch.full((batch, 64, H, W), float("nan"), dtype=dt, device="cuda:0")
        A.conv2d(x, 1, 1, out=out)
        torch.cuda.synchronize()
        assert np.array_equal(to_host(out).astype(np.float64), want)


@pytest.mark.parametrize("V", [16, 32, 64, 128])
@pytest.mark.parametrize("batch,C,H,W", [(1, 40, 2, 2), (2, 64, 4, 1), (3, 96, 1, 4), (17, 200, 2, 2), (300, 64, 2, 2)])
def test_1x1_on_images_of_four_positions(V, batch, C, H, W):
    """Two images per lane, the second of which may not exist; NaN right before or after the tensor."""
    import torch
    announce("choice, four positions", V, batch, C, H, W)
    p = synth.make_conv(batch, C, H, W, 2 * V, 1, 1, V, 0.5, seed=981 + batch + V, integer=True)
    want, _ = c_oracle.conv2d(p.W, p.mask, p.conv["input"], 1, 1, (1, 1), (0, 0))
    A = binding.compress(p.W, p.mask, p.perm, V).bind_device("cuda:0")
    n = p.conv["input"].size
    flat = torch.full((n + 1,), float("nan"), dtype=torch.float16, device="cuda:0")
    for base in (0, 1):
        flat.fill_(float("nan"))
        x = flat[base:base + n].view(p.conv["input"].shape)
        x.copy_(to_device(p.conv["input"]))
        for dt in (torch.float16, torch.float32):
            buf = torch.full((batch * 2 * V * 4 + 8,), float("nan"), dtype=dt, device="cuda:0")
            out = buf[4:-4].view(batch, 2 * V, H, W)
            A.conv2d(x, 1, 1, out=out)
            torch.cuda.synchronize()
            assert "shflbw_gather_kernel" in binding.last_kernel()
            assert np.array_equal(to_host(out).astype(np.float64), want)
            assert bool(torch.isnan(buf[:4]).all()) and bool(torch.isnan(buf[-4:]).all())


@pytest.mark.parametrize("V,batch,C,sparsity,staged", [
    (32, 512, 192, 0.0, False),      # 256 tiles
    (16, 2048, 192, 0.0, True),
    (16, 2048, 192, 0.5, False),
    (64, 2048, 192, 0.0, True),
    (128, 2048, 192, 0.0, False),
])
def test_1x1_on_many_images_of_four_positions(V, batch, C, sparsity, staged):
    import torch
    announce("choice, many images of four", V, batch, sparsity)
    M = 8 * V
    p = synth.make_conv(batch, C, 2, 2, M, 1, 1, V, sparsity, seed=983 + V, integer=True)
    want, _ = c_oracle.conv2d(p.W, p.mask, p.conv["input"], 1, 1, (1, 1), (0, 0))
    A = binding.compress(p.W, p.mask, p.perm, V).bind_device("cuda:0")
    out = torch.full((batch, M, 2, 2), float("nan"), dtype=torch.float32, device="cuda:0")
    A.conv2d(to_device(p.conv["input"]), 1, 1, out=out)
    torch.cuda.synchronize()
    assert ("shflbw_conv_kernel" in binding.last_kernel()) == staged, binding.last_kernel()
    assert np.array_equal(to_host(out).astype(np.float64), want)


@pytest.mark.parametrize("V,side", [(16, 14), (32, 14)])
def test_input_box_beyond_the_lds_is_gathered_in_runs(V, side):
    """A density that would be staged, with too many channels for that: not the element-wise geometry."""
    import torch
    announce("choice, too many channels to stage", V, side)
    p = synth.make_conv(2, 2048, side, side, 2 * V, 3, 3, V, 0.0, seed=985 + V, integer=True)
    want, _ = c_oracle.conv2d(p.W, p.mask, p.conv["input"], 3, 3, (1, 1), (1, 1))
    A = binding.compress(p.W, p.mask, p.perm, V).bind_device("cuda:0")
    out = torch.full((2, 2 * V, side, side), float("nan"), dtype=torch.float32, device="cuda:0")
    A.conv2d(to_device(p.conv["input"]), 3, 3, (1, 1), (1, 1), out=out)
    torch.cuda.synchronize()
    # few tiles: the runs share their k-steps between wavefronts, the element-wise geometry never does
    assert "gather" in binding.last_kernel() and "split k-steps by" in binding.last_kernel(), binding.last_kernel()
    assert np.array_equal(to_host(out).astype(np.float64), want)


@pytest.mark.parametrize("layout,V,batch,C,side,C_out,sparsity,staged", [
    ("NCHW", 32, 8, 64, 16, 64, 0.0, False),      # full runs
    ("NCHW", 32, 8, 64, 9, 64, 0.5, True),        # one element in the last run
    ("NCHW", 32, 8, 64, 9, 64, 0.75, False),
    ("NCHW", 32, 8, 64, 28, 64, 0.5, False),      # few groups
    ("NCHW", 32, 8, 64, 28, 256, 0.5, True),      # eight groups fetch every kept row
    ("NCHW", 32, 8, 64, 14, 256, 0.5, True),
    ("NCHW", 32, 8, 64, 12, 256, 0.5, False),
    ("NCHW", 16, 8, 64, 9, 64, 0.8, True),
    ("NCHW", 16, 8, 64, 14, 64, 0.8, False),
    ("NCHW", 16, 8, 64, 17, 64, 0.7, True),
    ("NCHW", 16, 8, 64, 20, 64, 0.65, False),
    ("NCHW", 16, 8, 32, 28, 64, 0.5, False),
    ("NCHW", 16, 8, 32, 28, 256, 0.5, True),
    ("NCHW", 64, 8, 64, 9, 64, 0.0, False),
    ("CHWN", 16, 9, 64, 6, 64, 0.5, True),        # one image in the last run
    ("CHWN", 16, 17, 64, 6, 64, 0.5, False),
    ("CHWN", 32, 17, 64, 6, 64, 0.5, True),
    ("CHWN", 32, 10, 64, 6, 64, 0.0, False),
])
def test_convolutions_are_staged_where_runs_are_badly_filled(layout, V, batch, C, side, C_out, sparsity, staged):
    import torch
    announce("choice, runs", layout, V, batch, side, C_out, sparsity)
    p = synth.make_conv(batch, C, side, side, C_out, 3, 3, V, sparsity, seed=987 + V + side, integer=True)
    want, _ = c_oracle.conv2d(p.W, p.mask, p.conv["input"], 3, 3, (1, 1), (1, 1))
    A = binding.compress(p.W, p.mask, p.perm, V).bind_device("cuda:0")
    x = to_device(p.conv["input"])
    if layout == "CHWN":
        x = x.permute(1, 2, 3, 0).contiguous()
    got = A.conv2d(x, 3, 3, (1, 1), (1, 1), layout=layout, out_dtype=torch.float32)
    torch.cuda.synchronize()
    assert ("shflbw_conv_kernel" in binding.last_kernel()) == staged, binding.last_kernel()
    if layout == "CHWN":
        got = got.permute(3, 0, 1, 2)
    assert np.array_equal(to_host(got.contiguous()).astype(np.float64), want)
