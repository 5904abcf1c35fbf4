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
