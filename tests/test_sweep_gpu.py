"""Wide seeded sweeps of shapes, group sizes, sparsities, output types and kernels against the CPU
oracle: a few hundred small products and convolutions, and a few dozen products large enough for
many tiles and for the automatic choice to reach every kernel."""
import numpy as np
import pytest

from oracle import c_oracle
from paper_2203_05016_amd import binding, synth
from conftest import assert_within_scaled_tolerance
from gpu_util import announce, run_spmm

pytestmark = pytest.mark.gpu


def test_sweep_of_small_products():
    rng = np.random.default_rng(777)
    ran = 0
    for it in range(200):
        V = int(rng.choice([16, 32, 64, 128]))
        G = int(rng.integers(1, 30))
        K = int(rng.integers(1, 300)) * 8 if rng.random() < 0.8 else int(rng.integers(8, 1500))
        N = int(rng.integers(1, 200)) * 8 if rng.random() < 0.7 else int(rng.integers(1, 1200))
        sp = float(rng.choice([0.0, 0.3, 0.5, 0.75, 0.875, 0.9, 0.97]))
        kernel = int(rng.choice([0, 0, 1, 2, 3]))
        ragged = bool(rng.random() < 0.3)
        out_dtype = str(rng.choice(["float16", "float32"]))
        announce("small product", it, V, G, K, N, sp, kernel, ragged, out_dtype)
        p = synth.make_spmm(G * V, K, N, V, sp, seed=90000 + it, ragged=ragged)
        try:
            Y = run_spmm(p, out_dtype=out_dtype, kernel=kernel)
        except binding.ShflbwError:
            if kernel in (2, 3):   # a forced kernel may refuse a shape (no windowed layout, misaligned N)
                continue
            raise
        Yr, S = c_oracle.spmm(p.W, p.mask, p.X)
        assert_within_scaled_tolerance(Y, Yr, S, what="small product %d" % it)
        ran += 1
    assert ran >= 180


def test_sweep_of_convolutions():
    import torch
    rng = np.random.default_rng(778)
    ran = 0
    staged_4_byte = 0
    for it in range(100):
        V = int(rng.choice([32, 64, 128, 16]))
        G = int(rng.integers(1, 12))
        B = int(rng.integers(1, 20)); C = int(rng.integers(1, 70))
        H = int(rng.integers(3, 40)); Wd = int(rng.integers(3, 40))
        R = int(rng.choice([1, 3, 5])); S_ = int(rng.choice([1, 3])) if R != 5 else 5
        st = (int(rng.choice([1, 2])), int(rng.choice([1, 2])))
        pad = (int(rng.choice([0, 1, 2])), int(rng.choice([0, 1, 2])))
        layout = str(rng.choice(["NCHW", "CHWN"]))
        sp = float(rng.choice([0.0, 0.5, 0.75, 0.9]))
        kernel = int(rng.choice([0, 0, 2, 1]))
        out_dtype = str(rng.choice(["float16", "float32"]))
        if H + 2 * pad[0] < R or Wd + 2 * pad[1] < S_:
            continue
        announce("convolution", it, V, G, B, C, H, Wd, R, S_, st, pad, layout, sp, kernel, out_dtype)
        p = synth.make_conv(B, C, H, Wd, G * V, R, S_, V, sp, seed=95000 + it, stride=st, pad=pad,
                            layout=layout)
        g = p.conv
        A = binding.compress(p.W, p.mask, p.perm, p.V)
        A.set_tuning(kernel, 0)
        A.bind_device("cuda:0")
        x = torch.from_numpy(g["input"]).to("cuda:0")
        shape = (g["batch"], g["Cout"], g["Ho"], g["Wo"]) if layout == "NCHW" else \
            (g["Cout"], g["Ho"], g["Wo"], g["batch"])
        out = torch.full(shape, float("nan"), dtype=getattr(torch, out_dtype), device="cuda:0")
        try:
            A.conv2d(x, g["R"], g["S"], g["stride"], g["pad"], layout, out=out)
        except binding.ShflbwError:
            if kernel == 2:   # the staged kernel may refuse a box that does not fit
                continue
            raise
        torch.cuda.synchronize()
        staged_4_byte += "4-byte staging" in binding.last_kernel()
        want, sc = c_oracle.conv2d(p.W, p.mask, g["input"], g["R"], g["S"], g["stride"], g["pad"], layout)
        assert_within_scaled_tolerance(out.cpu().numpy(), want, sc, what="convolution %d" % it)
        ran += 1
    assert ran >= 90 and staged_4_byte >= 10


def test_sweep_of_large_products():
    rng = np.random.default_rng(4242)
    kernels = set()
    for it in range(40):
        V = int(rng.choice([16, 32, 64, 128]))
        G = int(rng.integers(8, 4096 // V + 1))
        K = int(rng.integers(16, 512)) * 8
        N = int(rng.integers(16, 520)) * 8
        sp = float(rng.choice([0.0, 0.5, 0.75, 0.8, 0.875]))
        kernel = int(rng.choice([0, 0, 2, 1]))
        ragged = bool(rng.random() < 0.25)
        out_dtype = str(rng.choice(["float16", "float32"]))
        announce("large product", it, V, G, K, N, sp, kernel, ragged, out_dtype)
        p = synth.make_spmm(G * V, K, N, V, sp, seed=97000 + it, ragged=ragged)
        try:
            Y = run_spmm(p, out_dtype=out_dtype, kernel=kernel)
        except binding.ShflbwError:
            if kernel == 2:
                continue
            raise
        name = binding.last_kernel()
        if "resident" not in name:
            kernels.add(name.split(",")[0])
        Yr, S = c_oracle.spmm(p.W, p.mask, p.X)
        assert_within_scaled_tolerance(Y, Yr, S, what="large product %d" % it)
    # the ring kernel and the gather kernel, every group size (test_resident_gpu.py is the resident slab's)
    for V in (16, 32, 64, 128):
        assert "shflbw_slab_kernel<%d" % V in kernels and "shflbw_gather_kernel<%d" % V in kernels, kernels
