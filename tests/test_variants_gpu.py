"""Geometries of the gather kernel at the tiles and addresses that the automatic choice takes only for large
problems, forced here on small ones: 128-column tiles, rows further apart than 24-bit arithmetic, NaN between
the rows of X.  Small integers: every sum is exact and the comparison with the oracle is bit for bit."""
import numpy as np
import pytest

from oracle import c_oracle
from paper_2203_05016_amd import binding, synth
from gpu_util import announce, run_spmm, to_device, to_host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("V", [16, 32, 64])
@pytest.mark.parametrize("N,pad_ld,offset", [(8, 1, 0), (65, 0, 0), (127, 0, 1), (128, 3, 0), (129, 0, 0), (1023, 1, 3)])
def test_ragged_columns_in_wide_tiles_exact(V, N, pad_ld, offset):
    announce("wide tiles, rows", V, N, pad_ld, offset)
    p = synth.make_spmm(3 * V, 200, N, V, 0.6, seed=601 + N + V, integer=True, ragged=(V == 32))
    want, _ = c_oracle.spmm(p.W, p.mask, p.X)
    for out in ("float32", "float16"):
        got = run_spmm(p, out_dtype=out, tile_n=128, pad_ld=pad_ld, offset=offset, kernel=1).astype(np.float64)
        assert "<%d,128," % V in binding.last_kernel(), binding.last_kernel()
        assert np.array_equal(got, want), (out, np.argwhere(got != want)[:4])


@pytest.mark.parametrize("V", [16, 32, 64])
@pytest.mark.parametrize("batch,H,W", [(5, 2, 2), (40, 2, 2), (1, 1, 8), (9, 3, 3), (3, 5, 13), (20, 8, 8)])
def test_1x1_convolutions_in_wide_tiles_exact(V, batch, H, W):
    import torch
    announce("wide tiles, 1x1", V, batch, H, W)
    p = synth.make_conv(batch, 72, H, W, 2 * V, 1, 1, V, 0.6, seed=611 + H * W + V, integer=True)
    want, _ = c_oracle.conv2d(p.W, p.mask, p.conv["input"], 1, 1, (1, 1), (0, 0))
    A = binding.compress(p.W, p.mask, p.perm, V)
    A.set_tuning(0, 128)
    A.bind_device("cuda:0")
    for dt in (torch.float16, torch.float32):
        out = A.conv2d(to_device(p.conv["input"]), 1, 1, out_dtype=dt)
        torch.cuda.synchronize()
        assert "<%d,128," % V in binding.last_kernel(), binding.last_kernel()
        assert np.array_equal(to_host(out).astype(np.float64), want)


@pytest.mark.parametrize("V", [16, 32, 64])
@pytest.mark.parametrize("layout,batch,C,H,W,R,S,stride,pad", [
    ("NCHW", 2, 24, 8, 8, 3, 3, (1, 1), (1, 1)),
    ("NCHW", 3, 20, 9, 9, 3, 3, (1, 1), (1, 1)),
    ("NCHW", 2, 20, 5, 15, 3, 3, (2, 1), (1, 1)),
    ("NCHW", 2, 20, 9, 40, 5, 1, (1, 1), (2, 0)),
    ("CHWN", 9, 20, 7, 6, 3, 3, (2, 2), (1, 1)),
    ("CHWN", 23, 20, 5, 5, 5, 5, (1, 2), (2, 2)),
])
def test_convolutions_in_wide_tiles_exact(V, layout, batch, C, H, W, R, S, stride, pad):
    import torch
    announce("wide tiles, conv", V, layout, batch, H, W)
    p = synth.make_conv(batch, C, H, W, 2 * V, R, S, V, 0.6, seed=621 + C + W + V, stride=stride, pad=pad,
                        layout=layout, integer=True)
    want, _ = c_oracle.conv2d(p.W, p.mask, p.conv["input"], R, S, stride, pad, layout)
    A = binding.compress(p.W, p.mask, p.perm, V)
    A.set_tuning(1, 128)
    A.bind_device("cuda:0")
    for dt in (torch.float16, torch.float32):
        out = A.conv2d(to_device(p.conv["input"]), R, S, stride, pad, layout, out_dtype=dt)
        torch.cuda.synchronize()
        assert "<%d,128," % V in binding.last_kernel(), binding.last_kernel()
        assert np.array_equal(to_host(out).astype(np.float64), want)


@pytest.mark.parametrize("N,extra,base", [(73, 9, 0), (9, 1, 1), (72, 8, 1)])
def test_rows_far_apart_and_unaligned_exact(N, extra, base):
    """Rows 16 MiB apart whose starts or lengths are no multiples of 8: 64-bit addresses, element by element."""
    import torch
    announce("far rows", N, extra, base)
    p = synth.make_spmm(64, 40, N, 32, 0.5, seed=631 + N, integer=True)
    want, _ = c_oracle.spmm(p.W, p.mask, p.X)
    ld = (1 << 23) + extra
    A = binding.compress(p.W, p.mask, p.perm, p.V).bind_device("cuda:0")
    Xbuf = torch.full((p.K * ld + base,), float("nan"), dtype=torch.float16, device="cuda:0")
    Xd = Xbuf[base:].view(p.K, ld)[:, :N]
    Xd.copy_(to_device(p.X))
    Ybuf = torch.full((p.M * ld + base,), float("nan"), dtype=torch.float16, device="cuda:0")
    Yd = Ybuf[base:].view(p.M, ld)[:, :N]
    A.spmm(Xd, Yd)
    torch.cuda.synchronize()
    assert np.array_equal(to_host(Yd.contiguous()).astype(np.float64), want)
    assert torch.isnan(Ybuf[base:].view(p.M, ld)[:, N:N + 64]).all().item()
    del Xbuf, Ybuf, Xd, Yd
    torch.cuda.empty_cache()


@pytest.mark.parametrize("V", [16, 32, 64, 128])
@pytest.mark.parametrize("N,gap,base", [(1, 1, 0), (1, 7, 1), (2, 3, 0), (3, 1, 1), (4, 5, 1), (5, 8, 0), (6, 2, 1), (7, 1, 0), (7, 9, 3),
                                        (9, 2, 1), (13, 3, 0), (70, 2, 1)])
def test_what_lies_between_rows_is_never_mixed_in(V, N, gap, base):
    import torch
    announce("nan between rows", V, N, gap, base)
    p = synth.make_spmm(2 * V, 130, N, V, 0.5, seed=641 + N + V, integer=True)
    want, _ = c_oracle.spmm(p.W, p.mask, p.X)
    A = binding.compress(p.W, p.mask, p.perm, V).bind_device("cuda:0")
    Xbuf = torch.full((base + p.K * (N + gap) + 8,), float("nan"), dtype=torch.float16, device="cuda:0")
    Xd = Xbuf[base:base + p.K * (N + gap)].view(p.K, N + gap)[:, :N]
    Xd.copy_(to_device(p.X))
    for dt in (torch.float16, torch.float32):
        out = torch.empty((p.M, N), dtype=dt, device="cuda:0")
        A.spmm(Xd, out)
        torch.cuda.synchronize()
        assert np.array_equal(to_host(out).astype(np.float64), want)
