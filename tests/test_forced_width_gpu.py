"""set_tuning(1, 0) leaves the width of the gather kernel's tiles to the library, which takes 128 columns where there are
thousands of tiles of many steps.  Small integers: both widths give the same bits."""
import numpy as np
import pytest

from oracle import c_oracle
from paper_2203_05016_amd import binding, synth
from gpu_util import announce, run_spmm, to_device, to_host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("V,N,wide", [(16, 8192, True), (32, 8192, True), (64, 8192, True), (32, 8191, True), (32, 64, False), (64, 72, False),
                                      (128, 8192, False)])
def test_width_of_linear_layers_is_automatic(V, N, wide):
    announce("width, linear", V, N)
    p = synth.make_spmm(32 * V if V < 128 else 512, 800, N, V, 0.1, seed=1501 + V, integer=True)
    got = run_spmm(p, out_dtype="float32" if V < 64 else "float16", kernel=1)
    assert "<%d,%d,whole tiles" % (V, 128 if wide else 64) in binding.last_kernel(), binding.last_kernel()
    want, _ = c_oracle.spmm(p.W, p.mask, p.X)
    if V >= 64:
        want = want.astype(np.float16)   # sums of more than 2048 round
    assert np.array_equal(got.astype(np.float64), want.astype(np.float64))


@pytest.mark.parametrize("layout,V,batch,side,wide", [("NCHW", 32, 24, 48, True), ("CHWN", 32, 48, 32, True), ("NCHW", 32, 2, 16, False)])
def test_width_of_convolutions_is_automatic(layout, V, batch, side, wide):
    import torch
    announce("width, convolution", layout, V, batch, side)
    C = 40
    p = synth.make_conv(batch, C, side, side, 8 * V, 3, 3, V, 0.05, seed=1511 + side, pad=(1, 1), integer=True, layout=layout)
    A = binding.compress(p.W, p.mask, p.perm, V).bind_device("cuda:0")
    x = to_device(p.conv["input"])
    got = {}
    for tile in (0, 64):
        A.set_tuning(1, tile)
        got[tile] = A.conv2d(x, 3, 3, (1, 1), (1, 1), layout=layout, out_dtype=torch.float32)
        torch.cuda.synchronize()
        assert "<%d,%d,whole tiles" % (V, 128 if wide and not tile else 64) in binding.last_kernel(), binding.last_kernel()
    assert torch.equal(got[0], got[64])
    if not wide:
        want, _ = c_oracle.conv2d(p.W, p.mask, p.conv["input"], 3, 3, (1, 1), (1, 1), layout)
        assert np.array_equal(to_host(got[0]).astype(np.float64), want)
