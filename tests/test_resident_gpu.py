"""The slab kernel with a resident slab, as the automatic choice launches it: row groups that end at any step of four and at any
of a load's sixteen, more of them than wavefronts and fewer, unequal ones, groups without columns; columns at and beside the edges of
a tile, rows of no alignment and rows of images; the longest reduction.  Small integers: every sum is exact in 32 bits, and the
comparison with the oracle is bit for bit."""
import numpy as np
import pytest

from oracle import c_oracle
from paper_2203_05016_amd import binding, synth
from gpu_util import announce, run_spmm, to_device, to_host

pytestmark = pytest.mark.gpu


def _rounded(want, dtype):
    import torch
    return want if dtype == "float32" else torch.from_numpy(want).to(getattr(torch, dtype)).double().numpy()


@pytest.mark.parametrize("fmt", ["f16", "bf16"])
@pytest.mark.parametrize("V,G,K,N,sparsity,ragged", [
    (16, 256, 1024, 4096, 0.75, False),
    (16, 128, 1278, 3001, 0.70, True),     # the longest reduction; rows of no alignment, the last tile of 57 columns
    (16, 200, 300, 8160, 0.40, True),      # 8 wavefronts; the last tile of 32 columns
    (32, 128, 1024, 8192, 0.75, False),
    (32, 128, 1000, 8104, 0.75, True),     # rows of no whole blocks, the last tile of 40 columns
    (32, 96, 1278, 4097, 0.50, False),     # the last slot one column on from the one before
    (32, 100, 638, 6007, 0.50, True),      # the longest for 8 wavefronts
    (32, 100, 639, 6007, 0.50, True),      # the shortest for 16
    (64, 64, 1024, 8191, 0.50, True),
    (64, 64, 1278, 8189, 0.50, False),
    (128, 33, 1024, 8191, 0.30, True),     # two items of a group, an odd number of groups
])
def test_resident_slab_exact(V, G, K, N, sparsity, ragged, fmt):
    announce("resident slab", V, G, K, N, ragged, fmt)
    p = synth.make_spmm(G * V, K, N, V, sparsity, seed=1701 + N + V, integer=True, ragged=ragged, fmt=fmt)
    want, _ = c_oracle.spmm(p.W, p.mask, p.X)
    for out in ("float32", "bfloat16" if fmt == "bf16" else "float16"):
        got = run_spmm(p, out_dtype=out).astype(np.float64)
        assert "resident in %d wavefronts" % (8 if V >= 64 or K <= 638 else 16) in binding.last_kernel(), binding.last_kernel()
        assert np.array_equal(got, _rounded(want, out)), np.argwhere(got != _rounded(want, out))[:4]


def test_resident_slab_writes_its_window_only():
    """Padded leading dimensions and a base of no alignment: nothing outside the results is written (run_spmm looks)."""
    announce("resident slab, window")
    p = synth.make_spmm(128 * 32, 1024, 4090, 32, 0.75, seed=1711, integer=True)
    want, _ = c_oracle.spmm(p.W, p.mask, p.X)
    got = run_spmm(p, out_dtype="float32", pad_ld=13, offset=3)
    assert "resident" in binding.last_kernel(), binding.last_kernel()
    assert np.array_equal(got.astype(np.float64), want)


@pytest.mark.parametrize("V,batch,C,H,W,M", [(16, 32, 512, 7, 7, 2048), (32, 33, 640, 13, 13, 1024), (16, 32, 256, 14, 14, 2048)])
def test_resident_slab_images_exact(V, batch, C, H, W, M):
    """1x1 convolutions: slots that overlap at the end of every image."""
    import torch
    announce("resident slab, images", V, batch, C, H, W)
    p = synth.make_conv(batch, C, H, W, M, 1, 1, V, 0.5, seed=1721 + V, integer=True)
    want, _ = c_oracle.conv2d(p.W, p.mask, p.conv["input"], 1, 1, (1, 1), (0, 0))
    A = binding.compress(p.W, p.mask, p.perm, V).bind_device("cuda:0")
    for dt in (torch.float16, torch.float32):
        out = torch.full((batch, M, H, W), float("nan"), dtype=dt, device="cuda:0")
        A.conv2d(to_device(p.conv["input"]), 1, 1, out=out)
        torch.cuda.synchronize()
        assert "resident" in binding.last_kernel(), binding.last_kernel()
        assert np.array_equal(to_host(out).astype(np.float64), _rounded(want, "float16" if dt == torch.float16 else "float32"))


def test_resident_slab_keeps_infinities_apart():
    """A group of infinite weights and a row of X that no group keeps full of NaN: padded slots and steps beyond a group's end
    multiply zeros by zeros."""
    import torch
    announce("resident slab, infinities")
    V, G, K, N = 32, 128, 1024, 4096
    p = synth.make_spmm(G * V, K, N, V, 0.72, seed=1731, integer=True, ragged=True)
    W, X, mask = p.W.copy(), p.X.copy(), p.mask.copy()
    rows = p.perm[V:2 * V]
    W[np.ix_(rows, np.flatnonzero(mask[rows[0]]))] = np.float16(np.inf)
    X[0] = np.float16(np.nan)
    mask[:, 0] = 0
    want, _ = c_oracle.spmm(np.where(np.isinf(W), 0, W).astype(np.float16), mask, np.nan_to_num(X))
    A = binding.compress(W, mask, p.perm, V).bind_device("cuda:0")
    Y = torch.empty((G * V, N), dtype=torch.float32, device="cuda:0")
    A.spmm(torch.from_numpy(X).to("cuda:0"), Y)
    torch.cuda.synchronize()
    assert "resident" in binding.last_kernel(), binding.last_kernel()
    others = np.setdiff1d(np.arange(G * V), rows)
    assert np.array_equal(Y.cpu().numpy().astype(np.float64)[others], want[others])


def test_resident_slab_without_kept_columns_and_under_capture():
    import torch
    announce("resident slab, empty groups and a graph")
    V, G, K, N = 32, 128, 1024, 4096
    p = synth.make_spmm(G * V, K, N, V, 0.6, seed=1741, integer=True)
    mask = p.mask.copy()
    for g in (0, 5, 17, 127):
        mask[p.perm[g * V:(g + 1) * V]] = 0
    want, _ = c_oracle.spmm(p.W, mask, p.X)
    A = binding.compress(p.W, mask, p.perm, V).bind_device("cuda:0")
    X = to_device(p.X)
    Y = torch.full((G * V, N), float("nan"), dtype=torch.float32, device="cuda:0")
    A.spmm(X, Y)
    torch.cuda.synchronize()
    assert "resident" in binding.last_kernel(), binding.last_kernel()
    assert np.array_equal(Y.cpu().numpy().astype(np.float64), want)
    eager = Y.clone()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        A.spmm(X, Y)
    for _ in range(3):
        Y.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(Y, eager)
        A.spmm(X, Y)


@pytest.mark.parametrize("fmt", ["f16", "bf16"])
@pytest.mark.parametrize("layout,V,batch,C,H,W,M,R,stride,pad,sparsity", [
    ("NCHW", 16, 16, 128, 18, 18, 512, 3, 1, 1, 0.50),    # runs of 8, 8 and 2 columns; runs that begin before the image and end after it
    ("NCHW", 32, 16, 142, 21, 17, 1024, 3, 1, 1, 0.50),   # the longest reduction, one column in the last run
    ("NCHW", 32, 24, 70, 30, 32, 1024, 3, 1, 0, 0.50),    # no padding, 8 wavefronts
    ("NCHW", 16, 16, 48, 20, 64, 512, 5, 1, 1, 0.60),     # padding smaller than the kernel's half
    ("CHWN", 16, 20, 128, 16, 14, 512, 3, 1, 1, 0.50),    # images 12 .. 19 overlap 8 .. 15
    ("CHWN", 32, 33, 64, 30, 30, 1024, 3, 2, 1, 0.40),
    ("CHWN", 16, 32, 96, 14, 14, 768, 3, 2, 0, 0.50),
])
def test_resident_slab_convolution_exact(layout, V, batch, C, H, W, M, R, stride, pad, sparsity, fmt):
    """The unfolded matrix in the LDS; NaN right before and after the input."""
    import torch
    announce("resident slab, convolution", layout, V, batch, C, H, W, M, R, stride, pad, fmt)
    p = synth.make_conv(batch, C, H, W, M, R, R, V, sparsity, seed=1751 + V + H, pad=(pad, pad), stride=(stride, stride), integer=True, fmt=fmt)
    want, _ = c_oracle.conv2d(p.W, p.mask, p.conv["input"], R, R, (stride, stride), (pad, pad))
    A = binding.compress(p.W, p.mask, p.perm, V).bind_device("cuda:0")
    x = to_device(p.conv["input"])
    if layout == "CHWN":
        x = x.permute(1, 2, 3, 0).contiguous()
    flat = torch.full((x.numel() + 16,), float("nan"), dtype=x.dtype, device="cuda:0")
    flat[7:-9] = x.flatten()                              # no particular alignment
    out = A.conv2d(flat[7:-9].view(x.shape), R, R, (stride, stride), (pad, pad), layout=layout)
    torch.cuda.synchronize()
    assert "resident" in binding.last_kernel(), binding.last_kernel()
    if layout == "CHWN":
        out = out.permute(3, 0, 1, 2)
    want = _rounded(want, "bfloat16" if fmt == "bf16" else "float16")
    assert np.array_equal(to_host(out.contiguous()).astype(np.float64), want)


@pytest.mark.parametrize("fmt", ["f16", "bf16"])
@pytest.mark.parametrize("V,G,K,N,sparsity,ragged", [
    (16, 4, 1, 8, 0.0, False),             # one row of X, one slot of columns
    (16, 5, 33, 64, 0.4, True),            # one column tile
    (16, 7, 1278, 72, 0.5, False),
    (32, 4, 9, 1, 0.0, False),             # (refused: fewer than 8 columns that are no whole units)
    (32, 4, 640, 8, 0.9, True),
    (32, 17, 638, 65, 0.5, True),          # one column in the second tile
    (32, 35, 200, 130, 0.75, False),       # more groups than wavefronts of a workgroup
    (64, 4, 1278, 63, 0.3, True),
    (64, 19, 17, 128, 0.0, False),
    (128, 4, 100, 9, 0.5, False),
    (128, 9, 1278, 320, 0.8, True),
])
def test_resident_slab_as_asked_for(V, G, K, N, sparsity, ragged, fmt):
    """set_tuning(4, 0): far fewer tiles than the automatic choice gives it."""
    announce("resident slab, asked for", V, G, K, N, ragged, fmt)
    p = synth.make_spmm(G * V, K, N, V, sparsity, seed=1761 + N + V + K, integer=True, ragged=ragged, fmt=fmt)
    if N < 8:
        with pytest.raises(binding.ShflbwError):
            run_spmm(p, kernel=4)
        return
    want, _ = c_oracle.spmm(p.W, p.mask, p.X)
    for out in ("float32", "bfloat16" if fmt == "bf16" else "float16"):
        got = run_spmm(p, out_dtype=out, kernel=4, pad_ld=8 if N % 8 == 0 else 3).astype(np.float64)
        assert "resident" in binding.last_kernel(), binding.last_kernel()
        assert np.array_equal(got, _rounded(want, out)), np.argwhere(got != _rounded(want, out))[:4]


@pytest.mark.parametrize("layout,V,batch,C,H,W,M,R,stride,pad,sparsity", [
    ("NCHW", 16, 1, 3, 8, 8, 64, 3, 1, 1, 0.0),
    ("NCHW", 32, 2, 142, 9, 11, 128, 3, 1, 1, 0.6),
    ("NCHW", 16, 1, 51, 20, 19, 80, 5, 2, 1, 0.7),
    ("NCHW", 32, 3, 70, 15, 17, 128, 3, 2, 1, 0.5),
    ("NCHW", 128, 3, 65, 3, 3, 512, 1, 1, 0, 0.5),        # 1x1: a product per image
    ("CHWN", 32, 8, 20, 5, 6, 128, 3, 1, 1, 0.5),
    ("CHWN", 16, 13, 9, 7, 4, 64, 3, 2, 0, 0.2),
    ("CHWN", 64, 5, 30, 3, 3, 256, 1, 1, 0, 0.5),
])
def test_resident_slab_convolution_as_asked_for(layout, V, batch, C, H, W, M, R, stride, pad, sparsity):
    import torch
    announce("resident slab, convolution asked for", layout, V, batch, C, H, W, M, R, stride, pad)
    p = synth.make_conv(batch, C, H, W, M, R, R, V, sparsity, seed=1771 + V + H, pad=(pad, pad), stride=(stride, stride), integer=True)
    want, _ = c_oracle.conv2d(p.W, p.mask, p.conv["input"], R, R, (stride, stride), (pad, pad))
    A = binding.compress(p.W, p.mask, p.perm, V).bind_device("cuda:0")
    A.set_tuning(4, 0)
    x = to_device(p.conv["input"])
    out = A.conv2d(x if layout == "NCHW" else x.permute(1, 2, 3, 0).contiguous(), R, R, (stride, stride), (pad, pad), layout=layout)
    torch.cuda.synchronize()
    assert "resident" in binding.last_kernel(), binding.last_kernel()
    out = out if layout == "NCHW" else out.permute(3, 0, 1, 2).contiguous()
    assert np.array_equal(to_host(out).astype(np.float64), _rounded(want, "float16"))


def test_resident_slab_is_refused_where_it_cannot_run():
    import torch
    announce("resident slab, refused")
    def matrix(V, G, K):
        p = synth.make_spmm(G * V, K, 64, V, 0.5, seed=1781)
        A = binding.compress(p.W, p.mask, p.perm, V).bind_device("cuda:0")
        A.set_tuning(4, 0)
        return A
    X = torch.zeros((1279, 64), dtype=torch.float16, device="cuda:0")
    for V, G, K in ((32, 8, 1279), (32, 3, 64), (128, 3, 64)):
        with pytest.raises(binding.ShflbwError) as e:
            matrix(V, G, K).spmm(X[:K])
        assert e.value.status == -9
    x = torch.zeros((2, 16, 12, 12), dtype=torch.float16, device="cuda:0")
    for V, dt, w in ((64, torch.float16, 12), (32, torch.float32, 12), (32, torch.float16, 7)):   # too large groups, 32-bit results, no runs
        with pytest.raises(binding.ShflbwError) as e:
            matrix(V, 8, 144).conv2d(x[..., :w].contiguous(), 3, 3, (1, 1), (1, 1), out_dtype=dt)
        assert e.value.status == -9
