"""The cuts of the gather kernel at their edges: whole tiles that take their weights from the LDS chunk by chunk
(groups that end inside a chunk, at its end, before it, or have no step at all), the same without sharing,
128-column tiles whose k-steps are shared by 2 or 4 wavefronts, column counts at and beside the tiles'
edges.  Small integers: every sum is exact and the comparison with the oracle is bit for bit."""
import numpy as np
import pytest

from oracle import c_oracle
from paper_2203_05016_amd import binding, synth
from gpu_util import announce, run_spmm

pytestmark = pytest.mark.gpu

F32_WIDE = [(16, 1152, 3200, .6, 4), (16, 1153, 3200, .6, 4), (48, 2048, 2200, .6, 2), (64, 1409, 3200, .6, 2)]


def _check(p, out_dtype, want_name, **kw):
    import torch
    want, _ = c_oracle.spmm(p.W, p.mask, p.X)
    if out_dtype != "float32":   # sums of more than 2048 (256 in bfloat16) round
        want = torch.from_numpy(want).to(getattr(torch, out_dtype)).double().numpy()
    got = run_spmm(p, out_dtype=out_dtype, **kw).astype(np.float64)
    assert want_name in binding.last_kernel(), binding.last_kernel()
    assert np.array_equal(got, want), np.argwhere(got != want)[:4]


@pytest.mark.parametrize("V", [16, 32, 64, 128])
@pytest.mark.parametrize("tile_n", [64, 128])
@pytest.mark.parametrize("K,N,ragged", [
    (700, 8, False),       # one tile of four: wavefronts without a tile stay for the barriers
    (640, 256, True),      # unequal groups, some cut short inside a chunk
    (1100, 520, True),     # a last workgroup with one tile
    (600, 77, False),      # rows of no particular alignment
    (200, 264, True),
    (90, 264, True),       # too few steps to share the weights
])
def test_whole_tiles_exact(V, tile_n, K, N, ragged):
    announce("cuts, whole tiles", V, tile_n, K, N, ragged)
    p = synth.make_spmm(5 * V, K, N, V, 0.35, seed=1201 + N + V, integer=True, ragged=ragged)
    for out in ("float32", "float16"):
        _check(p, out, "<%d,%d,whole tiles" % (V, tile_n if V < 128 else 64), kernel=1, tile_n=tile_n)
        if K >= 600 and not (V == 16 and tile_n == 128 and ragged):   # V = 16: fewer than 13 steps of 32 columns of K
            assert "shared weights" in binding.last_kernel()
        elif K < 100 and tile_n == 128 and V < 128:
            assert "shared weights" not in binding.last_kernel()


@pytest.mark.parametrize("fmt", ["f16", "bf16"])
@pytest.mark.parametrize("V", [16, 32, 64])
@pytest.mark.parametrize("G,N,shares", [(32, 896, 4), (32, 889, 4), (64, 896, 2), (64, 889, 2)])
def test_wide_tiles_of_shared_steps_exact(V, G, N, shares, fmt):
    """Unequal groups, the last of them ending at any step of a wavefront's share."""
    announce("cuts, wide splits", V, G, N, fmt)
    p = synth.make_spmm(G * V, 2200, N, V, 0.4, seed=1301 + N + V, integer=True, ragged=True, fmt=fmt)
    for out in ("float16",) if V == 64 else ("float32", "float16"):   # V = 64 with 32-bit results: below
        out = "bfloat16" if (fmt, out) == ("bf16", "float16") else out
        _check(p, out, "<%d,128,split k-steps by %d" % (V, shares))


@pytest.mark.parametrize("fmt", ["f16", "bf16"])
@pytest.mark.parametrize("G,N,K,kept,shares", F32_WIDE)
def test_wide_tiles_of_two_row_blocks_with_32_bit_results_exact(G, N, K, kept, shares, fmt):
    """The one wide tile whose finished tile lies where the partial sums were, with a second row block to come."""
    announce("cuts, wide splits, f32", G, N, K, fmt)
    p = synth.make_spmm(G * 64, K, N, 64, 1 - kept, seed=1351 + N, integer=True, ragged=True, fmt=fmt)
    _check(p, "float32", "<64,128,split k-steps by %d" % shares)


@pytest.mark.parametrize("V", [32, 64])
def test_infinite_weights_do_not_reach_the_neighbours(V):
    """Padded slots and steps requested beyond a group's end (or a wavefront's share of one) multiply zeros: neither the
    next group's weights nor row 0 of X reach a result."""
    announce("cuts, infinities", V)
    p = synth.make_spmm(4 * V, 700, 136, V, 0.3, seed=1401 + V, integer=True, ragged=True)
    W = p.W.copy()
    rows = p.perm[V:2 * V]
    kept = np.flatnonzero(p.mask[rows[0]])
    W[np.ix_(rows, kept)] = np.float16(np.inf)
    X = p.X.copy()
    X[0] = np.float16(np.nan)
    mask = p.mask.copy()
    mask[:, 0] = 0
    A = binding.compress(W, mask, p.perm, V)
    want, _ = c_oracle.spmm(np.where(np.isinf(W), 0, W).astype(np.float16), mask, np.nan_to_num(X))
    import torch
    A.bind_device("cuda:0")
    Y = torch.empty((4 * V, 136), dtype=torch.float32, device="cuda:0")
    for kernel, tile, name in ((1, 64, "whole tiles"), (1, 128, "whole tiles"), (3, 0, "split k-steps by 8"), (0, 0, "split k-steps by 4")):
        A.set_tuning(kernel, tile)
        A.spmm(torch.from_numpy(X).to("cuda:0"), Y)
        assert name in binding.last_kernel(), binding.last_kernel()
        got = Y.cpu().numpy().astype(np.float64)
        others = np.setdiff1d(np.arange(4 * V), rows)
        assert np.array_equal(got[others], want[others]), (kernel, tile)
