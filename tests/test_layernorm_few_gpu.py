"""LayerNorm-side transposition of few tokens (blocks of 16 tokens, or of 8 with two wavefronts per token, whose features are
shared by several workgroups) at its edges, and of the next larger numbers of tokens, which the other kernels take
(test_choice.py holds which).  Bounds as in test_layernorm_gpu.py."""
import numpy as np
import pytest

from oracle import definition
from paper_2203_05016_amd import binding, synth
from gpu_util import announce, to_device, to_host
from test_layernorm_gpu import _check, _draw

pytestmark = pytest.mark.gpu


SHAPES = [
    (8, 8), (16, 16), (24, 72), (40, 504), (40, 520), (136, 1000),   # less than a run of 512 features, a run and a little, ragged slices
    (4096, 1024), (4104, 1024), (2048, 2048), (2056, 2048),          # the most tokens, and the next
    (8, 2056), (512, 2056), (520, 2056), (768, 3584), (776, 3584),   # 8 tokens: 64 blocks and 65, the most tokens and the next
    (8, 16384), (56, 16376), (768, 16384), (776, 16384), (776, 8192), (800, 5000),
]


@pytest.mark.parametrize("fmt", ["f16", "bf16"])
@pytest.mark.parametrize("N,K", SHAPES)
def test_few_tokens_parity(fmt, N, K):
    announce("layernorm, few tokens", fmt, N, K)
    x, gamma, beta = _draw(N, K, fmt, seed=1800 + N + K, offset=3.0)
    _check(x, gamma, beta, 1e-5, fmt)
    if N * K < 1 << 20:
        _check(x, None, beta, 1e-5, fmt)
        _check(x, gamma, None, 1e-5, fmt)


@pytest.mark.parametrize("N,K", [(40, 1000), (104, 4104)])
def test_few_tokens_write_their_window_only(N, K):
    """Padded leading dimensions on both sides; tokens far from zero with a small spread, constant tokens."""
    import torch
    announce("layernorm, few tokens, window", N, K)
    x, gamma, beta = _draw(N, K, "f16", seed=1900 + K, offset=100.0, scale=0.25)
    x[3] = x[3, 0]
    xd = torch.full((N, K + 24), float("nan"), dtype=torch.float16, device="cuda:0")[:, :K]
    xd.copy_(to_device(x))
    buf = torch.full((K, N + 16), float("nan"), dtype=torch.float16, device="cuda:0")
    binding.layernorm_transpose(xd, to_device(gamma), to_device(beta), 1e-5, out=buf[:, :N])
    got = to_host(buf)
    want, S = definition.layernorm_transpose(synth.as_float(x), synth.as_float(gamma), synth.as_float(beta), 1e-5)
    tol = 2.0 ** -10
    assert np.all(np.abs(got[:, :N].astype(np.float64) - want) <= tol * S + tol * 2.0 ** -4)
    assert np.isnan(got[:, N:]).all()
