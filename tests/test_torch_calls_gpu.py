"""The native calls on torch tensors: the plain case runs there and gives what the general way
gives; everything else is handed back to the binding's own checks, which refuse what they refused
and take what they took."""
import numpy as np
import pytest

from paper_2203_05016_amd import binding, synth
from gpu_util import announce, to_device, to_host

pytestmark = pytest.mark.gpu



def _tagged(t):
    import torch
    return t.as_subclass(type("TaggedTensor", (torch.Tensor,), {}))


def test_spmm_plain_case_and_what_is_handed_back():
    import torch
    announce("torch calls, spmm")
    p = synth.make_spmm(64, 96, 40, 32, 0.5, seed=11)
    A = binding.compress(p.W, p.mask, p.perm, 32).bind_device("cuda:0")
    native, plan = binding.calls(), A._plan
    X = to_device(p.X)
    Y = torch.empty((64, 40), dtype=torch.float16, device="cuda:0")
    assert native.spmm(plan, X, Y) == 0
    want = to_host(A.spmm(X, stream=torch.cuda.current_stream()))   # a stream argument takes the general way
    assert np.array_equal(to_host(Y), want)
    wide = torch.empty((64, 48), dtype=torch.float32, device="cuda:0")
    assert native.spmm(plan, X, wide[:, :40]) == 0                   # padded rows, 32-bit output
    # the current stream is the one that is used
    side = torch.cuda.Stream()
    Y2 = torch.zeros_like(Y)
    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        assert native.spmm(plan, X, Y2) == 0
    side.synchronize()
    assert np.array_equal(to_host(Y2), want)
    one = torch.empty((64, 1), dtype=torch.float16, device="cuda:0")
    assert native.spmm(plan, X[:, :1], one) == 0                     # one column: strides of 40 and 1
    for bad in (X.t().contiguous().t(), X[:, ::2], X.bfloat16(), X.cpu(), X[:95], _tagged(X), None, 3, p.X):
        assert native.spmm(plan, bad, Y) is None
    for bad in (Y[:, :39], Y.t(), Y.double(), Y.cpu(), _tagged(Y), Y[:32], None):
        assert native.spmm(plan, X, bad) is None
    assert np.array_equal(to_host(A.spmm(_tagged(X), Y)), want)      # taken before, taken still
    with pytest.raises(ValueError, match="must live on"):
        A.spmm(X, Y.cpu())
    with pytest.raises(ValueError, match="K = 96"):
        A.spmm(X[:95], Y)
    with pytest.raises(RuntimeError):                                # no memory stands behind a batched tensor
        torch.vmap(lambda v: A.spmm(v, Y))(torch.stack([X, X]))


def test_conv2d_and_layernorm_plain_case_and_what_is_handed_back():
    import torch
    announce("torch calls, conv2d and layernorm")
    p = synth.make_conv(9, 16, 8, 9, 64, 3, 3, 32, 0.5, seed=12, pad=(1, 1))
    A = binding.compress(p.W, p.mask, p.perm, 32).bind_device("cuda:0")
    native, plan = binding.calls(), A._plan
    x = to_device(p.conv["input"])
    for chwn in (False, True):
        xl = x.permute(1, 2, 3, 0).contiguous() if chwn else x
        shape = (64, 8, 9, 9) if chwn else (9, 64, 8, 9)
        out = torch.empty(shape, dtype=torch.float16, device="cuda:0")
        assert native.conv2d(plan, xl, 3, 3, (1, 1), (1, 1), chwn, out) == 0
        want = to_host(A.conv2d(xl, 3, 3, (1, 1), (1, 1), "CHWN" if chwn else "NCHW"))
        assert np.array_equal(to_host(out), want)
        assert native.conv2d(plan, xl, 3, 3, [1, 1], (1, 1), chwn, out) is None     # a list: the general way takes it
        assert np.array_equal(to_host(A.conv2d(xl, 3, 3, [1, 1], [1, 1], "CHWN" if chwn else "NCHW", out=out)), want)
        for args in ((xl, 3, 3, (0, 1), (1, 1), chwn, out), (xl, 3, 3, (1, 1), (1, 0), chwn, out),
                     (xl, 3, 1, (1, 1), (1, 1), chwn, out), (xl, 3, 3, (1, 1), (1, 1), not chwn, out),
                     (xl.cpu(), 3, 3, (1, 1), (1, 1), chwn, out), (xl, 3, 3, (1, 1), (-1, 1), chwn, out),
                     (xl.permute(0, 1, 3, 2), 3, 3, (1, 1), (1, 1), chwn, out)):
            assert native.conv2d(plan, *args) is None
    t = torch.randn((24, 64), device="cuda:0").half()
    g, b = torch.randn(64, device="cuda:0").half(), torch.randn(64, device="cuda:0").half()
    out = torch.empty((64, 24), dtype=torch.float16, device="cuda:0")
    assert native.layernorm_transpose(t, g, b, 1e-5, True, out) == 0
    want = to_host(binding.layernorm_transpose(t, g, b, 1e-5, True))
    assert np.array_equal(to_host(out), want)
    assert native.layernorm_transpose(t, None, None, 1e-5, False, out) == 0
    assert np.array_equal(to_host(out), to_host(t).T)
    for args in ((t, g.float(), b, 1e-5, True, out), (t, g[:63], b, 1e-5, True, out), (t.cpu(), g, b, 1e-5, True, out),
                 (t, g, b, 1, True, out), (t, g, b, 1e-5, 1, out), (t, g, b, 1e-5, True, out[:, :23]), (t.t(), g, b, 1e-5, True, out)):
        assert native.layernorm_transpose(*args) is None


def test_an_exception_out_of_the_library_is_handed_back():
    """The interpreter lock is held again when a C++ exception passes by (libstdc++'s own function that
    throws std::bad_alloc stands in for the library's entry points)."""
    import ctypes
    import torch
    announce("torch calls, exception")
    p = synth.make_spmm(64, 96, 40, 32, 0.5, seed=11)
    A = binding.compress(p.W, p.mask, p.perm, 32).bind_device("cuda:0")
    native, L = binding.calls(), binding.lib()
    X, Y = to_device(p.X), torch.empty((64, 40), dtype=torch.float16, device="cuda:0")
    img, out = torch.zeros((1, 96, 2, 4), dtype=torch.float16, device="cuda:0"), torch.empty((1, 64, 2, 4), dtype=torch.float16, device="cuda:0")
    t, tt = torch.zeros((40, 64), dtype=torch.float16, device="cuda:0"), torch.empty((64, 40), dtype=torch.float16, device="cuda:0")
    address = lambda f: ctypes.cast(f, ctypes.c_void_p).value
    throws = address(ctypes.CDLL("libstdc++.so.6")._ZSt17__throw_bad_allocv)
    raw_stream = torch._C._cuda_getCurrentRawStream
    native.connect(throws, throws, throws, raw_stream)
    try:
        for _ in range(3):
            assert native.spmm(A._plan, X, Y) is None
            assert native.conv2d(A._plan, img, 1, 1, (1, 1), (0, 0), False, out) is None
            assert native.layernorm_transpose(t, None, None, 1e-5, True, tt) is None
    finally:
        native.connect(address(L.shflbw_spmm), address(L.shflbw_conv2d), address(L.shflbw_layernorm_transpose), raw_stream)
    assert native.spmm(A._plan, X, Y) == 0
    assert np.array_equal(to_host(Y), to_host(A.spmm(X)))
