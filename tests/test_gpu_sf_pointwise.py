"""The kernel for 1x1 filters: planes whose size is no multiple of four or of a work-group's pixels, four pixels and fewer, empty filters and every
number of entries around the batches of eight, batches off every multiple of four through N4 tensors; activations and bias; bit for bit on
integers; precision; values that are not finite meet stored entries only; calls that capture without a plan."""
import numpy as np
import pytest
import torch

from paper_2212_08815_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def F():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2212_08815_amd import fscnn
    fscnn.lib()
    return fscnn


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def call(F, f, x, n4, bias=None, relu=False, leaky=None):
    if not n4:
        return F.conv2d_sparse_filter(f, x, bias=bias, relu=relu, leaky=leaky)
    y = F.conv2d_sparse_filter(f, F.layout_convert(x, F.NCHW), bias=bias, relu=relu, leaky=leaky, x_layout=F.N4, y_layout=F.N4, n=x.shape[0])
    return F.layout_convert(y, F.N4, n=x.shape[0])


def served(F, f, n, h, w, n4):
    lay = F.N4 if n4 else F.NCHW
    return F.sf_serves(f, n, h, w, x_layout=lay, y_layout=lay) == F.POINTWISE


def bank(k, c, integer, seed=0):
    """Filters of 0, 1, 2, ... entries."""
    rng = np.random.default_rng(seed + k + c)
    w = np.zeros((k, c, 1, 1), np.float32)
    for i in range(k):
        at = rng.choice(c, min(c, i % 35), replace=False)
        w[i, at, 0, 0] = rng.integers(1, 4, at.size) if integer else rng.standard_normal(at.size)
    return w


@pytest.mark.parametrize("n4", [False, True])
@pytest.mark.parametrize("n,c,k,h,w", [(1, 40, 37, 2, 2), (3, 64, 70, 5, 1), (1, 300, 71, 7, 9), (5, 33, 130, 16, 16), (2, 90, 36, 1, 257),
                                       (4, 50, 66, 15, 17), (7, 128, 40, 13, 13), (1, 1, 4, 30, 30), (1, 35, 35, 3, 1), (6, 200, 300, 31, 33)])
def test_sizes(F, n, c, k, h, w, n4):
    x = np.random.default_rng(n + h).integers(-3, 4, (n, c, h, w)).astype(np.float32)
    b = np.arange(k, dtype=np.float32) % 5 - 2
    wt = bank(k, c, True)
    f, xd, bd = F.filter_compress(dev(wt)), dev(x), dev(b)
    # (fewer than four pixels are not its own; the largest through N4 tensors is gathered)
    assert served(F, f, n, h, w, n4) == (h * w * (4 if n4 else 1) >= 4 and not (n4 and h == 31))
    want = torch.nn.functional.conv2d(torch.from_numpy(x), torch.from_numpy(wt))
    assert torch.equal(call(F, f, xd, n4).cpu(), want)
    want = want + torch.from_numpy(b).view(1, k, 1, 1)
    assert torch.equal(call(F, f, xd, n4, bd, True).cpu(), want.relu())
    assert torch.equal(call(F, f, xd, n4, bd, leaky=0.5).cpu(), torch.where(want > 0, want, 0.5 * want))


def test_precision(F):
    # n multiply-adds and three sums of parts: n + 3 roundings of half a unit (2^-24) each at the most
    n, c, k, h, w = 2, 120, 70, 20, 21
    x, wt = np.abs(inputs.random_layer(1, n, c, k, h, w, 1, 1, 1.0)[0]), np.abs(bank(k, c, False))
    want = torch.nn.functional.conv2d(torch.from_numpy(x).double(), torch.from_numpy(wt).double())
    f = F.filter_compress(dev(wt))
    assert served(F, f, n, h, w, False)
    got = call(F, f, dev(x), False).cpu().double()
    bound = torch.from_numpy((np.count_nonzero(wt, axis=(1, 2, 3)) + 3) * 2.0 ** -24).view(1, k, 1, 1)
    assert ((got - want).abs() <= bound * want).all()


def test_values_that_are_not_finite(F):
    x = np.ones((1, 64, 12, 12), np.float32)
    x[0, 5, 3, 4], x[0, 6, 0, 0], x[0, 63, 11, 11] = np.inf, np.nan, -np.inf
    wt = bank(64, 64, True)
    want = np.einsum("kc,chw->khw", wt[:, :, 0, 0], np.where(np.isfinite(x[0]), x[0], 0))
    met = np.einsum("kc,chw->khw", wt[:, :, 0, 0] != 0, ~np.isfinite(x[0])) > 0
    f = F.filter_compress(dev(wt))
    assert served(F, f, 1, 12, 12, False)
    got = call(F, f, dev(x), False)[0].cpu().numpy()
    assert np.array_equal(np.isfinite(got), ~met) and np.array_equal(got[~met], want[~met]) and met.any()


def test_emitting_call_captured_after_prepare(F):
    """(The 1x1 kernel prepares no plan, and it does not serve emitting calls that can make one.)"""
    n, c, k, h, w = 2, 256, 128, 22, 21
    x = dev(np.random.default_rng(4).integers(-3, 4, (n, c, h, w)).astype(np.float32))
    f1, wt = F.filter_compress(dev(bank(k, c, True, 1))), bank(k, c, True)
    want = torch.nn.functional.conv2d(x.cpu(), torch.from_numpy(wt)).relu()
    into, f = F.conv2d_sparse_filter_emit(f1, x, relu=True), F.filter_compress(dev(wt))
    assert served(F, f, n, h, w, False)
    F.filter_prepare(f, n, h, w)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        F.conv2d_sparse_filter_emit(f, x, relu=True, into=into)
    for _ in range(3):
        F.conv2d_sparse_filter_emit(f1, x, relu=True, into=into)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        into._nnz = None
        prow, cidx, val = F.input_export(into)
        got = np.zeros((n * h * w, k), np.float32)
        got[np.repeat(np.arange(n * h * w), np.diff(prow)), cidx] = val
        assert np.array_equal(got.reshape(n, h, w, k).transpose(0, 3, 1, 2), want.numpy())


@pytest.mark.parametrize("n4", [False, True])
def test_captured_without_a_plan(F, n4):
    """(What would serve these calls otherwise builds a plan, which a capture refuses.)"""
    x = dev(np.random.default_rng(2).integers(-3, 4, (4, 256, 22, 22)).astype(np.float32))
    wt = bank(128, 256, True)
    want = torch.nn.functional.conv2d(x.cpu(), torch.from_numpy(wt))
    f, xx, lay = F.filter_compress(dev(wt)), F.layout_convert(x, F.NCHW) if n4 else x, F.N4 if n4 else F.NCHW
    assert F.sf_variant_choice(f, 4, 22, 22, n4=n4) > 0 and served(F, f, 4, 22, 22, n4)
    y = torch.zeros(F.n4_shape(4, 128, 22, 22) if n4 else want.shape, device="cuda")
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        F.conv2d_sparse_filter(f, xx, x_layout=lay, y_layout=lay, n=4, out=y)
    for _ in range(3):
        y.zero_()
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal((F.layout_convert(y, F.N4, n=4) if n4 else y).cpu(), want)
        F.conv2d_sparse_filter(f, xx, x_layout=lay, y_layout=lay, n=4)
