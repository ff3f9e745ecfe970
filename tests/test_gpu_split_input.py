"""Compressed activations through the contraction in bfloat16 parts: every tile at ragged sizes, with prepared banks
and banks as the caller holds them, from compressed and from emitted handles; counts just below and at the number of
stored values from which it serves; Inf and NaN; graphs; a handle that is refilled with its result elsewhere."""
import numpy as np
import pytest
import torch

import oracle
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


def calls(F, s, w, b, relu=True):
    return (F.conv2d_sparse_input(s, w, (1, 1), (1, 1), b, relu),
            F.conv2d_sparse_input_prepared(s, F.dense_filter_prepare(w), (1, 1), (1, 1), b, relu))


SIZES = [
    (8, 64, 256, 28, 28), (9, 200, 130, 29, 31), (3, 130, 300, 57, 11), (16, 257, 190, 13, 64), (5, 77, 68, 33, 41), (2, 300, 65, 20, 23),
    (12, 40, 120, 45, 61), (16, 512, 512, 7, 7), (1, 64, 64, 4, 100), (2, 48, 96, 64, 9)]


@pytest.mark.parametrize("n,c,k,h,w", SIZES)
def test_integer_data_is_exact(F, n, c, k, h, w):
    x, wt, b = inputs.random_layer(n + c + k + h + w, n, c, k, h, w, 3, 3, 1.0, integer=True, x_zero_frac=0.5)
    xs = F.input_compress(dev(x))
    want = torch.nn.functional.conv2d(torch.from_numpy(x), torch.from_numpy(wt), torch.from_numpy(b), (1, 1), (1, 1)).relu_()
    for y in calls(F, xs, dev(wt), dev(b)):
        assert torch.equal(y.cpu(), want)


def test_sizes_above_take_every_kind_of_tile(F):
    tiles = set()
    for n, c, k, h, w in SIZES:
        for prepared in (True, False):
            start, tile, _ = F.si_split_choice(n, c, h, w, k, (1, 1), prepared)
            if start <= 0.5 * n * c * h * w:
                tiles.add(tile)
    assert len(tiles) >= 5


@pytest.mark.parametrize("emitted", [False, True])
@pytest.mark.parametrize("n,c,k,h,w", [(8, 40, 256, 28, 28), (9, 33, 300, 53, 57), (8, 16, 130, 28, 30)])
def test_the_kernel_goes_by_the_stored_values(F, n, c, k, h, w, emitted):
    """One value more takes a call to the contraction in parts; an emitted activation takes the same kernel whether or
    not its number is known; results hold to the fp32 bound on both sides."""
    start = F.si_split_choice(n, c, h, w, k, (1, 1), True)[0]
    assert 0 < start < n * c * h * w
    rng = np.random.default_rng(c)
    order = rng.permutation(n * c * h * w)
    wt = dev(rng.standard_normal((k, c, 3, 3)).astype(np.float32))
    eye = torch.zeros(c, c, 3, 3, device="cuda")
    eye[range(c), range(c), 1, 1] = 1.0
    f, d = F.filter_compress(eye), F.dense_filter_prepare(wt)
    for nnz in (start - 1, start):
        x = np.zeros(n * c * h * w, np.float32)
        x[order[:nnz]] = rng.standard_normal(nnz) + 3.0
        xd = dev(x.reshape(n, c, h, w))
        s = F.conv2d_sparse_filter_emit(f, xd, (1, 1), (1, 1)) if emitted else F.input_compress(xd)
        want = torch.nn.functional.conv2d(xd.double().cpu(), wt.double().cpu(), None, 1, 1)
        before = F.conv2d_sparse_input_prepared(s, d, (1, 1), (1, 1))
        rows = F.conv2d_sparse_input(s, wt, (1, 1), (1, 1))
        assert s.nnz == nnz
        assert torch.equal(before, F.conv2d_sparse_input_prepared(s, d, (1, 1), (1, 1)))
        assert torch.equal(rows, F.conv2d_sparse_input(s, wt, (1, 1), (1, 1)))
        for y in (before, rows):
            assert (y.double().cpu() - want).norm() <= 3e-7 * want.norm()     # 4.4e-7 is the fp32 unit's at 4608 products


def test_non_finite_values_meet_stored_values_only(F):
    n, c, k, h, w = 8, 64, 256, 28, 28
    x, wt, b = inputs.random_layer(8, n, c, k, h, w, 3, 3, 1.0, integer=True, x_zero_frac=0.5)
    assert F.si_split_choice(n, c, h, w, k, (1, 1), True)[0] <= np.count_nonzero(x)
    x[0, 11, :7] = 0.0
    wt[3, 11, 1, 1] = np.inf
    want = oracle.conv2d_dense(x, np.where(np.isinf(wt), 0, wt).astype(np.float32), (1, 1), (1, 1), None, False)
    for y in calls(F, F.input_compress(dev(x)), dev(wt), None, False):
        y = y.cpu().numpy()
        assert np.array_equal(np.isfinite(y[:, 3]), x[:, 11] == 0)
        assert np.array_equal(y[:, 3][x[:, 11] == 0], want[:, 3][x[:, 11] == 0])
        assert np.array_equal(np.delete(y, 3, 1), np.delete(want, 3, 1))


def test_refilled_with_the_result_in_a_tensor_of_the_caller(F):
    """The handle's own dense result is renewed then as well."""
    n, c, k, h, w = 8, 64, 256, 28, 28
    x, wt, _ = inputs.random_layer(5, n, c, k, h, w, 3, 3, 1.0, integer=True, x_zero_frac=0.5)
    eye = torch.zeros(c, c, 3, 3, device="cuda")
    eye[range(c), range(c), 1, 1] = 1.0
    f, xd = F.filter_compress(eye), dev(x)
    s = F.conv2d_sparse_filter_emit(f, torch.ones_like(xd), (1, 1), (1, 1))
    F.conv2d_sparse_filter_emit(f, xd, (1, 1), (1, 1), dense_out=(y := torch.empty_like(xd)), into=s)
    want = torch.nn.functional.conv2d(torch.from_numpy(x), torch.from_numpy(wt), None, 1, 1)
    y.zero_()
    for got in calls(F, s, dev(wt), None, False):
        assert torch.equal(got.cpu(), want)



@pytest.mark.parametrize("prepared", [True, False])
def test_fills_and_uses_in_graphs_and_outside_of_them(F, prepared):
    """A captured convolution reads what the handle holds when it is replayed, wherever the fill left the dense result; and a
    replayed fill renews what an eager convolution reads."""
    n, c, k, h, w = 8, 64, 256, 28, 28
    a, wt, _ = inputs.random_layer(5, n, c, k, h, w, 3, 3, 1.0, integer=True, x_zero_frac=0.5)
    b = inputs.random_layer(6, n, c, k, h, w, 3, 3, 1.0, integer=True, x_zero_frac=0.5)[0]
    want = [torch.nn.functional.conv2d(torch.from_numpy(x), torch.from_numpy(wt), None, 1, 1) for x in (a, b)]
    a, b, wd = dev(a), dev(b), dev(wt)
    eye = torch.zeros(c, c, 3, 3, device="cuda")
    eye[range(c), range(c), 1, 1] = 1.0
    f, d, one = F.filter_compress(eye), F.dense_filter_prepare(wd), (1, 1)
    x, elsewhere, y = a.clone(), torch.empty_like(a), torch.empty(n, k, h, w, device="cuda")
    conv = lambda **kw: F.conv2d_sparse_input_prepared(s, d, one, one, **kw) if prepared else F.conv2d_sparse_input(s, wd, one, one, **kw)  # noqa: E731
    s = F.conv2d_sparse_filter_emit(f, x, one, one)
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        conv()
        F.conv2d_sparse_filter_emit(f, x, one, one, dense_out=elsewhere, into=s)
    torch.cuda.synchronize()
    use, fill = torch.cuda.CUDAGraph(), torch.cuda.CUDAGraph()
    F.conv2d_sparse_filter_emit(f, x, one, one, into=s)
    torch.cuda.synchronize()
    with torch.cuda.graph(use, stream=side):
        conv(out=y)
    with torch.cuda.graph(fill, stream=side):
        F.conv2d_sparse_filter_emit(f, x, one, one, dense_out=elsewhere, into=s)
    for _ in range(3):
        F.conv2d_sparse_filter_emit(f, b, one, one, dense_out=elsewhere, into=s)
        use.replay()
        torch.cuda.synchronize()
        assert torch.equal(y.cpu(), want[1])
        F.conv2d_sparse_filter_emit(f, b, one, one, into=s)
        fill.replay()
        assert torch.equal(conv().cpu(), want[0])
        use.replay()
        torch.cuda.synchronize()
        assert torch.equal(y.cpu(), want[0])


def test_a_graph_beside_calls_on_the_stream_that_captured_it(F):
    n, c, k, h, w = 8, 64, 256, 28, 28
    x, wt, _ = inputs.random_layer(5, n, c, k, h, w, 3, 3, 1.0, integer=True, x_zero_frac=0.5)
    banks = [wt, np.ascontiguousarray(wt[::-1]), -wt]
    want = [torch.nn.functional.conv2d(torch.from_numpy(x), torch.from_numpy(b), None, 1, 1).cuda() for b in banks]
    banks, s = [dev(b) for b in banks], F.input_compress(dev(x))
    side, y = torch.cuda.Stream(), torch.empty(2, *want[0].shape, device="cuda")
    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        F.conv2d_sparse_input(s, banks[0], (1, 1), (1, 1))
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        for i in range(2):
            F.conv2d_sparse_input(s, banks[i], (1, 1), (1, 1), out=y[i])
    for _ in range(60):
        graph.replay()
        with torch.cuda.stream(side):
            beside = [F.conv2d_sparse_input(s, banks[2], (1, 1), (1, 1)) for _ in range(3)]
        torch.cuda.synchronize()
        assert torch.equal(y[0], want[0]) and torch.equal(y[1], want[1])
        assert all(torch.equal(b, want[2]) for b in beside)


def test_captured_with_the_bank_as_the_caller_holds_it(F):
    """With room for the parts from an eager call on the stream, and without (the contraction in fp32)."""
    n, c, k, h, w = 8, 64, 256, 28, 28
    x, wt, b = inputs.random_layer(5, n, c, k, h, w, 3, 3, 1.0, integer=True, x_zero_frac=0.5)
    want = torch.nn.functional.conv2d(torch.from_numpy(x), torch.from_numpy(wt), torch.from_numpy(b), 1, 1)
    wd, bd = dev(wt), dev(b)
    side = torch.cuda.Stream()
    for warm in (True, False):
        s, y = F.input_compress(dev(x)), torch.zeros(want.shape, device="cuda")
        torch.cuda.synchronize()
        if warm:
            with torch.cuda.stream(side):
                F.conv2d_sparse_input(s, wd, (1, 1), (1, 1), bd, False)
            torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=side):
            F.conv2d_sparse_input(s, wd, (1, 1), (1, 1), bd, False, out=y)
        for _ in range(3):
            y.zero_()
            torch.cuda.synchronize()
            graph.replay()
            torch.cuda.synchronize()
            assert torch.equal(y.cpu(), want)
            assert torch.equal(F.conv2d_sparse_input(s, wd, (1, 1), (1, 1), bd, False).cpu(), want)
