"""The contraction on the matrix cores: dense-ish filter banks, filter extents without a gather
configuration, compressed activations with dense banks.  Every tile of it, for each source and form of
bank, with what the choice says asserted; sizes at the edges: one pixel, tiles that end inside a row, rows that
cross images, panels of wide images, channel counts around the slices of 16 and the rows of 16, chunks
that end early; Inf and NaN.  Which calls it serves."""
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


@pytest.mark.parametrize("tile,wide,n,c,k,h,w,r,s,stride", [
    (0, False, 8, 75, 131, 46, 48, 3, 3, (1, 1)), (0, True, 6, 120, 91, 44, 91, 3, 3, (1, 1)),
    (1, False, 8, 125, 65, 35, 51, 3, 3, (1, 1)), (1, False, 9, 56, 148, 48, 43, 3, 3, (2, 1)),
    (2, False, 7, 58, 96, 28, 41, 3, 3, (1, 1)), (2, True, 4, 140, 34, 24, 122, 3, 3, (1, 1)),
    (2, True, 9, 70, 111, 41, 61, 3, 3, (1, 3)), (3, False, 9, 120, 84, 43, 21, 3, 3, (1, 1)),
    (4, False, 6, 118, 139, 25, 12, 3, 3, (1, 1)), (4, True, 2, 88, 33, 17, 139, 3, 3, (1, 1)),
    (4, False, 6, 63, 148, 50, 18, 3, 3, (2, 1)), (5, True, 3, 94, 25, 3, 35, 3, 3, (1, 1)),
    (6, False, 9, 113, 79, 25, 22, 3, 3, (1, 1)), (7, False, 3, 76, 129, 34, 16, 3, 3, (1, 1)),
    (0, True, 4, 14, 104, 40, 128, 5, 5, (1, 1)), (1, False, 8, 14, 146, 37, 32, 5, 5, (1, 1)),
    (2, False, 9, 21, 130, 49, 22, 5, 5, (2, 2)), (2, True, 5, 19, 103, 46, 118, 5, 5, (2, 2)),
    (3, False, 8, 56, 144, 45, 10, 5, 5, (1, 1)), (4, False, 9, 134, 72, 29, 11, 5, 5, (1, 1)),
    (6, False, 9, 42, 140, 29, 12, 5, 5, (1, 1)), (7, False, 6, 72, 141, 16, 17, 5, 5, (1, 1)),
    (2, False, 1, 4, 41, 46, 16, 7, 3, (1, 3)), (4, True, 7, 42, 105, 21, 49, 7, 3, (2, 1)),
    (7, False, 9, 20, 91, 50, 11, 7, 3, (2, 1)),     # uneven strides
    (1, True, 7, 49, 42, 46, 147, 2, 4, (2, 1)), (4, True, 9, 28, 77, 25, 42, 2, 4, (1, 3)),
    (5, True, 3, 2, 72, 32, 30, 2, 4, (2, 2)),       # ... filter no wider than the stride
    (1, False, 8, 107, 82, 20, 89, 1, 1, (1, 1)), (2, True, 8, 12, 8, 27, 145, 1, 1, (2, 2)),
])
def test_every_tile_is_exact_on_integers(F, tile, wide, n, c, k, h, w, r, s, stride):
    # integers: every partial sum is exact in fp32, so any order of summation gives the same bits
    pad = (r // 2, s // 2)
    x, wt, b = inputs.random_layer(n + c + k + h + w, n, c, k, h, w, r, s, 0.7, integer=True)
    f = F.filter_compress(dev(wt))
    assert F.sf_contract_choice(f, n, h, w, stride, pad)[0] == tile
    assert (F.sf_contract_choice(f, n, h, w, stride, pad)[1] > 1) == wide
    want = torch.nn.functional.conv2d(torch.from_numpy(x), torch.from_numpy(wt), torch.from_numpy(b), stride, pad).relu_()
    assert torch.equal(F.conv2d_sparse_filter(f, dev(x), stride, pad, dev(b), True).cpu(), want)


@pytest.mark.parametrize("n,c,k,r,hw,keep", [
    (31, 139, 369, 1, 12, 0.05), (15, 23, 62, 1, 79, 0.21), (9, 82, 50, 1, 102, 0.07),   # 1x1: 2 to 3 times as long contracted
    (27, 29, 327, 3, 46, 0.35),
    (8, 512, 512, 3, 28, 0.20),
    (6, 40, 35, 5, 96, 0.02),       # the direct kernel
])
def test_layers_that_are_faster_gathered_are_not_contracted(F, n, c, k, r, hw, keep):
    _, wt, _ = inputs.random_layer(4, 1, c, k, 3, 3, r, r, keep)
    assert F.sf_contract_choice(F.filter_compress(dev(wt)), n, hw, hw, (1, 1), (r // 2, r // 2))[0] == -1


@pytest.mark.parametrize("n,c,k,h,w,r,s,stride,pad", [
    (1, 1, 1, 1, 1, 3, 3, (1, 1), (1, 1)),        # one pixel, one channel
    (1, 16, 64, 14, 14, 3, 3, (1, 1), (1, 1)),    # whole slices and rows
    (2, 17, 65, 13, 17, 3, 3, (1, 1), (1, 1)),    # one past them; tiles end inside a row
    (13, 33, 31, 3, 5, 3, 3, (1, 1), (0, 1)),     # one output row per image: a tile crosses many images
    (1, 70, 20, 9, 131, 3, 3, (1, 1), (1, 1)),    # panels, the last one narrower
    (7, 128, 130, 11, 11, 3, 3, (1, 1), (1, 1)),  # several chunks, ragged last rows
    (2, 40, 33, 12, 19, 5, 5, (1, 1), (2, 2)),    # an extent without a gather configuration
    (4, 9, 50, 10, 10, 2, 4, (1, 3), (0, 2)),     # ... that the direct kernel may serve
])
def test_integer_data_is_exact(F, n, c, k, h, w, r, s, stride, pad):
    # integers: every partial sum is exact in fp32, so any order of summation gives the same bits
    x, wt, b = inputs.random_layer(n + c + k + h + w, n, c, k, h, w, r, s, 0.7, integer=True)
    want = oracle.conv2d_dense(x, wt, stride, pad, b, True)
    got = F.conv2d_sparse_filter(F.filter_compress(dev(wt)), dev(x), stride, pad, dev(b), True).cpu().numpy()
    assert np.array_equal(got, want)
    if (r, s) == (3, 3):
        xs = F.input_compress(dev(x))
        for y in (F.conv2d_sparse_input(xs, dev(wt), stride, pad, dev(b), True),
                  F.conv2d_sparse_input_prepared(xs, F.dense_filter_prepare(dev(wt)), stride, pad, dev(b), True)):
            assert np.array_equal(y.cpu().numpy(), want)


@pytest.mark.parametrize("tile,wide,n,c,k,h,w", [
    (0, True, 8, 17, 65, 29, 78), (1, False, 7, 25, 68, 38, 53), (1, True, 6, 17, 65, 30, 46), (2, False, 7, 20, 33, 32, 73),
    (2, True, 2, 17, 68, 34, 62), (3, False, 4, 37, 138, 40, 34), (3, True, 8, 35, 33, 19, 56), (4, False, 8, 17, 44, 40, 14),
    (4, True, 6, 17, 34, 13, 54), (5, False, 2, 23, 35, 3, 4), (5, True, 1, 20, 41, 3, 10), (6, False, 5, 35, 132, 27, 22),
    (6, True, 8, 36, 65, 9, 57), (7, False, 5, 18, 65, 34, 14), (7, True, 3, 17, 65, 12, 59),
])
def test_every_tile_is_exact_on_lists(F, tile, wide, n, c, k, h, w):
    x, wt, b = inputs.random_layer(n + c + k + h + w, n, c, k, h, w, 3, 3, 1.0, integer=True, x_zero_frac=0.5)
    xs = F.input_compress(dev(x))
    want = torch.nn.functional.conv2d(torch.from_numpy(x), torch.from_numpy(wt), torch.from_numpy(b), (1, 1), (1, 1)).relu_()
    for prepared in (False, True):
        start, t, panels = F.si_contract_choice(n, c, h, w, k, (1, 1), prepared)
        assert start <= xs.nnz and t == tile and (panels > 1) == wide
        y = (F.conv2d_sparse_input_prepared(xs, F.dense_filter_prepare(dev(wt)), (1, 1), (1, 1), dev(b), True) if prepared
             else F.conv2d_sparse_input(xs, dev(wt), (1, 1), (1, 1), dev(b), True))
        assert torch.equal(y.cpu(), want)


@pytest.mark.parametrize("n,c,k,h,w", [(1, 4, 8, 2, 40001), (2, 21, 70, 1, 40003), (1, 17, 65, 40001, 2)])
def test_sizes_the_contraction_does_not_serve_are_gathered(F, n, c, k, h, w):
    # images beyond 40000 rows or columns; ragged channels, rows and columns of the gather kernels' tiles
    x, wt, b = inputs.random_layer(n + c + k, n, c, k, h, w, 3, 3, 1.0, integer=True, x_zero_frac=0.7)
    xs = F.input_compress(dev(x))
    want = torch.nn.functional.conv2d(torch.from_numpy(x), torch.from_numpy(wt), torch.from_numpy(b), (1, 1), (1, 1)).relu_()
    for prepared in (False, True):
        assert F.si_contract_choice(n, c, h, w, k, (1, 1), prepared)[0] > n * c * h * w
        y = (F.conv2d_sparse_input_prepared(xs, F.dense_filter_prepare(dev(wt)), (1, 1), (1, 1), dev(b), True) if prepared
             else F.conv2d_sparse_input(xs, dev(wt), (1, 1), (1, 1), dev(b), True))
        assert torch.equal(y.cpu(), want)


@pytest.mark.parametrize("n,c,k,h,w,shift", [
    (8, 40, 256, 28, 28, -2.5), (8, 40, 256, 28, 28, 0.0),      # below and above the number from which it is contracted
    (9, 33, 300, 53, 57, -2.5), (9, 33, 300, 53, 57, 0.0),      # ... 16-wave form of the gather
    (8, 40, 256, 28, 28, -99.0),                                # nothing stored
])
def test_emitted_activations_go_by_what_they_store(F, n, c, k, h, w, shift):
    """The kernel that serves an emitted activation goes by its stored values, whether or not the caller has asked for
    their number: the same bits before and after, and those of the gather kernel exactly where that is to serve."""
    g = torch.Generator().manual_seed(3)
    x = torch.randn(n, 8, h, w, generator=g).cuda()
    f = F.filter_compress((torch.randn(c, 8, 3, 3, generator=g) / 8.5).cuda())
    d = F.dense_filter_prepare(torch.randn(k, c, 3, 3, generator=g).cuda())
    s = F.conv2d_sparse_filter_emit(f, x, (1, 1), (1, 1), torch.full((c,), shift).cuda(), True)
    start = F.si_contract_choice(n, c, h, w, k, (1, 1), True)[0]
    assert 0 < start < n * c * h * w
    before = F.conv2d_sparse_input_prepared(s, d, (1, 1), (1, 1))
    below = s.nnz < start
    assert below == (shift < 0)
    after = F.conv2d_sparse_input_prepared(s, d, (1, 1), (1, 1))
    assert torch.equal(before, after)
    patches = n * -(-h // 4) * -(-w // 4) * -(-k // 256)
    gathered = F.conv2d_sparse_input_prepared(s, d, (1, 1), (1, 1), variant=4 if patches >= 2048 else 1)
    assert torch.equal(before, gathered) == below
    assert torch.allclose(before, gathered, rtol=1e-4, atol=1e-4)


def test_contracted_layers_can_be_captured_unprepared(F):
    """A layer without a gather configuration needs no device data of its own under capture: the direct kernel."""
    x, wt, b = inputs.random_layer(21, 2, 24, 40, 20, 17, 5, 5, 0.5, integer=True)
    want = torch.nn.functional.conv2d(torch.from_numpy(x), torch.from_numpy(wt), torch.from_numpy(b), (1, 1), (2, 2)).relu_()
    f, xd, bd, y = F.filter_compress(dev(wt)), dev(x), dev(b), torch.zeros(want.shape, device="cuda")
    assert F.sf_contract_choice(f, 2, 20, 17, (1, 1), (2, 2))[0] >= 0
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        F.conv2d_sparse_filter(f, xd, (1, 1), (2, 2), bd, True, out=y)
    for _ in range(3):
        y.zero_()
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(y.cpu(), want)
        assert torch.equal(F.conv2d_sparse_filter(f, xd, (1, 1), (2, 2), bd, True).cpu(), want)   # eager: contracted


def test_no_room_for_the_dense_copy_of_a_bank(F):
    """A sparse bank of a large extent on a nearly full card: its dense copy (679 MB) does not fit, the direct kernel
    serves the call, and fscnn_filter_prepare does not fail either."""
    k, c, r = 1024, 2048, 9
    wt = torch.zeros(k, c, r, r, device="cuda")
    wt.view(-1)[::47] = 1.0
    f = F.filter_compress(wt)
    x = (torch.arange(c * 49, device="cuda") % 5 - 2).float().view(1, c, 7, 7)
    want = torch.nn.functional.conv2d(x.cpu(), wt.cpu(), None, 1, 4)
    assert F.sf_contract_choice(f, 1, 7, 7, (1, 1), (4, 4))[0] >= 0
    del wt
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    held = []
    try:
        while (free := torch.cuda.mem_get_info()[0]) > (600 << 20):
            held.append(torch.empty(min(free - (512 << 20), 64 << 30), dtype=torch.uint8, device="cuda"))
        with pytest.raises(torch.OutOfMemoryError):
            torch.empty(679 << 20, dtype=torch.uint8, device="cuda")
        F.filter_prepare(f, 1, 7, 7, (1, 1), (4, 4))
        got = F.conv2d_sparse_filter(f, x, (1, 1), (4, 4))
        torch.cuda.synchronize()
    finally:
        del held
        torch.cuda.empty_cache()
    assert torch.equal(got.cpu(), want)
    assert torch.equal(F.conv2d_sparse_filter(f, x, (1, 1), (4, 4)).cpu(), want)     # room again


def test_only_stored_entries_meet_non_finite_values(F):
    """0 * Inf never appears: a filter without an entry at a tap does not see the Inf there, a zero
    activation does not meet an Inf weight."""
    n, c, k, h, w = 1, 40, 48, 14, 14
    x, wt, b = inputs.random_layer(7, n, c, k, h, w, 3, 3, 0.8, integer=True)
    x[0, 5, 6, 7], x[0, 39, 0, 0] = np.inf, np.nan
    wt[::2, 5] = 0.0
    wt[1::4, 39] = 0.0
    fin = np.isfinite(x)
    want = oracle.conv2d_dense(np.where(fin, x, 0).astype(np.float32), wt, (1, 1), (1, 1), b, False)
    met = oracle.conv2d_dense((~fin).astype(np.float32), (wt != 0).astype(np.float32), (1, 1), (1, 1), None, False) > 0
    got = F.conv2d_sparse_filter(F.filter_compress(dev(wt)), dev(x), (1, 1), (1, 1), dev(b), False).cpu().numpy()
    assert np.array_equal(np.isfinite(got), ~met) and np.array_equal(got[~met], want[~met])
    assert 0 < met.sum() < met.size
    # an extent that only the direct kernel serves otherwise: entries outside the image meet nothing, so an
    # Inf weight gives Inf or a finite sum there and no NaN
    x, wt, b = inputs.random_layer(9, 2, c, k, 24, 19, 5, 5, 0.8, integer=True)
    x = np.abs(x) + 1
    wt[3, 7, 0, 0] = np.inf                                         # meets x at (oy - 2, ox - 2)
    want = oracle.conv2d_dense(x, np.where(np.isinf(wt), 0, wt).astype(np.float32), (1, 1), (2, 2), b, False)
    want[:, 3, 2:, 2:] = np.inf
    got = F.conv2d_sparse_filter(F.filter_compress(dev(wt)), dev(x), (1, 1), (2, 2), dev(b), False).cpu().numpy()
    assert np.array_equal(got, want)
    # compressed activation, Inf in the bank: outputs whose taps at that channel are all zero stay finite
    x, wt, b = inputs.random_layer(8, n, c, k, h, w, 3, 3, 1.0, integer=True, x_zero_frac=0.5)
    x[0, 11, :7] = 0.0
    wt[3, 11, 1, 1] = np.inf
    want = oracle.conv2d_dense(x, np.where(np.isinf(wt), 0, wt).astype(np.float32), (1, 1), (1, 1), None, False)
    xs = F.input_compress(dev(x))
    for y in (F.conv2d_sparse_input(xs, dev(wt), (1, 1), (1, 1)),
              F.conv2d_sparse_input_prepared(xs, F.dense_filter_prepare(dev(wt)), (1, 1), (1, 1))):
        y = y.cpu().numpy()
        assert np.array_equal(y[0, 3, :6], want[0, 3, :6])          # rows 0..5 see channel 11 only where it is zero
        hit = x[0, 11, 7:13] != 0
        assert np.array_equal(np.isfinite(y[0, 3, 7:13]), ~hit)
        assert np.isfinite(y[0, :3]).all() and np.isfinite(y[0, 4:]).all()
