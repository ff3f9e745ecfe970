"""The contraction in bfloat16 parts: every tile, for both extents, at sizes where it can go wrong (one pixel per row,
tiles that end inside a row, rows that cross images, panels, rows whose last load of four overlaps the one before,
channel and filter counts off every multiple), that all parts of both operands count, values of any magnitude and of one sign, Inf
and NaN, and calls that capture or leave no room for its copy of the bank."""
import numpy as np
import pytest
import torch

import oracle
from paper_2212_08815_amd import inputs
from parity import assert_parity

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


TILES = [
    (0, True, 8, 9, 33, 56, 109, 3, (1, 1)), (1, False, 9, 58, 132, 57, 31, 3, (1, 1)), (1, True, 8, 12, 17, 44, 130, 3, (1, 1)),
    (2, False, 9, 9, 86, 52, 43, 3, (1, 1)), (2, True, 8, 10, 17, 36, 125, 3, (1, 1)), (3, False, 7, 12, 138, 37, 41, 3, (1, 1)),
    (3, True, 8, 9, 17, 57, 57, 3, (1, 1)), (4, False, 7, 11, 78, 48, 13, 3, (1, 1)), (4, True, 5, 11, 17, 18, 100, 3, (1, 1)),
    (5, True, 9, 9, 65, 26, 127, 3, (1, 1)), (6, False, 9, 48, 74, 55, 49, 3, (1, 1)), (6, True, 5, 9, 73, 41, 101, 3, (1, 1)),
    (7, False, 1, 10, 67, 4, 4, 3, (2, 2)), (7, True, 4, 10, 17, 4, 20, 3, (2, 2)), (8, False, 5, 35, 143, 53, 11, 3, (1, 1)),
    (8, True, 7, 33, 18, 33, 37, 3, (1, 1)), (9, False, 1, 15, 33, 5, 5, 3, (1, 1)), (9, True, 1, 14, 25, 3, 16, 3, (1, 1)),
    (3, False, 9, 67, 135, 57, 17, 5, (1, 1)), (3, True, 7, 9, 20, 57, 78, 5, (1, 1)), (4, False, 8, 9, 138, 47, 9, 5, (1, 1)),
    (4, True, 8, 9, 17, 14, 104, 5, (1, 1)), (7, True, 9, 10, 69, 41, 34, 5, (1, 1)), (8, False, 9, 40, 69, 56, 9, 5, (1, 1)),
    (8, True, 6, 36, 18, 31, 46, 5, (1, 1)), (9, False, 1, 70, 19, 5, 5, 5, (1, 1)), (9, True, 1, 104, 24, 8, 8, 5, (1, 1)),
]


@pytest.mark.parametrize("tile,wide,n,c,k,h,w,r,stride", TILES)
def test_every_tile(F, tile, wide, n, c, k, h, w, r, stride):
    pad = (r // 2, r // 2)
    conv = torch.nn.functional.conv2d
    # integers: every partial sum is exact, so any order of summation gives the same bits
    x, wt, b = inputs.random_layer(n + c + k + h + w, n, c, k, h, w, r, r, 1.0, integer=True)
    f = F.filter_compress(dev(wt))
    t, panels = F.sf_split_choice(f, n, h, w, stride, pad)
    assert t == tile and (panels > 1) == wide
    want = conv(torch.from_numpy(x), torch.from_numpy(wt), torch.from_numpy(b), stride, pad).relu_()
    assert torch.equal(F.conv2d_sparse_filter(f, dev(x), stride, pad, dev(b), True).cpu(), want)
    # every bit of x, then of w: each output is one product by 1 (or its taps lie outside: 0)
    rng = np.random.default_rng(c)
    bits = (rng.integers(1 << 23, 1 << 24, (n, c, h, w)) * rng.choice([-1.0, 1.0], (n, c, h, w))).astype(np.float32)
    one = np.ones((k, c, r, r), np.float32)
    ch = c - 1
    one[:, ch] = 0
    one[:, ch, r // 2, r // 2] = 1
    xs = np.zeros_like(bits)
    xs[:, ch] = bits[:, ch]
    f = F.filter_compress(dev(one))
    assert F.sf_split_choice(f, n, h, w, stride, pad)[0] == tile
    got = F.conv2d_sparse_filter(f, dev(xs), stride, pad).cpu()
    assert torch.equal(got, conv(torch.from_numpy(xs), torch.from_numpy(one), None, stride, pad))
    wb = (rng.integers(1 << 23, 1 << 24, (k, c, r, r)) * rng.choice([-1.0, 1.0], (k, c, r, r))).astype(np.float32)
    xs = np.zeros_like(bits)
    xs[n - 1, ch, h // 2, w // 2] = 0.5
    f = F.filter_compress(dev(wb))
    got = F.conv2d_sparse_filter(f, dev(xs), stride, pad).cpu()
    assert torch.equal(got, conv(torch.from_numpy(xs), torch.from_numpy(wb), None, stride, pad))


@pytest.mark.parametrize("n,c,k,h,w,r,scale", [
    (8, 155, 130, 29, 31, 3, 0), (8, 33, 40, 27, 27, 5, 0),
    (8, 140, 128, 33, 30, 3, 60),         # magnitudes from 2^-60 to 2^60, different from pixel to pixel
    (8, 128, 128, 28, 32, 3, -1),         # all tiny: products are subnormal
])
def test_random_data_stays_within_the_fp32_bound(F, n, c, k, h, w, r, scale):
    x, wt, b = inputs.random_layer(n + c + k, n, c, k, h, w, r, r, 0.7, bias=scale == 0)
    if scale > 0:
        x = np.ldexp(x, np.random.default_rng(1).integers(-scale, scale + 1, x.shape)).astype(np.float32)
    elif scale < 0:
        x = np.ldexp(x, -100).astype(np.float32)
        wt = np.ldexp(wt, -20).astype(np.float32)
    f = F.filter_compress(dev(wt))
    assert F.sf_split_choice(f, n, h, w, (1, 1), (r // 2, r // 2))[0] >= 0
    csr = oracle.filter_compress(wt)
    want, a = oracle.conv2d_sparse_filter(x, csr, wt.shape, (1, 1), (r // 2, r // 2), b, False, want_abs=True)
    got = F.conv2d_sparse_filter(f, dev(x), (1, 1), (r // 2, r // 2), None if b is None else dev(b), False).cpu().numpy()
    assert_parity(got, want, a, int(np.diff(csr[0]).max()), "parts")


# The fp32 unit's error is 2e-7 of the result in 2-norm here (1152 products), this one's 0.5e-7 to 1e-7.  Rounding to nearest leaves no
# mean over a million results (1e-10 .. 1e-9 of the mean magnitude, 1e-7 over the root of their number); an accumulator of
# the 72 instructions that cut towards zero would move sums of one sign by some 2^-24 of it.
@pytest.mark.parametrize("xe,we", [(0, 0), (-110, 60), (-124, 60), (-140, 100), (60, -124), (100, -140), (-60, -60), (110, -110), (120, -120)])
@pytest.mark.parametrize("sign", [False, True])
def test_precision_holds_at_any_magnitude_and_for_one_sign(F, xe, we, sign):
    n, c, k, h, w = 4, 128, 128, 44, 40
    x, wt, _ = inputs.random_layer(5, n, c, k, h, w, 3, 3, 1.0, bias=False)
    if sign:
        x, wt = np.abs(x), np.abs(wt)
    x = np.ldexp(np.maximum(x, 0).astype(np.float64), xe).astype(np.float32)     # (subnormals keep the bits they have)
    wt = np.ldexp(wt.astype(np.float64), we).astype(np.float32)
    want = torch.nn.functional.conv2d(torch.from_numpy(x).double(), torch.from_numpy(wt).double(), None, 1, 1)
    f = F.filter_compress(dev(wt))
    assert F.sf_split_choice(f, n, h, w, (1, 1), (1, 1))[0] >= 0
    assert F.si_split_choice(n, c, h, w, k, (1, 1))[0] <= np.count_nonzero(x)
    for got in (F.conv2d_sparse_filter(f, dev(x), (1, 1), (1, 1)), F.conv2d_sparse_input(F.input_compress(dev(x)), dev(wt), (1, 1), (1, 1))):
        off = got.double().cpu() - want
        assert off.norm() <= 1.5e-7 * want.norm()
        assert not sign or abs(off.mean()) <= 1e-8 * want.mean()


def test_values_that_are_not_finite_or_round_to_infinity(F):
    """Only stored entries meet them, a filter without an entry there does not see them; the largest floats
    have no finite first part and are multiplied all the same."""
    n, c, k, h, w = 8, 120, 128, 34, 32
    x, wt, b = inputs.random_layer(7, n, c, k, h, w, 3, 3, 0.8, integer=True)
    x[0, 5, 6, 7], x[1, 119, 0, 0], x[1, 3, 12, 12] = np.inf, np.nan, -np.inf
    wt[::2, [3, 5]] = 0.0
    wt[1::4, 119] = 0.0
    fin = np.isfinite(x)
    want = oracle.conv2d_dense(np.where(fin, x, 0).astype(np.float32), wt, (1, 1), (1, 1), b, False)
    met = oracle.conv2d_dense((~fin).astype(np.float32), (wt != 0).astype(np.float32), (1, 1), (1, 1), None, False) > 0
    f = F.filter_compress(dev(wt))
    assert F.sf_split_choice(f, n, h, w, (1, 1), (1, 1))[0] >= 0
    got = F.conv2d_sparse_filter(f, dev(x), (1, 1), (1, 1), dev(b), False).cpu().numpy()
    assert np.array_equal(np.isfinite(got), ~met) and np.array_equal(got[~met], want[~met])
    # an Inf weight: Inf where it meets a pixel, finite where it falls outside the image
    x, wt, b = inputs.random_layer(9, n, c, k, h, w, 3, 3, 0.8, integer=True)
    x = np.abs(x) + 1
    wt[3, 7, 0, 0] = np.inf
    want = oracle.conv2d_dense(x, np.where(np.isinf(wt), 0, wt).astype(np.float32), (1, 1), (1, 1), b, False)
    want[:, 3, 1:, 1:] = np.inf
    got = F.conv2d_sparse_filter(F.filter_compress(dev(wt)), dev(x), (1, 1), (1, 1), dev(b), False).cpu().numpy()
    assert np.array_equal(got, want)
    big = np.float32(3.4e38)
    x = np.zeros_like(x)
    x[:, 7, 5, 5] = big
    wt = np.where(wt == 0, 0, np.float32(0.5)).astype(np.float32)
    want = oracle.conv2d_dense(x, wt, (1, 1), (1, 1), None, False)
    got = F.conv2d_sparse_filter(F.filter_compress(dev(wt)), dev(x), (1, 1), (1, 1)).cpu().numpy()
    assert np.array_equal(got, want) and (got == big / 2).any()


def test_captured_with_and_without_its_plan(F):
    x, wt, b = inputs.random_layer(21, 8, 130, 128, 36, 33, 3, 3, 0.5, integer=True)
    want = torch.nn.functional.conv2d(torch.from_numpy(x), torch.from_numpy(wt), torch.from_numpy(b), (1, 1), (1, 1)).relu_()
    xd, bd = dev(x), dev(b)
    for prepared in (True, False):
        f, y = F.filter_compress(dev(wt)), torch.zeros(want.shape, device="cuda")
        assert F.sf_split_choice(f, 8, 36, 33, (1, 1), (1, 1))[0] >= 0
        if prepared:
            F.filter_prepare(f, 8, 36, 33, (1, 1), (1, 1))
        else:     # what serves it then is a gather configuration, whose plan has to be there
            F.filter_prepare(f, 8, 36, 33, (1, 1), (1, 1), F.sf_variant_choice(f, 8, 36, 33))
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, capture_error_mode="relaxed"):
            F.conv2d_sparse_filter(f, xd, (1, 1), (1, 1), bd, True, out=y)
        for _ in range(3):
            y.zero_()
            torch.cuda.synchronize()
            graph.replay()
            torch.cuda.synchronize()
            assert torch.equal(y.cpu(), want)
            assert torch.equal(F.conv2d_sparse_filter(f, xd, (1, 1), (1, 1), bd, True).cpu(), want)
