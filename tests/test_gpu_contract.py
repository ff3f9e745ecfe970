"""The contraction on the matrix cores: dense-ish filter banks, filter extents without a gather
configuration, compressed activations with dense banks.  Sizes at the edges of its tiles: one pixel,
tiles that end inside a row, rows that cross images, panels of wide images, channel counts around the
slices of 16 and the rows of 16, chunks that end early; Inf and NaN."""
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


@pytest.mark.parametrize("n,c,k,h,w,r,s,stride,pad", [
    (1, 1, 1, 1, 1, 3, 3, (1, 1), (1, 1)),        # one pixel, one channel
    (1, 16, 64, 14, 14, 3, 3, (1, 1), (1, 1)),    # whole slices and rows
    (2, 17, 65, 13, 17, 3, 3, (1, 1), (1, 1)),    # one past them; tiles end inside a row
    (13, 33, 31, 3, 5, 3, 3, (1, 1), (0, 1)),     # one output row per image: a tile crosses many images
    (1, 70, 20, 9, 131, 3, 3, (1, 1), (1, 1)),    # panels, the last one narrower
    (7, 128, 130, 11, 11, 3, 3, (1, 1), (1, 1)),  # several chunks, ragged last rows
    (2, 40, 33, 12, 19, 5, 5, (1, 1), (2, 2)),    # an extent without a gather configuration
    (3, 20, 40, 23, 9, 7, 3, (2, 1), (3, 0)),     # ... at uneven strides
    (4, 9, 50, 10, 10, 2, 4, (1, 3), (0, 2)),     # ... filter narrower than the stride
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
