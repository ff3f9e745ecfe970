"""The contraction in bfloat16 parts through N4 tensors and with the merged pool: tiles that end inside a row, odd heights and widths under the
pool, widths of one and two, batches off every multiple of four, panels, strides, channels divided over work-groups; bit for bit on
integers, fp32's bound on random data, values that are not finite, captures without its plan."""
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


def call(F, f, x, n4, out4, pool, s, bias=None, relu=False, **kw):
    n = x.shape[0]
    xx = F.layout_convert(x, F.NCHW) if n4 else x
    y = F.conv2d_sparse_filter(f, xx, (s, s), (1, 1), bias, relu, x_layout=F.N4 if n4 else F.NCHW, y_layout=F.N4 if out4 else F.NCHW, n=n,
                               pool=pool, **kw)
    return F.layout_convert(y, F.N4, n=n) if out4 else y


def gathered(F, f, x, n4, pool, s):
    """The configuration that would serve the call otherwise."""
    return F.sf_variant_choice(f, x.shape[0], x.shape[2], x.shape[3], (s, s), n4, pool)


def parts(F, f, x, n4, out4, pool, s):
    n, _, h, w = x.shape
    return F.sf_serves(f, n, h, w, (s, s), (1, 1), F.N4 if n4 else F.NCHW, F.N4 if out4 else F.NCHW, pool) == F.SPLIT


CASES = [   # n, c, k, h, w, stride, N4 in, N4 out, pool
    (18, 512, 1024, 4, 4, 1, True, True, False), (5, 256, 130, 8, 8, 1, True, True, False), (8, 128, 96, 28, 28, 1, True, True, False),
    (6, 130, 70, 17, 19, 1, True, True, False), (9, 100, 65, 30, 3, 1, True, False, False), (4, 512, 96, 7, 1, 1, True, True, False),
    (7, 200, 80, 2, 2, 1, True, False, False), (4, 64, 64, 56, 61, 1, True, True, False), (8, 256, 256, 8, 8, 2, True, True, False),
    (11, 96, 130, 15, 9, 2, True, False, False), (3, 300, 64, 13, 13, 1, True, True, False), (1, 400, 64, 14, 14, 1, True, True, False),
    (1, 256, 256, 28, 28, 1, False, False, True), (3, 128, 100, 29, 31, 1, False, False, True), (2, 512, 512, 14, 14, 1, False, False, True),
    (1, 512, 70, 4, 7, 1, False, False, True), (5, 96, 160, 9, 33, 1, False, False, True), (2, 64, 128, 60, 44, 1, False, False, True),
    (8, 512, 512, 16, 16, 1, True, True, True), (6, 130, 96, 17, 19, 1, True, True, True), (9, 256, 70, 5, 4, 1, True, False, True),
    (4, 512, 64, 2, 2, 1, True, True, True), (12, 128, 128, 30, 31, 1, True, False, True), (4, 70, 64, 40, 62, 1, True, True, True),
]


@pytest.mark.parametrize("n,c,k,h,w,s,n4,out4,pool", CASES)
def test_layouts_and_pool(F, n, c, k, h, w, s, n4, out4, pool):
    # integers: every partial sum is exact, so any order of summation gives the same bits
    x, wt, b = inputs.random_layer(n + c + k + h + w, n, c, k, h, w, 3, 3, 1.0, integer=True)
    want = torch.nn.functional.conv2d(torch.from_numpy(x), torch.from_numpy(wt), torch.from_numpy(b), s, 1)
    want = (torch.nn.functional.max_pool2d(want, 2) if pool else want).relu_()
    f = F.filter_compress(dev(wt))
    assert parts(F, f, x, n4, out4, pool, s)
    assert torch.equal(call(F, f, dev(x), n4, out4, pool, s, dev(b), True).cpu(), want)
    # values of any size: not the gather kernel's sums, and within fp32's bound of the exact ones
    x, wt, b = inputs.random_layer(n + c + k, n, c, k, h, w, 3, 3, 1.0)
    f, xd = F.filter_compress(dev(wt)), dev(x)
    got = call(F, f, xd, n4, out4, pool, s)
    v = gathered(F, f, xd, n4, pool, s)
    assert v > 0 and not torch.equal(got, call(F, f, xd, n4, out4, pool, s, variant=v))
    exact = torch.nn.functional.conv2d(torch.from_numpy(x).double(), torch.from_numpy(wt).double(), None, s, 1)
    exact = torch.nn.functional.max_pool2d(exact, 2) if pool else exact
    assert (got.cpu().double() - exact).norm() <= 2.5e-7 * exact.norm()      # (9 c <= 4608 products: 1.7e-7 at the most)


@pytest.mark.parametrize("n4,pool", [(True, False), (True, True), (False, True)])
@pytest.mark.parametrize("n,c,k,h,w", [(6, 128, 128, 30, 32), (2, 512, 96, 14, 14)])     # whole; channels divided
def test_values_that_are_not_finite(F, n4, pool, n, c, k, h, w):
    """Only stored entries meet them."""
    x, wt, b = inputs.random_layer(7, n, c, k, h, w, 3, 3, 0.8, integer=True)
    x[0, 5, 6, 7], x[1, c - 1, 0, 0], x[1, 3, 12, 12] = np.inf, np.nan, -np.inf
    wt[::2, [3, 5]] = 0.0
    wt[1::4, c - 1] = 0.0
    fin = np.isfinite(x)
    want = torch.from_numpy(oracle.conv2d_dense(np.where(fin, x, 0).astype(np.float32), wt, (1, 1), (1, 1), b, False))
    met = torch.from_numpy(oracle.conv2d_dense((~fin).astype(np.float32), (wt != 0).astype(np.float32), (1, 1), (1, 1), None, False))
    if pool:
        want, met = torch.nn.functional.max_pool2d(want, 2), torch.nn.functional.max_pool2d(met, 2)
    met = met > 0
    f = F.filter_compress(dev(wt))
    assert parts(F, f, x, n4, n4, pool, 1)
    got = call(F, f, dev(x), n4, n4, pool, 1, dev(b)).cpu()
    assert torch.equal(got[~met], want[~met]) and 0 < met.sum() < met.numel()
    if not pool:                       # (a maximum over a unit with -Inf or NaN may be one of the others)
        assert torch.equal(torch.isfinite(got), ~met)


def test_images_past_the_last_one(F):
    """What an N4 tensor holds for them reaches nobody's results."""
    x, wt, b = inputs.random_layer(3, 6, 128, 128, 20, 20, 3, 3, 1.0, integer=True)
    want = torch.nn.functional.conv2d(torch.from_numpy(x), torch.from_numpy(wt), torch.from_numpy(b), 1, 1)
    f, x4 = F.filter_compress(dev(wt)), F.layout_convert(dev(x), F.NCHW)
    x4[1, :, :, :, 2:] = float("nan")
    for out4 in (True, False):
        assert parts(F, f, x, True, out4, False, 1)
        y = F.conv2d_sparse_filter(f, x4, (1, 1), (1, 1), dev(b), False, x_layout=F.N4, y_layout=F.N4 if out4 else F.NCHW, n=6)
        assert torch.equal((F.layout_convert(y, F.N4, n=6) if out4 else y).cpu(), want)


@pytest.mark.parametrize("n4,pool", [(True, False), (False, True)])
def test_captured_with_and_without_its_plan(F, n4, pool):
    n, c, k, h, w = 4, 256, 128, 16, 17
    x, wt, b = inputs.random_layer(21, n, c, k, h, w, 3, 3, 0.5, integer=True)
    want = torch.nn.functional.conv2d(torch.from_numpy(x), torch.from_numpy(wt), torch.from_numpy(b), 1, 1)
    want = torch.nn.functional.max_pool2d(want, 2) if pool else want
    lay = F.N4 if n4 else F.NCHW
    xd, bd = F.layout_convert(dev(x), F.NCHW) if n4 else dev(x), dev(b)
    for prepared in (True, False):
        f = F.filter_compress(dev(wt))
        assert parts(F, f, x, n4, n4, pool, 1)
        v = 0 if prepared else F.sf_variant_choice(f, n, h, w, n4=n4, pool=pool)
        F.filter_prepare(f, n, h, w, (1, 1), (1, 1), v, lay, lay, pool)
        run = lambda out=None: F.conv2d_sparse_filter(f, xd, (1, 1), (1, 1), bd, x_layout=lay, y_layout=lay, n=n, pool=pool, out=out)
        y = torch.zeros_like(run()) if prepared else torch.zeros(F.n4_shape(n, k, h, w) if n4 else want.shape, device="cuda")
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, capture_error_mode="relaxed"):
            run(y)
        for _ in range(3):
            y.zero_()
            torch.cuda.synchronize()
            graph.replay()
            torch.cuda.synchronize()
            assert torch.equal((F.layout_convert(y, F.N4, n=n) if n4 else y).cpu(), want)
            run()
