"""Filters of a few entries among filters of many: the contraction in bfloat16 parts, whose single products are off by up to 2^-24 before they are
rounded, leaves a bank with a filter of one to three entries to kernels that multiply in fp32; empty filters do not count.  Banks that one
work-group counts and scans, and larger ones."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def F():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2212_08815_amd import fscnn
    fscnn.lib()
    return fscnn


def bank(k, c, entries):
    """entries: of the first filters, the last of which stand for the others"""
    rng = np.random.default_rng(k + len(entries))
    w = np.zeros((k, c * 9), np.float32)
    for i in range(k):
        n = entries[min(i, len(entries) - 1)]
        w[i, rng.choice(c * 9, n, replace=False)] = rng.standard_normal(n)
    return w.reshape(k, c, 3, 3)


@pytest.mark.parametrize("n4,pool", [(False, False), (True, False), (False, True), (True, True)])
def test_short_rows_are_as_exact_as_gathered(F, n4, pool):
    n, c, k, h = 8, 64, 256, 28
    w = bank(k, c, [1, 2, 3, 4] * 16 + [400])
    x = np.maximum(np.random.default_rng(2).standard_normal((n, c, h, h)), 0).astype(np.float32)
    lay = F.N4 if n4 else F.NCHW
    f, xd = F.filter_compress(torch.from_numpy(w).cuda()), torch.from_numpy(x).cuda()
    xx = F.layout_convert(xd, F.NCHW) if n4 else xd
    assert F.sf_serves(f, n, h, h, (1, 1), (1, 1), lay, lay, pool) != F.SPLIT
    y = F.conv2d_sparse_filter(f, xx, (1, 1), (1, 1), x_layout=lay, y_layout=lay, n=n, pool=pool)
    y = (F.layout_convert(y, F.N4, n=n) if n4 else y)[:, :64].cpu().double()
    want = torch.nn.functional.conv2d(torch.from_numpy(x).double(), torch.from_numpy(w[:64]).double(), None, 1, 1)
    size = torch.nn.functional.conv2d(torch.from_numpy(x).double(), torch.from_numpy(w[:64]).double().abs(), None, 1, 1)
    if pool:
        want, size = torch.nn.functional.max_pool2d(want, 2), torch.nn.functional.max_pool2d(size, 2)
    # one rounding of half a unit per entry, each of a sum no larger than the sum of magnitudes
    entries = torch.tensor([1, 2, 3, 4] * 16, dtype=torch.float64).view(1, 64, 1, 1)
    assert ((y - want).abs() <= entries * 2.0 ** -24 * size).all()


@pytest.mark.parametrize("k,c,n,h", [(256, 64, 8, 28), (4096, 32, 8, 8), (4100, 32, 8, 8), (16500, 16, 8, 8)])
def test_the_fewest_decide(F, k, c, n, h):
    for few, served in ((3, False), (4, True), (0, True)):
        many = min(300, 9 * c - 20)
        entries = [many] * 70 + [0, few] + [many]
        w = bank(72, c, entries)
        w = np.concatenate([w, np.repeat(w[:1], k - 72, 0)])[np.random.default_rng(few).permutation(k)]
        f = F.filter_compress(torch.from_numpy(w).cuda())
        assert (F.sf_serves(f, n, h, h, (1, 1), (1, 1)) == F.SPLIT) == served, few
