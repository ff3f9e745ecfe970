"""The direct kernel with one and with four rows a thread, lanes that skip taps outside the image and lanes that do not: heights around its tiles, several output channels a work-group with a ragged last one,
strides, filters of no entry; bit for bit on integers, and an Inf weight that meets nothing outside the image."""
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


@pytest.mark.parametrize("n,c,k,h,w,r,s,pad", [(1, 6, 20, 7, 9, 5, 1, 2), (26, 5, 83, 40, 70, 5, 1, 2), (2, 4, 130, 33, 65, 7, 2, 3), (64, 3, 41, 17, 20, 5, 3, 1),
                                               (3, 3, 500, 9, 64, 7, 1, 3), (128, 2, 37, 16, 16, 5, 1, 0),
                                               (20, 3, 71, 8, 70, 5, 1, 2), (60, 4, 40, 2, 5, 5, 1, 2)])
def test_rows(F, n, c, k, h, w, r, s, pad):
    rng = np.random.default_rng(n + k)
    wt = rng.integers(1, 4, (k, c, r, r)).astype(np.float32) * (rng.random((k, c, r, r)) < 0.03)
    wt[::6] = 0.0
    x = rng.integers(1, 5, (n, c, h, w)).astype(np.float32)
    b = (np.arange(k) % 5 - 2).astype(np.float32)
    dev = lambda a: torch.from_numpy(a).cuda()
    want = torch.nn.functional.conv2d(torch.from_numpy(x), torch.from_numpy(wt), torch.from_numpy(b), s, pad)
    f = F.filter_compress(dev(wt))
    assert F.sf_serves(f, n, h, w, (s, s), (pad, pad)) == F.DIRECT
    assert torch.equal(F.conv2d_sparse_filter(f, dev(x), (s, s), (pad, pad), dev(b), True).cpu(), want.relu())
    if pad:
        wt[3] = 0.0
        wt[3, 0, 0, 0] = np.inf                    # meets x at (oy*s - pad, ox*s - pad)
        f = F.filter_compress(dev(wt))
        assert F.sf_serves(f, n, h, w, (s, s), (pad, pad)) == F.DIRECT
        got = F.conv2d_sparse_filter(f, dev(x), (s, s), (pad, pad)).cpu()[:, 3]
        first = -(-pad // s)
        assert (got[:, :first] == 0).all() and (got[:, :, :first] == 0).all() and torch.isinf(got[:, first:, first:]).all()


@pytest.mark.parametrize("n,c,k,h,w,r,s,entries,kind", [(1, 40, 300, 16, 16, 5, 1, 10, "DIRECT"), (3, 2, 30, 68, 74, 3, 3, 6, "DIRECT"), (4, 15, 75, 35, 21, 3, 3, 3, "DIRECT"),
                                                       (1, 3, 504, 215, 215, 5, 1, 15, "DIRECT"), (5, 15, 16, 26, 20, 3, 3, 18, "CONTRACT"),
                                                       (2, 3, 33, 63, 58, 5, 1, 17, "SPLIT"), (2, 95, 415, 24, 21, 5, 1, 130, "SPLIT")])
def test_choice(F, n, c, k, h, w, r, s, entries, kind):
    """By time where the direct kernel's sums are as exact as the contractions'; those keep filters of many entries."""
    rng = np.random.default_rng(1)
    wt = np.zeros((k, c * r * r), np.float32)
    for row in wt:
        row[rng.choice(c * r * r, entries, replace=False)] = 1.0
    f = F.filter_compress(torch.from_numpy(wt.reshape(k, c, r, r)).cuda())
    assert F.sf_serves(f, n, h, w, (s, s), (r // 2, r // 2)) == getattr(F, kind)
