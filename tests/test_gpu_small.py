"""Small problems through NCHW tensors: configurations that stage through registers, the channel split
that the last part to arrive finishes.  Chunks that do not divide into the parts, an odd part, ragged
tiles and bands, the merged pool, leaky activation, emission; calls in a row and on two streams share no
state.  Integer data: any order of summation gives the same bits."""
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


@pytest.mark.parametrize("n,c,k,h,w,keep,pool", [
    (1, 512, 512, 14, 14, 0.10, False),   # deep: the channels split eight ways
    (1, 512, 500, 14, 14, 0.10, True),    # ... with the merged pool, ragged last channel group
    (1, 257, 33, 7, 7, 0.10, False),      # one channel past whole chunks; a part with fewer chunks
    (2, 130, 70, 9, 21, 0.30, True),      # odd bands under the pool
    (3, 100, 40, 13, 18, 0.10, False),    # three images: no bands, an idle image slot
    (5, 40, 72, 45, 61, 0.10, False),     # a second image group with three idle slots
    (1, 33, 17, 1, 3, 0.60, False),       # less than a band per row
])
def test_small_problems_are_exact_on_integers(F, n, c, k, h, w, keep, pool):
    x, wt, b = inputs.random_layer(n + c + k + h + w, n, c, k, h, w, 3, 3, keep, integer=True)
    want = oracle.conv2d_dense(x, wt, (1, 1), (1, 1), b, True)
    if pool:
        want = oracle.maxpool2x2(want)
    f, xd, bd = F.filter_compress(dev(wt)), dev(x), dev(b)
    for _ in range(3):   # the counters are clear again after every launch
        assert np.array_equal(F.conv2d_sparse_filter(f, xd, (1, 1), (1, 1), bd, True, pool=pool).cpu().numpy(), want)
    streams = [torch.cuda.Stream() for _ in range(2)]
    got = []
    for i in range(6):
        s = streams[i % 2]
        s.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(s):
            got.append(F.conv2d_sparse_filter(f, xd, (1, 1), (1, 1), bd, True, pool=pool))
    torch.cuda.synchronize()
    assert all(np.array_equal(g.cpu().numpy(), want) for g in got)
    if not pool:
        y = F.conv2d_sparse_filter(f, xd, (1, 1), (1, 1), bd, leaky=0.5).cpu().numpy()
        lin = oracle.conv2d_dense(x, wt, (1, 1), (1, 1), b, False)
        assert np.array_equal(y, np.where(lin > 0, lin, 0.5 * lin).astype(np.float32))
        rows, idx, val = F.input_export(F.conv2d_sparse_filter_emit(f, xd, (1, 1), (1, 1), bd, True))
        flat = want.transpose(0, 2, 3, 1).reshape(-1, k)
        p, ch = np.nonzero(flat)
        assert np.array_equal(idx, ch) and np.array_equal(val, flat[p, ch])
        assert np.array_equal(rows, np.concatenate([[0], np.cumsum((flat != 0).sum(1))]))


@pytest.mark.parametrize("k,c,r", [(1, 1, 3), (3, 683, 3), (65, 228, 3), (2, 2048, 1), (17, 40, 5)])
def test_bank_compression_at_the_edges_of_its_rounds(F, k, c, r):
    # rows of one element, of whole rounds of 2048, one short and one past them
    _, w, _ = inputs.random_layer(k + c, 1, c, k, 4, 4, r, r, 0.3)
    w[0] = 1.0
    if k > 1:
        w[1] = 0.0
    want = oracle.filter_compress(w)
    rp, ix, vl = F.filter_export(F.filter_compress(dev(w)))
    assert np.array_equal(rp, want[0]) and np.array_equal(ix, want[1]) and np.array_equal(vl.view(np.uint32), want[2].view(np.uint32))


@pytest.mark.parametrize("n,c,h,w", [(1, 8, 1, 1), (1, 8, 31, 33), (1, 8, 32, 32), (1, 128, 32, 32), (1, 9, 89, 92), (1, 17, 75, 73)])
def test_scan_at_the_edges_of_its_rounds(F, n, c, h, w):
    # (pixel, step of 8 channels) counts: 1, 1023, 1024, 16384 (the single work-group's last), 16376, 16425
    rng = np.random.default_rng(c * h)
    x = (rng.standard_normal((n, c, h, w)) * (rng.random((n, c, h, w)) < 0.4)).astype(np.float32)
    rows, idx, val = F.input_export(F.input_compress(dev(x)))
    flat = x.transpose(0, 2, 3, 1).reshape(-1, c)
    p, ch = np.nonzero(flat)
    assert np.array_equal(rows, np.concatenate([[0], np.cumsum((flat != 0).sum(1))]))
    assert np.array_equal(idx, ch) and np.array_equal(val, flat[p, ch])
