"""The contraction in bfloat16 parts where the input channels of a tile are divided over several work-groups: every number of parts
(a last one with fewer chunks among them) at ragged sizes, both extents, strides and the emitting call, bit for bit on integers;
Inf and NaN; two streams and graphs with and without the scratch."""
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


SIZES = [(1, 512, 512, 14, 14, 3, 1), (1, 512, 70, 7, 9, 3, 1), (2, 500, 130, 13, 11, 3, 1), (1, 390, 33, 17, 5, 3, 1), (3, 270, 64, 9, 8, 3, 1),
         (1, 210, 40, 7, 7, 5, 1), (1, 512, 96, 21, 23, 3, 2), (1, 1024, 65, 6, 7, 3, 1), (4, 320, 40, 7, 7, 3, 1), (1, 640, 128, 4, 40, 3, 1)]


@pytest.mark.parametrize("n,c,k,h,w,r,s", SIZES)
def test_integer_data_is_exact(F, n, c, k, h, w, r, s):
    x, wt, b = inputs.random_layer(n + c + k + h, n, c, k, h, w, r, r, 0.6, integer=True)
    f, xd, bd, st, pad = F.filter_compress(dev(wt)), dev(x), dev(b), (s, s), (r // 2, r // 2)
    assert F.sf_split_parts(f, n, h, w, st, pad) > 1
    want = torch.nn.functional.conv2d(torch.from_numpy(x), torch.from_numpy(wt), torch.from_numpy(b), st, pad).relu_()
    assert torch.equal(F.conv2d_sparse_filter(f, xd, st, pad, bd, True).cpu(), want)
    e = F.conv2d_sparse_filter_emit(f, xd, st, pad, bd, True)
    rows, idx, val = F.input_export(e)
    flat = want.permute(0, 2, 3, 1).reshape(-1, k).numpy()
    p, ch = np.nonzero(flat)
    assert np.array_equal(idx, ch) and np.array_equal(val, flat[p, ch])


def test_sizes_above_take_many_numbers_of_parts(F):
    seen = set()
    for n, c, k, h, w, r, s in SIZES:
        f = F.filter_compress(torch.ones(k, c, r, r, device="cuda"))
        seen.add(F.sf_split_parts(f, n, h, w, (s, s), (r // 2, r // 2)))
    assert len(seen) >= 4 and max(seen) >= 8


def test_random_data_and_repeats(F):
    x, wt, b = inputs.random_layer(3, 1, 500, 130, 13, 14, 3, 3, 0.3)
    f, xd, bd = F.filter_compress(dev(wt)), dev(x), dev(b)
    assert F.sf_split_parts(f, 1, 13, 14, (1, 1), (1, 1)) > 1
    csr = oracle.filter_compress(wt)
    want, a = oracle.conv2d_sparse_filter(x, csr, wt.shape, (1, 1), (1, 1), b, False, want_abs=True)
    got = F.conv2d_sparse_filter(f, xd, (1, 1), (1, 1), bd, False)
    assert_parity(got.cpu().numpy(), want, a, int(np.diff(csr[0]).max()), "parts")
    for _ in range(5):
        assert torch.equal(F.conv2d_sparse_filter(f, xd, (1, 1), (1, 1), bd, False), got)


def test_non_finite_values_meet_stored_entries_only(F):
    n, c, k, h, w = 1, 512, 128, 14, 14
    x, wt, b = inputs.random_layer(7, n, c, k, h, w, 3, 3, 0.8, integer=True)
    x[0, 5, 6, 7], x[0, 300, 0, 0] = np.inf, np.nan
    wt[::2, 5] = 0.0
    wt[1::4, 300] = 0.0
    fin = np.isfinite(x)
    want = oracle.conv2d_dense(np.where(fin, x, 0).astype(np.float32), wt, (1, 1), (1, 1), b, False)
    met = oracle.conv2d_dense((~fin).astype(np.float32), (wt != 0).astype(np.float32), (1, 1), (1, 1), None, False) > 0
    f = F.filter_compress(dev(wt))
    assert F.sf_split_parts(f, n, h, w, (1, 1), (1, 1)) > 1
    got = F.conv2d_sparse_filter(f, dev(x), (1, 1), (1, 1), dev(b), False).cpu().numpy()
    assert np.array_equal(np.isfinite(got), ~met) and np.array_equal(got[~met], want[~met])


@pytest.mark.parametrize("prepared", [True, False])
def test_streams_and_graphs(F, prepared):
    """A stream without scratch of its own captures the launch with one work-group per tile."""
    x, wt, b = inputs.random_layer(9, 1, 512, 140, 14, 13, 3, 3, 0.5, integer=True)
    f, xd, bd = F.filter_compress(dev(wt)), dev(x), dev(b)
    want = torch.nn.functional.conv2d(torch.from_numpy(x), torch.from_numpy(wt), torch.from_numpy(b), 1, 1).relu_()
    side = torch.cuda.Stream()
    F.filter_prepare(f, 1, 14, 13, (1, 1), (1, 1))
    torch.cuda.synchronize()
    if prepared:
        with torch.cuda.stream(side):
            F.filter_prepare(f, 1, 14, 13, (1, 1), (1, 1))
        torch.cuda.synchronize()
    y = torch.zeros(want.shape, device="cuda")
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        F.conv2d_sparse_filter(f, xd, (1, 1), (1, 1), bd, True, out=y)
    for _ in range(3):
        y.zero_()
        torch.cuda.synchronize()
        graph.replay()
        eager = F.conv2d_sparse_filter(f, xd, (1, 1), (1, 1), bd, True)      # at the same time, on the default stream
        torch.cuda.synchronize()
        assert torch.equal(y.cpu(), want) and torch.equal(eager.cpu(), want)
