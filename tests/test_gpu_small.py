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


def test_split_scratch_made_under_capture_is_clear_before_the_first_replay(F):
    """A call of the channel split that was prepared on another stream only, captured (relaxed mode): its counters are
    clear for eager calls on that stream that come before the first replay, and after."""
    x, wt, b = inputs.random_layer(11, 1, 130, 26, 8, 8, 3, 3, 0.1, integer=True)
    want = oracle.conv2d_dense(x, wt, (1, 1), (1, 1), b, True)
    f, xd, bd = F.filter_compress(dev(wt)), dev(x), dev(b)
    run = lambda out=None: F.conv2d_sparse_filter(f, xd, (1, 1), (1, 1), bd, True, out=out)
    assert np.array_equal(run().cpu().numpy(), want)
    side, graph, y = torch.cuda.Stream(), torch.cuda.CUDAGraph(), torch.zeros(want.shape, device="cuda")
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=side, capture_error_mode="relaxed"):
        run(y)
    for _ in range(3):
        with torch.cuda.stream(side):
            eager = run(torch.zeros_like(y))
        torch.cuda.synchronize()
        assert np.array_equal(eager.cpu().numpy(), want)
        y.zero_()
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert np.array_equal(y.cpu().numpy(), want)


def test_graph_outlives_larger_calls_on_its_stream(F):
    """A captured call keeps its scratch when a later call on the same stream needs more."""
    side = torch.cuda.Stream()
    layers = {h: inputs.random_layer(12, 1, 130, 26, h, 8, 3, 3, 0.1, integer=True) for h in (8, 30)}
    wt, b = layers[8][1], layers[8][2]
    f, bd = F.filter_compress(dev(wt)), dev(b)
    x = {h: dev(layers[h][0]) for h in layers}
    want = {h: oracle.conv2d_dense(layers[h][0], wt, (1, 1), (1, 1), b, True) for h in layers}
    run = lambda h, out: F.conv2d_sparse_filter(f, x[h], (1, 1), (1, 1), bd, True, out=out)
    y = {h: torch.zeros(want[h].shape, device="cuda") for h in layers}
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.stream(side):
        run(8, y[8])
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=side):
        run(8, y[8])
    for _ in range(3):
        with torch.cuda.stream(side):
            run(30, y[30])
        y[8].zero_()
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert all(np.array_equal(y[h].cpu().numpy(), want[h]) for h in y)


def test_pool_of_scratch_is_bounded_and_given_back(F):
    _, wt, _ = inputs.random_layer(13, 1, 512, 512, 3, 3, 3, 3, 0.05)
    w, x, y = dev(wt), torch.randn(6, 512, 28, 28, device="cuda"), torch.empty(6, 512, 28, 28, device="cuda")
    F.pool_trim()
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    handles = [F.filter_compress(w) for _ in range(4)]
    for f in handles:
        F.conv2d_sparse_filter(f, x, (1, 1), (1, 1), out=y)
    torch.cuda.synchronize()
    scratch = before - torch.cuda.mem_get_info()[0]
    assert scratch > 4 * (16 << 20)               # a split launch: its parts are 16 MB and more
    for f in handles:
        f.destroy()
    kept = before - torch.cuda.mem_get_info()[0]
    assert 0 < kept <= 66 << 20
    F.pool_trim()
    assert before - torch.cuda.mem_get_info()[0] <= 2 << 20


@pytest.mark.parametrize("n,c,k,h,w,r,stride,pool,n4", [
    (1, 64, 40, 9, 9, 3, 1, False, False),     # parts of 16 KB: the last one to arrive adds them up
    (1, 512, 70, 14, 14, 3, 1, True, False),   # parts of a work-group beyond 128 KB: a launch of its own, merged pool
    (5, 120, 70, 17, 19, 3, 2, False, False),  # stride 2
    (5, 120, 70, 17, 19, 3, 2, False, True),   # ... N4 tensors, three idle image slots
    (6, 300, 70, 9, 11, 3, 1, True, True),     # N4, merged pool, odd rows
    (6, 300, 33, 15, 8, 3, 1, False, True),
    (4, 171, 393, 7, 7, 3, 1, False, True),    # tiles that are mostly padding, whose lanes leave and read nothing
    (5, 120, 35, 3, 5, 3, 1, False, True),     # ... three idle image slots, waves without a channel
    (7, 130, 70, 5, 7, 3, 1, True, True),      # ... merged pool: the odd row and column have no result
    (32, 256, 130, 8, 8, 3, 1, True, True),    # many parts into N4 tensors: the last one to arrive
    (4, 500, 40, 13, 13, 1, 1, False, True),   # 1x1
    (3, 400, 37, 12, 20, 1, 1, False, False),
])
def test_both_ways_to_add_up_the_parts_of_a_split(F, n, c, k, h, w, r, stride, pool, n4):
    x, wt, b = inputs.random_layer(n + c + k + h + w, n, c, k, h, w, r, r, 0.05, integer=True)
    pad = (r // 2, r // 2)
    want = oracle.conv2d_dense(x, wt, (stride, stride), pad, b, True)
    if pool:
        want = oracle.maxpool2x2(want)
    f, xd, lay = F.filter_compress(dev(wt)), dev(x), F.NCHW
    if n4:
        xd, lay = F.layout_convert(xd, F.NCHW), F.N4
    for _ in range(3):
        y = F.conv2d_sparse_filter(f, xd, (stride, stride), pad, dev(b), True, x_layout=lay, y_layout=lay, n=n, pool=pool)
        y = F.layout_convert(y, F.N4, n) if n4 else y
        assert np.array_equal(y.cpu().numpy(), want)


def test_choice_between_large_tiles_and_register_staging(F):
    """192 to 383 work-groups of the large tiles: they stay where records outweigh chunks (16 images, or 10 % stored at
    eight), the register-staged forms (35 and up) take nearly empty banks.  More groups: never."""
    def choice(n, c, k, hw, keep):
        _, wt, _ = inputs.random_layer(5, 1, c, k, 3, 3, 3, 3, keep)
        return F.sf_variant_choice(F.filter_compress(dev(wt)), n, hw, hw)
    assert choice(16, 512, 512, 28, 0.20) < 35
    assert choice(8, 512, 512, 28, 0.01) >= 35
    assert choice(32, 512, 512, 28, 0.01) < 35 and choice(4, 512, 512, 14, 0.10) >= 35


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


@pytest.mark.parametrize("k", [1, 1023, 1024, 1025, 16383, 16384, 16385, 20481])
def test_scan_at_the_edges_of_its_rounds(F, k):
    # one count per filter is scanned: rows of 1024, and from 16385 on tiles of 4096 instead of one work-group
    rng = np.random.default_rng(k)
    w = (rng.standard_normal((k, 3, 1, 1)) * (rng.random((k, 3, 1, 1)) < 0.4)).astype(np.float32)
    want = oracle.filter_compress(w)
    rp, ix, vl = F.filter_export(F.filter_compress(dev(w)))
    assert np.array_equal(rp, want[0]) and np.array_equal(ix, want[1]) and np.array_equal(vl.view(np.uint32), want[2].view(np.uint32))


@pytest.mark.parametrize("n,c,h,w", [
    (1, 8, 1, 1), (1, 8, 31, 33), (1, 8, 32, 32), (1, 128, 32, 32), (1, 9, 89, 92), (1, 17, 75, 73),
    # sums of groups of 32 pixels that are scanned: 1023, 1024, 1025; 16384, 16385
    (1, 3, 31, 1056), (1, 3, 32, 1024), (1, 3, 41, 800), (1, 1, 512, 1024), (1, 1, 3, 174763),
])
def test_activation_compression_at_the_edges_of_its_groups(F, n, c, h, w):
    rng = np.random.default_rng(c * h)
    x = (rng.standard_normal((n, c, h, w)) * (rng.random((n, c, h, w)) < 0.4)).astype(np.float32)
    rows, idx, val = F.input_export(F.input_compress(dev(x)))
    flat = x.transpose(0, 2, 3, 1).reshape(-1, c)
    p, ch = np.nonzero(flat)
    assert np.array_equal(rows, np.concatenate([[0], np.cumsum((flat != 0).sum(1))]))
    assert np.array_equal(idx, ch) and np.array_equal(val, flat[p, ch])
