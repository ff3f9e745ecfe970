"""Device memory that passes from a destroyed handle to the next one: results where the next handle is made, filled and used while
the earlier one's work is still queued, other sizes on top of it, handles that other streams have used (their destruction
waits), how much is held, and that it is given back."""
import threading

import numpy as np
import pytest
import torch

from paper_2212_08815_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def F():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2212_08815_amd import fscnn
    fscnn.lib()
    return fscnn


def layer(seed, n, c, k, h, w, keep=0.4):
    x, wt, b = inputs.random_layer(seed, n, c, k, h, w, 3, 3, keep, integer=True, x_zero_frac=0.5)
    want = torch.nn.functional.conv2d(torch.from_numpy(x), torch.from_numpy(wt), torch.from_numpy(b), 1, 1).relu_()
    return tuple(torch.from_numpy(a).cuda() for a in (x, wt, b)) + (want,)


def passes(F, layers):
    """Handles live for one call; nothing waits for the device but the library."""
    out = []
    for x, wt, b, _ in layers:
        out.append(F.conv2d_sparse_input(F.input_compress(x), wt, (1, 1), (1, 1), b, True))
        out.append(F.conv2d_sparse_filter(F.filter_compress(wt), x, (1, 1), (1, 1), b, True))
    return out


# 8 x 130 x 36 x 33: 16 MB a handle; the smaller ones take the same memory, the largest does not fit it
SHAPES = [(8, 130, 140, 36, 33), (8, 100, 140, 33, 36), (8, 130, 140, 36, 33), (5, 60, 40, 28, 30), (8, 256, 140, 36, 33)]


def test_handles_in_turn_and_on_two_streams(F):
    layers = [layer(i, *s) for i, s in enumerate(SHAPES)]
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    got = passes(F, layers) + passes(F, layers)
    with torch.cuda.stream(side):
        other = passes(F, layers)
    got += passes(F, layers)
    s = F.input_compress(layers[0][0])             # filled on the default stream, used on both
    with torch.cuda.stream(side):
        y = F.conv2d_sparse_input(s, layers[0][1], (1, 1), (1, 1), layers[0][2], True)
    s.destroy()
    got += passes(F, layers)
    torch.cuda.synchronize()
    want = [w for *_, w in layers for _ in range(2)]
    assert torch.equal(y.cpu(), layers[0][3])
    for g, w in zip(got + other, want * 5):
        assert torch.equal(g.cpu(), w)


def test_threads_on_the_default_stream(F):
    layers = [layer(20 + i, *s) for i, s in enumerate(SHAPES)]
    torch.cuda.synchronize()
    results = {}
    threads = [threading.Thread(target=lambda t=t: results.update({t: passes(F, layers[t:] + layers[:t])})) for t in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    torch.cuda.synchronize()
    for t in range(4):
        for i, (*_, w) in enumerate(layers[t:] + layers[:t]):
            assert torch.equal(results[t][2 * i].cpu(), w) and torch.equal(results[t][2 * i + 1].cpu(), w)


def kept(F):
    """Bytes that destroyed handles have left."""
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    F.pool_trim()
    return torch.cuda.mem_get_info()[0] - before


def test_handles_of_a_stream_of_the_callers(F):
    """Their destruction waits for what is queued; the memory then serves any stream."""
    layers = [layer(40 + i, *s) for i, s in enumerate(SHAPES)]
    sides = [torch.cuda.Stream() for _ in range(2)]
    slow = torch.randn(4096, 4096, device="cuda")
    kept(F)
    got = []
    for turn in range(4):
        with torch.cuda.stream(sides[turn % 2]):
            got += passes(F, layers)
    got += passes(F, layers)
    kept(F)
    x, wt, b, want = layers[0]
    with torch.cuda.stream(sides[0]):
        s, f, done = F.input_compress(x), F.filter_compress(wt), torch.cuda.Event()
        for _ in range(20):
            slow @ slow
        y = F.conv2d_sparse_input(s, wt, (1, 1), (1, 1), b, True)
        done.record()
    s.destroy()
    assert done.query()
    torch.cuda.synchronize()
    for g, w in zip(got + [y], [w for *_, w in layers for _ in range(2)] * 5 + [want]):
        assert torch.equal(g.cpu(), w)
    f.destroy()
    assert kept(F) >= 16 << 20                              # the activation


def test_destroyed_inside_a_relaxed_capture(F):
    x, wt, b, want = layer(70, *SHAPES[0])
    side, y = torch.cuda.Stream(), torch.zeros(want.shape, device="cuda")
    f = F.filter_compress(wt)
    F.filter_prepare(f, 8, 36, 33, (1, 1), (1, 1))
    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        gone = [F.input_compress(x), F.filter_compress(wt)]
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=torch.cuda.Stream(), capture_error_mode="relaxed"):
        for h in gone:
            h.destroy()
        F.conv2d_sparse_filter(f, x, (1, 1), (1, 1), b, True, out=y)
    for _ in range(2):
        y.zero_()
        graph.replay()
        assert torch.equal(y.cpu(), want)


def test_a_divided_banks_memory_on_a_stream_of_the_callers(F):
    x, wt, _, _ = layer(60, 2, 512, 512, 14, 14, 1.0)
    kept(F)
    with torch.cuda.stream(torch.cuda.Stream()):
        f = F.filter_compress(wt)
        parts = F.sf_split_parts(f, 2, 14, 14, (1, 1), (1, 1))
        F.conv2d_sparse_filter(f, x, (1, 1), (1, 1))
        stored = f.nnz
        f.destroy()
    sums = 4 * parts * 2 * 512 * 14 * 14
    assert parts > 1 and sums >= 2 << 20                    # (smaller blocks are not kept)
    assert kept(F) >= 512 * 512 * 9 * 6 + 8 * stored + sums


def test_what_activations_leave_is_bounded_and_given_back(F):
    F.pool_trim()
    torch.cuda.synchronize()
    x = torch.zeros(8, 512, 64, 64, device="cuda")          # 201 MB a handle
    before = torch.cuda.mem_get_info()[0]
    handles = [F.input_compress(x) for _ in range(4)]
    for s in handles:
        s.destroy()
    torch.cuda.synchronize()
    kept = before - torch.cuda.mem_get_info()[0]
    assert 0 < kept <= 514 << 20
    F.pool_trim()
    assert before - torch.cuda.mem_get_info()[0] <= 2 << 20
    s = F.input_compress(x)
    assert s.nnz == 0
    rows, idx, _ = F.input_export(s)
    assert idx.size == 0 and not np.any(rows)
