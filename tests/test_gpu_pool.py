"""Device memory that passes from a destroyed handle to the next one: results where the next handle is made, filled and used while
the earlier one's work is still queued, other sizes on top of it, handles that a second stream has used (their memory does
not pass), how much is held, and that it is given back."""
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
