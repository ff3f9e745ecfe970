"""The launches that compress a bank and build its plan, at the edges of their work: one row and thousands (beyond what one work-group scans),
empty and full rows, rows longer than a round, more chunks than the plan kernel keeps in LDS; calls of two threads at once, whose counts
and words are apart; activations around the number of groups that the fill pass adds up itself."""
import threading

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


def bank(seed, k, c, keep):
    rng = np.random.default_rng(seed)
    w = rng.integers(1, 4, (k, c, 3, 3)).astype(np.float32) * (rng.random((k, c, 3, 3)) < keep)
    w[::5] = 0.0
    w[1::7] = 1.0
    return w


def same(F, f, w):
    rp, ix, vl = oracle.filter_compress(w)
    got = F.filter_export(f)
    assert np.array_equal(got[0], rp) and np.array_equal(got[1], ix) and np.array_equal(got[2], vl)


@pytest.mark.parametrize("k,c,keep", [(1, 1, 1.0), (1, 700, 0.3), (15, 3, 0.5), (17, 512, 0.1), (300, 513, 0.05), (4096, 2, 0.4), (4097, 2, 0.4),
                                      (20, 4700, 0.02), (9, 4, 0.0)])
def test_banks_and_plans(F, k, c, keep):
    w = bank(k + c, k, c, keep)
    f = F.filter_compress(dev(w))
    same(F, f, w)
    # as every configuration's plan has it: the convolution of integers, bit for bit
    x = np.random.default_rng(3).integers(-3, 4, (4, c, 6, 5)).astype(np.float32)
    want = torch.nn.functional.conv2d(torch.from_numpy(x), torch.from_numpy(w), None, 1, 1)
    for v in (1, 3, 6, 7, 13, 26, 32, 38, 42):
        assert torch.equal(F.conv2d_sparse_filter(f, dev(x), (1, 1), (1, 1), variant=v).cpu(), want), v


def test_two_threads_at_once(F):
    ws = [bank(s, 200 + s, 64, 0.1) for s in range(2)]
    wd = [dev(w) for w in ws]
    torch.cuda.synchronize()
    got = [[], []]

    def work(i):
        with torch.cuda.stream(torch.cuda.Stream()):
            for _ in range(40):
                f = F.filter_compress(wd[i])
                F.filter_prepare(f, 1, 14, 14, (1, 1), (1, 1), 38)
                got[i].append(f)
            torch.cuda.current_stream().synchronize()

    threads = [threading.Thread(target=work, args=(i,)) for i in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for i in range(2):
        assert len(got[i]) == 40
        for f in got[i]:
            same(F, f, ws[i])


def test_a_handle_is_there_for_every_stream_at_once(F):
    """Compressed and planned on one stream, used on another without an event between."""
    w = bank(11, 256, 128, 0.2)
    wd = dev(w)
    x = dev(np.random.default_rng(5).integers(-3, 4, (1, 128, 20, 20)).astype(np.float32))
    want = torch.nn.functional.conv2d(x.cpu(), torch.from_numpy(w), None, 1, 1)
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    for _ in range(20):
        f = F.filter_compress(wd)
        F.filter_prepare(f, 1, 20, 20, (1, 1), (1, 1), 38)
        with torch.cuda.stream(side):
            y = F.conv2d_sparse_filter(f, x, (1, 1), (1, 1), variant=38)
            side.synchronize()
        assert torch.equal(y.cpu(), want)


@pytest.mark.parametrize("c", [8, 96])
@pytest.mark.parametrize("pixels", [2047 * 32 - 5, 2048 * 32, 2048 * 32 + 1])
def test_activations_around_the_scan(F, c, pixels):
    g = torch.Generator(device="cuda").manual_seed(pixels + c)
    x = torch.relu(torch.randn(1, c, 1, pixels, device="cuda", generator=g))
    rows, idx, val = F.input_export(F.input_compress(x))
    flat = x[0, :, 0].t().cpu().numpy()
    p, ch = np.nonzero(flat)
    assert np.array_equal(idx, ch) and np.array_equal(val, flat[p, ch])
    assert np.array_equal(rows, np.concatenate([[0], np.cumsum((flat != 0).sum(1))]))
