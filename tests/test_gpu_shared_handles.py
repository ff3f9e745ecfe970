"""One handle, several host threads, one stream: calls whose first launch leaves something in scratch for the second one
(the caller's bank taken apart, the sums of divided input channels) get their own operands' result, whatever the order in
which the threads come to launch.  Integers: every result has one right value, bit for bit."""
import threading

import numpy as np
import pytest
import torch

from paper_2212_08815_amd import inputs

pytestmark = pytest.mark.gpu

THREADS, CALLS = 4, 120


@pytest.fixture(scope="module")
def F():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2212_08815_amd import fscnn
    fscnn.lib()
    return fscnn


def together(call, want):
    """call(i) CALLS times in thread i, all on the default stream; how many results are not want[i]."""
    torch.cuda.synchronize()
    wrong, failed = [0] * THREADS, []

    def work(i):
        try:
            ys = [call(i) for _ in range(CALLS)]
            torch.cuda.synchronize()
            wrong[i] = sum(not torch.equal(y, want[i]) for y in ys)
        except Exception as e:   # noqa: BLE001 - a thread's failure has to reach the test
            failed.append(e)

    threads = [threading.Thread(target=work, args=(i,)) for i in range(THREADS)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    if failed:
        raise failed[0]
    return wrong


def test_an_activation_and_banks_of_several_callers(F):
    n, c, k, h, w = 2, 256, 256, 28, 28
    x = inputs.random_layer(1, n, c, k, h, w, 3, 3, 1.0, integer=True, x_zero_frac=0.5)[0]
    banks = [inputs.random_layer(10 + i, n, c, k, h, w, 3, 3, 1.0, integer=True)[1] for i in range(THREADS)]
    assert F.si_split_choice(n, c, h, w, k, (1, 1))[0] <= np.count_nonzero(x)
    want = [torch.nn.functional.conv2d(torch.from_numpy(x), torch.from_numpy(b), None, 1, 1).cuda() for b in banks]
    banks = [torch.from_numpy(b).cuda() for b in banks]
    s = F.input_compress(torch.from_numpy(x).cuda())
    assert together(lambda i: F.conv2d_sparse_input(s, banks[i], (1, 1), (1, 1)), want) == [0] * THREADS


@pytest.mark.parametrize("keep,pool", [(1.0, False), (0.1, True)])
def test_a_bank_and_activations_of_several_callers(F, keep, pool):
    """Divided over input channels: by the contraction in parts, and by the gather with the merged pool."""
    n, c, k, h, w = 1, 512, 512, 14, 14
    wt = inputs.random_layer(2, n, c, k, h, w, 3, 3, keep, integer=True)[1]
    xs = [inputs.random_layer(20 + i, n, c, 8, h, w, 3, 3, 1.0, integer=True)[0] for i in range(THREADS)]
    want = [torch.nn.functional.conv2d(torch.from_numpy(x), torch.from_numpy(wt), None, 1, 1) for x in xs]
    if pool:
        want = [torch.nn.functional.max_pool2d(y, 2) for y in want]
    want = [y.cuda() for y in want]
    xs = [torch.from_numpy(x).cuda() for x in xs]
    f = F.filter_compress(torch.from_numpy(wt).cuda())
    assert pool or F.sf_split_parts(f, n, h, w, (1, 1), (1, 1)) > 1
    assert together(lambda i: F.conv2d_sparse_filter(f, xs[i], (1, 1), (1, 1), pool=pool), want) == [0] * THREADS
