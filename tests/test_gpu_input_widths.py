"""The compressor's work-group shapes: channel counts around every change of pixels and threads per group, and pixel counts that
leave the last group nearly empty, against the definition, bit for bit."""
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


# steps x pixels of a group: 256 and 257+ (C = 64, 65), the largest of each pixel count (327, 655, ... channels), 8192 channels;
# values per thread of the first pass: below and from four on (C = 127, 128)
@pytest.mark.parametrize("c", [1, 3, 64, 65, 72, 127, 128, 320, 321, 328, 648, 656, 1304, 1312, 2616, 2624, 5240, 5248, 8192])
@pytest.mark.parametrize("n,h,w", [(1, 1, 1), (2, 3, 11), (1, 1, 65)])
def test_lists_at_every_shape_of_a_group(F, c, n, h, w):
    rng = np.random.default_rng(c)
    for keep in (0.3, 1.0):
        x = rng.standard_normal((n, c, h, w)).astype(np.float32)
        x[rng.random(x.shape) >= keep] = 0.0
        x.flat[-1] = 0.5
        rows, idx, val = F.input_export(F.input_compress(torch.from_numpy(x).cuda()))
        flat = x.transpose(0, 2, 3, 1).reshape(-1, c)
        p, ch = np.nonzero(flat)
        assert np.array_equal(rows, np.concatenate([[0], np.cumsum((flat != 0).sum(1))]))
        assert np.array_equal(idx, ch)
        assert np.array_equal(val.view(np.uint32), flat[p, ch].view(np.uint32))


@pytest.mark.parametrize("k,c,r", [(1, 1, 1), (3, 255, 1), (2, 256, 3), (5, 257, 3), (2, 512, 3), (2, 513, 3), (1, 93, 5)])
def test_counts_of_a_filter_row(F, k, c, r):
    rng = np.random.default_rng(c)
    w = rng.standard_normal((k, c, r, r)).astype(np.float32) * (rng.random((k, c, r, r)) < 0.5)
    w = w.astype(np.float32)
    rows, idx, _ = F.filter_export(F.filter_compress(torch.from_numpy(w).cuda()))
    assert np.array_equal(rows, np.concatenate([[0], np.cumsum((w.reshape(k, -1) != 0).sum(1))]))
    assert np.array_equal(idx, np.nonzero(w.reshape(k, -1))[1])
