"""Fits of batches between the sizes that the kernels' division was made for: the results at its lines, bit for bit against the
CPU oracle, and times that a batch must not exceed, each against other fits on the same card."""
import numpy as np
import pytest

import parity
import timing

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def f2(require_gpu):
    from paper_2608_20532_amd import f2gpu
    return f2gpu


@pytest.mark.parametrize("C", [4097, 24575, 24576, 24577, 24833])
def test_list_dealt_or_with_a_tail(f2, C):
    """Up to 96 contexts per workgroup the list is dealt out whole; beyond, its second half is taken in chunks."""
    rng = np.random.default_rng(C)
    n = rng.integers(0, 40, size=C).astype(np.int32)
    m = np.minimum(rng.geometric(1 / 8, size=C) - 1, 100)
    off = np.concatenate([[0], np.cumsum(m * ((n.astype(np.int64) + 64) // 64 + 2))])
    rows = rng.integers(0, 2 ** 63, size=max(int(off[-1]), 1), dtype=np.uint64) * np.uint64(2) + np.uint64(1)
    ref = parity.oracle_fit_threads(rows, off, n)
    parity.compare_fit(parity.gpu_fit(f2, rows, off, n), ref)


def test_time_of_8000_contexts(f2):
    """8,000 short contexts take no longer than two fits of 4,000 (measured 39 us against 2 x 26; 70 us with a list tail in chunks of 2)."""
    half, whole = (timing.fit_call(f2, np.full(C, 40), np.full(C, 60))[0] for C in (4000, 8000))
    t_half, t_whole = timing.medians([half, whole])
    assert t_whole < 2.1 * t_half, (t_half, t_whole)
