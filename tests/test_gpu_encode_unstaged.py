"""Encode of mid-sized batches over many contexts, where the grouped order is not staged (bins of several contexts, no
regrouping): a lane per query, wide contexts among them, bit for bit against the CPU oracle."""
import numpy as np
import pytest

import synth
from test_gpu_encode_mixed import _check, _queries
from test_gpu_parity import _large_context

pytestmark = pytest.mark.gpu

WIDE = [(300, 0), (300, 90), (320, 310), (383, 200), (447, 440), (500, 100), (511, 300), (511, 560),      # 5 to 8 words
        (512, 20), (513, 520), (600, 590), (700, 350), (1000, 300), (1500, 24)]                            # a wavefront each, or a lane


@pytest.mark.parametrize("max_n_bits", [None, -1])
@pytest.mark.parametrize("nq,share", [(196_608, 0.05), (198_399, 0.3)])
def test_unstaged_batch_with_wide_contexts(require_gpu, nq, share, max_n_bits):
    from paper_2608_20532_amd import f2gpu as f2
    rng = np.random.default_rng(nq)
    C = 12_400                                                      # above 8,192 bins, and 16 C above nq: neither fine bins nor regrouping
    assert 4 * C <= nq < 16 * C
    n_bits = rng.integers(2, 9, size=C)
    m = rng.integers(0, 9, size=C)
    at = rng.permutation(C)[:len(WIDE)]
    n_bits[at], m[at] = [n for n, _ in WIDE], [k for _, k in WIDE]
    rows = [_large_context(rng, int(n), int(k), "uniform") for n, k in zip(n_bits, m)]
    wl = synth.custom_workload(list(n_bits), list(m), rows)
    ctx = np.where(rng.random(nq) < share, rng.choice(at, size=nq), rng.integers(-1, C + 1, size=nq)).astype(np.int32)
    flags = _check(f2, wl, ctx, _queries(rng, wl, ctx, 24), max_n_bits)
    assert (flags == 0).any() and (flags[np.isin(ctx, at)] == 0).any()
