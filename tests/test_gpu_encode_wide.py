"""Encode of wide contexts (more than 8 feature words: a wavefront per query), bit for bit against the CPU oracle."""
import numpy as np
import pytest

import synth
import parity
from test_gpu_parity import _large_context

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def f2(require_gpu):
    from paper_2608_20532_amd import f2gpu
    return f2gpu


def _mixed_contexts(rng):
    """Widths around the word boundaries, narrow and wide; ranks from zero through few rows and just over
    half (encoded by the basis) to nearly full and full (parity-check rows), contradictions among them."""
    specs = [(40, 60, "uniform"), (255, 300, "uniform"), (256, 0, "pool"), (256, 300, "uniform"), (319, 200, "uniform"),
             (320, 30, "pool"), (511, 70, "uniform"), (512, 300, "uniform"), (513, 700, "uniform"), (600, 380, "uniform"), (575, 64, "pool"),
             (1000, 65, "uniform"), (520, 350, "uniform"), (639, 560, "uniform"), (4094, 70, "pool"), (4095, 40, "uniform"), (4031, 3, "uniform"), (5, 9, "uniform")]
    n_bits, rows = [], []
    for n, m, kind in specs:
        n_bits.append(n)
        rows.append(_large_context(rng, n, m, "uniform" if n < 513 else kind))
    return synth.custom_workload(n_bits, [len(r) for r in rows], rows)


@pytest.mark.parametrize("nq,stride", [(1, 64), (777, 64), (777, 3), (777, 70), (20011, 17), (200000, 9)])
def test_encode_wide_contexts(f2, nq, stride):
    rng = np.random.default_rng(nq + stride)
    wl = _mixed_contexts(rng)
    ref = parity.oracle_fit_threads(wl.rows, wl.row_off, wl.n_bits)
    model = parity.gpu_fit(f2, wl.rows, wl.row_off, wl.n_bits)
    parity.compare_fit(model, ref)
    ctx = rng.integers(-1, wl.num_ctx + 1, size=nq).astype(np.int32)   # ids just out of range too
    if nq > 100000:                                                    # mostly cheap contexts for the oracle
        ctx = np.where(rng.random(nq) < 0.9, rng.integers(0, 7, size=nq), ctx).astype(np.int32)
    x = np.zeros((nq, stride), np.uint64)
    for c in range(wl.num_ctx):
        q = np.nonzero(ctx == c)[0]
        n, m = int(wl.n_bits[c]), int(wl.m_rows[c])
        fw = (n + 64) // 64
        if m == 0 or len(q) == 0:
            continue
        feat = wl.rows[wl.row_off[c]:wl.row_off[c + 1]].reshape(m, fw + 2)[:, :fw].copy()
        v = feat[rng.integers(0, m, size=len(q))] ^ feat[rng.integers(0, m, size=len(q))] ^ feat[rng.integers(0, m, size=len(q))]
        v[:, fw - 1] &= np.uint64((1 << (n & 63)) - 1)                 # x alone: constant and padding off
        w = min(fw, stride)
        x[q, :w] = v[:, :w]
    x[rng.random(nq) < 0.05, rng.integers(0, stride)] ^= np.uint64(1) << np.uint64(int(rng.integers(0, 64)))
    words, qf = f2.encode(model, parity.to_dev(ctx), parity.to_dev(x.reshape(-1)), stride)
    rw, rq = parity.oracle_encode_threads(ref, ctx, x.reshape(-1), stride)
    parity.compare_encode(words, qf, rw, rq)
    assert (rq == 0).any() or nq == 1
