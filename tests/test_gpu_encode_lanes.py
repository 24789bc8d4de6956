"""Encode with a lane per query, bit for bit against the CPU oracle: every number of feature words up to 8, at numbers of basis
rows and of parity-check rows around the rows that are read at a time."""
import numpy as np
import pytest

import parity
import synth
from test_gpu_parity import _large_context

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nq,stride", [(3000, 8), (200_000, 8), (3000, 4), (5000, 2)])
def test_encode_lane_rows(require_gpu, nq, stride):
    from paper_2608_20532_amd import f2gpu as f2
    rng = np.random.default_rng(nq + stride)
    n_bits, rows = [], []
    for n in (5, 62, 63, 64, 127, 128, 190, 192, 255, 256, 320, 383, 447, 500, 511):
        if (n + 63) // 64 > stride:
            continue
        d = n + 1
        for m in sorted({0, 1, 2, 3, 4, 5, d // 2 - 1, d // 2, (d + 1) // 2, d - 5, d - 4, d - 3, d - 2, d - 1, d + 40}):
            n_bits.append(n)
            rows.append(_large_context(rng, n, max(m, 0), "uniform"))
    wl = synth.custom_workload(n_bits, [len(r) for r in rows], rows)
    ref = parity.oracle_fit_threads(wl.rows, wl.row_off, wl.n_bits)
    model = parity.gpu_fit(f2, wl.rows, wl.row_off, wl.n_bits)
    ctx = rng.integers(0, wl.num_ctx, size=nq).astype(np.int32)
    x = np.zeros((nq, stride), np.uint64)
    W = (wl.n_bits.astype(np.int64) + 64) // 64 + 2
    for q in range(nq):                                     # sums of observations (in the span), some with a bit flipped
        c = int(ctx[q])
        m = int(wl.m_rows[c])
        n = int(wl.n_bits[c])
        if m:
            r = rows[c][rng.integers(0, m, size=1 if q % 3 else min(m, 3))]
            v = np.bitwise_xor.reduce(r, axis=0)[:W[c] - 2].copy()
            v[n // 64] &= ~np.uint64(1 << (n % 64)) if n % 64 else np.uint64(0)
            x[q, :min(stride, len(v))] = v[:stride]
        if q % 7 == 0 and n:
            b = int(rng.integers(0, n))
            x[q, b // 64] ^= np.uint64(1 << (b % 64))
    words, flags = f2.encode(model, parity.to_dev(ctx), parity.to_dev(x.reshape(-1)), stride)
    import torch
    torch.cuda.synchronize()
    r_words, r_flags = parity.oracle_encode_threads(ref, ctx, x.reshape(-1), stride)
    parity.compare_encode(words, flags, r_words, r_flags)
