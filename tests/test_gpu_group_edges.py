"""Interleaved-stream grouping at the edges of its kernels' tiles and of its dispatch, exactly, against a stable sort of the
rows by context (itself held against the row-by-row oracle below)."""
import numpy as np
import pytest

import parity
from oracle import group as G

MAX_N = G.MAX_N


def _by_sort(ids, rows, n_bits):
    """The grouping by a stable sort: (rows_out, row_off, dropped)."""
    S = rows.shape[1]
    W = (n_bits.astype(np.int64) + 64) // 64 + 2
    W = np.where((n_bits < 0) | (n_bits > MAX_N) | (W > S), 0, W)
    C = len(n_bits)
    known = (ids >= 0) & (ids < C)
    w = np.where(known, W[np.where(known, ids, 0)], 0)
    order = np.argsort(np.where(w > 0, ids, C), kind="stable")[:int((w > 0).sum())]
    take = np.arange(S)[None, :] < w[order, None]
    off = np.concatenate([[0], np.cumsum(W * np.bincount(ids[known], minlength=C))])
    return rows[order][take], off, int((w == 0).sum())


def _stream(C, R, S, skew, seed):
    rng = np.random.default_rng(seed)
    n_bits = rng.integers(0, max(1, min(64 * (S - 2), 4200)), size=C).astype(np.int32)
    if C > 8:
        n_bits[[1, 3, 5]] = [-1, 4096, min(64 * (S - 2), 4095)]   # two widths that are never valid, one above the stride
    ids = rng.integers(-2, C + 2, size=R) if not skew else np.minimum((C + 1) * rng.random(R) ** 12, C + 1).astype(np.int64) - 1
    return ids.astype(np.int32), rng.integers(0, 2 ** 63, size=(R, S), dtype=np.uint64), n_bits


@pytest.mark.parametrize("C,R,S,skew", [(1, 1, 3, False), (9, 300, 5, False), (40, 900, 9, True), (700, 2000, 70, False)])
def test_sort_equals_the_row_by_row_oracle(C, R, S, skew):
    ids, rows, n_bits = _stream(C, R, S, skew, R)
    for a, b in zip(_by_sort(ids, rows, n_bits), G.group_rows(ids, rows, S, n_bits)):
        assert np.array_equal(a, b)


# blocks of 8,192 rows up to 256 of them, tiles of 16,384 rows beyond; wavefronts of 64 rows; 9 bits of context per pass
# (511 | 512, 2^18 - 1 | 2^18); 4 | 8 lanes per row (stride 4 | 5); a scan of the offsets beyond 2^20 contexts
@pytest.mark.gpu
@pytest.mark.parametrize("C,R,S,skew", [
    (1, 1, 3, False), (2, 63, 4, False), (511, 8191, 4, True), (512, 8193, 5, False), (100, 65537, 11, True),
    (262143, 40000, 3, False), (262144, 40000, 3, False), (3, 2 ** 21 + 1, 3, True), (1000, 256 * 16384, 3, False),
    (600, 256 * 16384 + 1, 4, True), (80000, 256 * 16384 + 70001, 3, False), (2 ** 20, 5000, 3, False),
    (2 ** 20 + 1, 5000, 3, False), (30, 3000, 70, False)])
def test_group_edges(require_gpu, C, R, S, skew):
    import torch
    from paper_2608_20532_amd import f2gpu as f2
    ids, rows, n_bits = _stream(C, R, S, skew, C + R)
    out, off, dropped = f2.group(parity.to_dev(ids), parity.to_dev(rows.reshape(-1)), S, parity.to_dev(n_bits))
    torch.cuda.synchronize()
    r_out, r_off, r_drop = _by_sort(ids, rows, n_bits)
    off = parity.host(off, np.int64)
    assert int(parity.host(dropped, np.int64)[0]) == r_drop and np.array_equal(off, r_off)
    assert np.array_equal(parity.host(out, np.uint64)[:int(off[-1])], r_out)
