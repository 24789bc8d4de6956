"""The wide fit at the edges of its words, blocks and groups, bit for bit against the CPU oracle: widths around 64-bit and
128-column boundaries, rows around the 64-row blocks, full rank with rows left to check, and batches that give a context
eight, four, two or one workgroup."""
import numpy as np
import pytest

import parity
import synth
from test_gpu_parity import _large_context

pytestmark = pytest.mark.gpu

WIDTHS = [512, 513, 574, 575, 576, 639, 640, 703, 767, 1023, 1024, 1087, 2048, 4095]


@pytest.mark.parametrize("count,more", [(1, 1), (2, 0), (9, 0), (40, 3), (70, 0), (140, 2)])
def test_fit_wide_edges(require_gpu, count, more):
    from paper_2608_20532_amd import f2gpu as f2
    rng = np.random.default_rng(count)
    n_bits, rows = [], []
    for k in range(count):
        n = WIDTHS[(k * 5 + count) % len(WIDTHS)]
        m = [65, 64, 0, 1, 129, 63, 2, 200, 127][k % 9]
        if k % 10 == 0 and n <= 640:
            m = n + 1 + 90                                 # full rank, then a check of what is left
        r = _large_context(rng, n, m, "pool" if k % 4 == 3 and m else "uniform")
        if k % 5 == 1 and m > 3:                           # rows of the constant alone, the second contradictory
            r[1:3, :] = 0
            r[1:3, n // 64] = np.uint64(1) << np.uint64(n % 64)
            r[2, -1] = 5
        n_bits.append(n)
        rows.append(r)
    for k in range(more):                                  # and narrow contexts in the same batch
        n_bits.insert(k, 30 + 100 * k)
        rows.insert(k, _large_context(rng, 30 + 100 * k, 90, "uniform"))
    wl = synth.custom_workload(n_bits, [len(r) for r in rows], rows)
    ref = parity.oracle_fit_threads(wl.rows, wl.row_off, wl.n_bits)
    parity.compare_fit(parity.gpu_fit(f2, wl.rows, wl.row_off, wl.n_bits), ref)


@pytest.mark.parametrize("count", [5, 20, 70])
def test_full_rank_of_neighbours_of_other_widths(require_gpu, count):
    """Adjacent contexts of different widths at full rank (their areas meet within a cache line), groups of eight, four and
    two workgroups; some a few columns short of it, so that the whole basis is written."""
    from paper_2608_20532_amd import f2gpu as f2
    rng = np.random.default_rng(count)
    widths = ([641, 1023, 702, 1100, 831] * count)[:count] if count < 50 else rng.integers(600, 700, size=count)
    n_bits, rows = [], []
    for k, n in enumerate(widths):
        m = int(n) + 1 + [70, 0, 130, -1, 64, -3, 200][k % 7]
        r = _large_context(rng, int(n), m, "uniform")
        if k % 3 == 1:
            r[-2, -1] ^= np.uint64(3)
        n_bits.append(int(n))
        rows.append(r)
    wl = synth.custom_workload(n_bits, [len(r) for r in rows], rows)
    ref = parity.oracle_fit_threads(wl.rows, wl.row_off, wl.n_bits)
    parity.compare_fit(parity.gpu_fit(f2, wl.rows, wl.row_off, wl.n_bits), ref)
    assert (ref.rank == np.asarray(n_bits) + 1).any()


def test_more_blocks_than_the_tags_hold(require_gpu):
    """A context of more blocks than a list entry can name is one workgroup's: 2^19 blocks of rows that repeat seven, then
    a new row and a contradictory one, against the oracle's fit of the rows that differ."""
    import torch
    import oracle
    from paper_2608_20532_amd import f2gpu as f2
    rng = np.random.default_rng(9)
    n, m = 512, (1 << 19) * 64 + 100
    few = _large_context(rng, n, 8, "uniform")
    last = few[3:4].copy()
    last[0, -1] ^= np.uint64(1)
    rows = torch.empty((m, few.shape[1]), dtype=torch.int64, device="cuda")
    rows.copy_(parity.to_dev(few[:7])[torch.arange(m, device="cuda") % 7])
    rows[m - 40] = parity.to_dev(few[7])
    rows[m - 2] = parity.to_dev(last[0])
    wl = synth.custom_workload([n], [9], [np.concatenate([few, last])])
    ref = parity.oracle_fit_threads(wl.rows, wl.row_off, wl.n_bits)
    assert ref.rank[0] == 8 and ref.first_contra[0] == 8
    ref.first_contra[0] = m - 2
    model = f2.fit(rows.reshape(-1), torch.tensor([0, rows.numel()], device="cuda"), np.array([n], np.int32))
    torch.cuda.synchronize()
    parity.compare_fit(model, ref)
