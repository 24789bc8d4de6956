"""The wide fit on streams whose rank grows by a few rows per block of 64, bit for bit against the CPU oracle: the chunks
of its list that are merged, where blocks complete them, and the ranks where they end."""
import numpy as np
import pytest

import parity
import timing

pytestmark = pytest.mark.gpu


def _growing(rng, n, new):
    """Rows of one context: block k brings new[k] generators of its own; its other rows are sums of earlier ones."""
    fw = (n + 64) // 64
    total = int(np.sum(new))
    gen = rng.integers(0, 2 ** 63, size=(max(total, 1), fw + 2), dtype=np.uint64) * np.uint64(2) + rng.integers(0, 2, size=(max(total, 1), fw + 2), dtype=np.uint64)
    gen[:, fw - 1] &= np.uint64((1 << ((n & 63) + 1)) - 1 if (n & 63) < 63 else 2 ** 64 - 1)
    rows, seen = [], 0
    for k in new:
        first, seen = seen, seen + int(k)
        r = np.zeros((64, fw + 2), np.uint64)
        if seen:
            for _ in range(3):
                r ^= gen[rng.integers(0, seen, size=64)]
            at = rng.permutation(64)[:int(k)]
            r[at] = gen[first:seen]
        rows.append(r)
    return np.concatenate(rows)


def _fit(f2, n_bits, rows):
    off = np.concatenate([[0], np.cumsum([r.size for r in rows])]).astype(np.int64)
    flat = np.concatenate([r.reshape(-1) for r in rows])
    n_bits = np.asarray(n_bits, np.int32)
    ref = parity.oracle_fit_threads(flat, off, n_bits)
    parity.compare_fit(parity.gpu_fit(f2, flat, off, n_bits), ref)
    return ref


PATTERNS = [[1] * 70, [5] * 14, [6] * 14, [7] * 11, [8] * 9, [3, 0, 2, 0, 1] * 14, [64, 1, 1, 1, 1, 60, 1, 1, 1, 28, 2, 2, 2, 2, 2, 30] * 2,
            [31, 1, 1, 31, 1, 1, 1, 29, 32, 1, 1, 1, 1, 28, 64], [33] + [1] * 31, [27, 1, 1, 1, 1, 1], [28, 1, 1, 1, 33, 1, 1, 1, 1, 1, 30, 64, 3]]


@pytest.mark.parametrize("count", [1, 2, 11, 40, 70, 140])
def test_rank_grows_slowly(require_gpu, count):
    """Eight, four, two and one workgroup for a context; contradictory rows among the last ones."""
    from paper_2608_20532_amd import f2gpu as f2
    rng = np.random.default_rng(count)
    n_bits, rows = [], []
    for k in range(count):
        n = [512, 575, 640, 1023, 1100][(k + count) % 5]
        r = _growing(rng, n, PATTERNS[k % len(PATTERNS)])
        if k % 3 == 1:
            r[-5:, -1] ^= np.uint64(9)
        n_bits.append(n)
        rows.append(r[:len(r) - k % 7])
    _fit(f2, n_bits, rows)


@pytest.mark.parametrize("count", [1, 70])
def test_rank_grows_to_full(require_gpu, count):
    """Full rank out of merged chunks, then rows that are only checked; or all but a few columns."""
    from paper_2608_20532_amd import f2gpu as f2
    rng = np.random.default_rng(count)
    n_bits, rows = [], []
    for k in range(count):
        if k < 2:
            n = 512 + k
            r = _growing(rng, n, [13] * 45 if k else [4] * 128 + [1, 0, 0])
            e = np.zeros((n + 1, r.shape[1]), np.uint64)          # every column by itself
            e[np.arange(n + 1), np.arange(n + 1) // 64] = np.uint64(1) << (np.arange(n + 1) % 64).astype(np.uint64)
            r = np.concatenate([r, e[k:], r[:100]])
        else:
            n, r = 520, _growing(rng, 520, [2] * (20 + k % 30))
        n_bits.append(n)
        rows.append(r)
    ref = _fit(f2, n_bits, rows)
    assert ref.rank[0] == 513


def test_time_of_slow_growth(require_gpu):
    """A stream that brings one new row in each block takes a few times what it does backwards, where the first
    blocks hold nearly all of its span (16 contexts of 600 bits and 256 blocks: measured 5.5 ms against 1.0 ms; 14 ms with a round for each batch)."""
    import torch
    from paper_2608_20532_amd import f2gpu as f2
    C, n, blocks = 16, 600, 256
    rng = np.random.default_rng(1)
    one = _growing(rng, n, [1] * blocks)
    calls = []
    for r in (np.ascontiguousarray(one[::-1]), one):
        rows = parity.to_dev(np.tile(r.reshape(-1), C))
        off = torch.arange(C + 1, device="cuda", dtype=torch.int64) * r.size
        model = f2.Model(np.full(C, n, np.int32))
        nb = f2.f2_fit_workspace_bytes(C)
        ws = f2.workspace(nb)

        def call(rows=rows, off=off, model=model, ws=ws):
            assert f2.f2_fit_batch(rows, rows.numel(), off, model, ws, nb) == f2.F2_OK
        calls.append(call)
    t = timing.medians(calls, rounds=3)
    assert t[1] < 8 * t[0], t


def test_time_of_many_tiny_contexts(require_gpu):
    """Wide contexts of one row, a workgroup each: 2,000 take less than three times what 64 of 64 rows do with four each (measured
    225 us against 97 us; 355 us where each workgroup invalidated its die's cache for its own data)."""
    from paper_2608_20532_amd import f2gpu as f2
    t = timing.medians([timing.fit_call(f2, np.full(C, 512), np.full(C, m))[0] for C, m in ((64, 64), (2000, 1))])
    assert t[1] < 3 * t[0], t


def test_timeout_with_merged_chunks(require_gpu, monkeypatch):
    """A wait that gives up at once leaves members with different lists: every one still finishes, the contexts are
    reported, narrow ones are right, and a fit with waits into the same buffers is exact."""
    import torch
    from paper_2608_20532_amd import f2gpu as f2
    rng = np.random.default_rng(5)
    n_bits = [512, 700, 1023, 40, 575]
    rows = [_growing(rng, n, PATTERNS[k]) for k, n in enumerate(n_bits)]
    off = np.concatenate([[0], np.cumsum([r.size for r in rows])]).astype(np.int64)
    flat = np.concatenate([r.reshape(-1) for r in rows])
    ref = parity.oracle_fit_threads(flat, off, np.asarray(n_bits, np.int32))
    monkeypatch.setenv("F2GPU_GROUP_SPIN_LIMIT", "0")
    model = parity.gpu_fit(f2, flat, off, n_bits)
    flags = parity.model_to_host(model)["flags"]
    assert (flags[[0, 1, 2, 4]] & f2.CTX_SYNC_TIMEOUT).all() and flags[3] == ref.flags[3]
    monkeypatch.delenv("F2GPU_GROUP_SPIN_LIMIT")
    nb = f2.f2_fit_workspace_bytes(model.num_ctx)
    ws, dev = f2.workspace(nb), parity.to_dev(flat)
    assert f2.f2_fit_batch(dev, dev.numel(), parity.to_dev(off), model, ws, nb) == f2.F2_OK
    torch.cuda.synchronize()
    parity.compare_fit(model, ref)
