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


def _mix(rng, shapes):
    """(n, m) of every context, shuffled, from (count, widths, rows) entries."""
    n = np.concatenate([rng.choice(w, size=c) for c, w, _ in shapes])
    m = np.concatenate([rng.choice(r, size=c) for c, _, r in shapes])
    p = rng.permutation(len(n))
    return n[p].astype(np.int32), m[p]


SHORT, LONG, FOUR_LONG, FOUR, GROUP = ([3, 30, 62], [2, 20, 40]), ([20, 60], [400, 700]), ([193, 255], [321, 400]), ([192, 250], [30, 320]), ([300, 40], [130, 4100])


@pytest.mark.parametrize("short,long,four_long,four,group", [
    (0, 65, 0, 0, 0), (0, 0, 65, 0, 0), (300, 100, 100, 3, 56), (300, 100, 100, 3, 57), (300, 70, 190, 9, 2), (1200, 280, 0, 5, 3),
    (1200, 280, 9, 300, 3), (4096, 250, 5, 5, 5), (4096, 250, 5, 5, 1), (4095, 250, 2, 5, 5), (4095, 769, 2, 0, 1), (4096, 4, 0, 2, 257), (4096, 260, 3, 300, 257),
    (4095, 4, 0, 2, 257), (100, 200, 0, 300, 60),
    (40, 300, 20, 3, 60), (96, 300, 20, 3, 60), (1700, 280, 3, 600, 3), (1690, 280, 3, 599, 3), (4096, 4, 0, 2, 513), (0, 260, 0, 0, 1),
    (0, 0, 300, 10, 5), (78, 0, 300, 10, 5), (79, 0, 300, 10, 5), (0, 0, 300, 300, 5), (20, 9, 700, 60, 8), (20, 9, 700, 61, 8)])
def test_division_at_its_lines(f2, short, long, four_long, four, group):
    """A workgroup for each long and group context, or one too few; long ones beside short ones or behind them; more
    group contexts than workgroups."""
    rng = np.random.default_rng(short + 3 * long + 5 * four_long + 7 * four + 11 * group)
    n, m = _mix(rng, [(c, *k) for c, k in zip((short, long, four_long, four, group), (SHORT, LONG, FOUR_LONG, FOUR, GROUP))])
    off = np.concatenate([[0], np.cumsum(m * ((n.astype(np.int64) + 64) // 64 + 2))])
    rows = rng.integers(0, 2 ** 63, size=max(int(off[-1]), 1), dtype=np.uint64) * np.uint64(2) + np.uint64(1)
    ref = parity.oracle_fit_threads(rows, off, n)
    parity.compare_fit(parity.gpu_fit(f2, rows, off, n), ref)


@pytest.mark.parametrize("count", [65, 257, 900])
def test_lines_between_short_and_long(f2, count):
    """Contexts on both sides of 320 rows and of 20,480 rows x columns, of one to four words."""
    shapes = np.array([(63, 320), (63, 321), (39, 512), (39, 513), (31, 640), (31, 641), (127, 320), (127, 321), (191, 320), (191, 321), (255, 320), (255, 321),
                       (10, 30)])
    rng = np.random.default_rng(count)
    n, m = shapes[rng.integers(0, len(shapes), size=count)].T
    n = n.astype(np.int32)
    off = np.concatenate([[0], np.cumsum(m * ((n.astype(np.int64) + 64) // 64 + 2))])
    rows = rng.integers(0, 2 ** 63, size=int(off[-1]), dtype=np.uint64) * np.uint64(2) + np.uint64(1)
    ref = parity.oracle_fit_threads(rows, off, n)
    parity.compare_fit(parity.gpu_fit(f2, rows, off, n), ref)


def test_time_of_a_few_long_contexts(f2):
    """20 long contexts beside 4,000 short ones take little more than by themselves (67 us against 59; 107 us with one
    wavefront for each), and 400 beside 1,600 or 8,000 no more than one batch after the other (77 against 24 + 62, 94 against 38 + 65; 117 and 138 us so)."""
    few, alone, mixed, short, long, many, shorts = (
        timing.fit_call(f2, np.repeat([40, 30], c), np.repeat([60, 4000], c))[0]
        for c in ((4000, 20), (0, 65), (1600, 400), (1600, 0), (0, 400), (8000, 400), (8000, 0)))
    t = timing.medians([few, alone, mixed, short, long, many, shorts])
    assert t[0] < 1.45 * t[1], t
    assert t[2] < 1.15 * (t[3] + t[4]), t
    assert t[5] < 1.15 * (t[6] + t[4]), t


def test_time_of_a_few_short_contexts(f2):
    """75 short contexts among 425 long ones take little more than the long ones alone (54 us against 52; 68 us with the
    short ones in a kernel before the others)."""
    n = np.random.default_rng(500).integers(40, 98, 425)
    n2 = np.concatenate([n, np.full(75, 24)])
    t = timing.medians([timing.fit_call(f2, k, 20 * k)[0] for k in (n, n2)])
    assert t[1] < 1.2 * t[0], t


def test_time_of_long_contexts_of_four_words(f2):
    """65 contexts of 221 columns and 500 rows take little more than 64, which have a workgroup of eight wavefronts each
    (measured 129 us; 166 us with one wavefront for each), and 300 little more than 256 (145 us against 129 us; 181 us so)."""
    t = timing.medians([timing.fit_call(f2, np.full(C, 220), np.full(C, 500))[0] for C in (64, 65, 256, 300)])
    assert t[1] < 1.2 * t[0], t
    assert t[3] < 1.25 * t[2], t
