"""The fit's division of a batch among its kernels, bit for bit against the CPU oracle: contexts at the edges of every class
(short, long, one, group) in batches that send each class to one kernel or the other, and batches whose list has a shared tail."""
import numpy as np
import pytest

import parity
import synth
from test_gpu_parity import _large_context

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def f2(require_gpu):
    from paper_2608_20532_amd import f2gpu
    return f2gpu


# (inputs, rows): half a word of features and one (31 | 32), one to five words, blocks of 64 rows, the lines between the classes
# (256 rows, where small batches change; rows x columns of 16,384 and 131,072; 4,096 rows; the lines at
# 320 rows and 20,480 are in test_gpu_fit_batches)
SHORT = [(0, 3), (1, 0), (1, 9), (30, 64), (31, 63), (31, 200), (32, 65), (40, 256), (40, 399), (62, 257), (63, 128), (63, 256), (64, 130), (100, 162),
         (126, 256), (127, 129), (128, 250), (190, 191), (191, 256), (7, 2048)]
LONG = [(40, 400), (63, 257), (127, 1023), (191, 683), (31, 4096), (190, 300)]
ONE = [(192, 5), (192, 256), (193, 65), (254, 257), (255, 256), (255, 512)]
GROUP = [(256, 130), (31, 4097), (191, 684), (255, 513), (319, 100), (320, 321), (383, 64), (384, 70), (447, 90), (511, 300), (5, 4200)]


def _contexts(rng, shapes, count):
    out = []
    for k in range(count):
        n, m = shapes[k % len(shapes)] if k < 2 * len(shapes) else shapes[int(rng.integers(len(shapes)))]
        rows = _large_context(rng, n, m, "pool" if k % 3 == 1 and m and n > 30 else "uniform")
        if k % 4 == 2 and m > 4:                                   # rows that repeat, one of them with another output
            rows[m // 2:] = rows[:m - m // 2]
            rows[m // 2, -1] ^= np.uint64(1 << 40)
        out.append((n, rows))
    return out


@pytest.mark.parametrize("short,long,one,group", [
    (70, 0, 0, 0), (60, 6, 6, 11), (300, 40, 13, 30), (40, 14, 12, 22), (0, 70, 0, 0), (0, 0, 70, 0), (0, 0, 0, 66), (24, 6, 300, 5),
    (30, 0, 0, 270), (10, 260, 6, 11)])
def test_fit_classes(f2, short, long, one, group):
    rng = np.random.default_rng(short + 7 * long + 11 * one + 13 * group)
    ctx = _contexts(rng, SHORT, short) + _contexts(rng, LONG, long) + _contexts(rng, ONE, one) + _contexts(rng, GROUP, group)
    ctx = [ctx[i] for i in rng.permutation(len(ctx))]
    wl = synth.custom_workload([n for n, _ in ctx], [len(r) for _, r in ctx], [r for _, r in ctx])
    ref = parity.oracle_fit_threads(wl.rows, wl.row_off, wl.n_bits)
    parity.compare_fit(parity.gpu_fit(f2, wl.rows, wl.row_off, wl.n_bits), ref)


@pytest.mark.parametrize("C,top", [(4095, 30), (4097, 130), (8193, 31), (30011, 62)])
def test_fit_shared_tail(f2, C, top):
    """Lists dealt out whole, around a context per wavefront and two, and one whose second half is taken in chunks."""
    rng = np.random.default_rng(C)
    n = rng.integers(0, top, size=C).astype(np.int32)
    m = np.minimum(rng.geometric(1 / 12, size=C) - 1, 200)
    fw = (n.astype(np.int64) + 64) // 64
    off = np.concatenate([[0], np.cumsum(m * (fw + 2))])
    rows = rng.integers(0, 2 ** 63, size=max(int(off[-1]), 1), dtype=np.uint64) * np.uint64(2) + np.uint64(1)
    ref = parity.oracle_fit_threads(rows, off, n)
    parity.compare_fit(parity.gpu_fit(f2, rows, off, n), ref)
