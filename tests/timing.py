"""Times of calls on the GPU, for tests that hold one call's time against another's on the same card."""
import statistics

import numpy as np


def medians(calls, rounds=7, budget_ms=2.0):
    """Median time in microseconds of each call (enqueued back to back, the calls taking turns)."""
    import torch
    reps = []
    for f in calls:
        f()
        torch.cuda.synchronize()
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        f()
        b.record()
        torch.cuda.synchronize()
        reps.append(max(3, min(100, int(budget_ms / max(a.elapsed_time(b), 1e-3)))))
    times = [[] for _ in calls]
    for _ in range(rounds):
        for f, n, t in zip(calls, reps, times):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(n):
                f()
            b.record()
            torch.cuda.synchronize()
            t.append(1000 * a.elapsed_time(b) / n)
    return [statistics.median(t) for t in times]


def fit_call(f2, n_bits, m, seed=1, max_n_bits=None):
    """A fit of contexts of widths n_bits and m rows of random bits each, ready to be called; (call, model)."""
    import torch
    n, m = np.asarray(n_bits, np.int64), np.asarray(m, np.int64)
    off = np.concatenate([[0], np.cumsum(m * ((n + 64) // 64 + 2))])
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    rows = torch.randint(-2 ** 63, 2 ** 63 - 1, (max(int(off[-1]), 1),), generator=g, device="cuda", dtype=torch.int64)
    model = f2.Model(n.astype(np.int32), max_n_bits=max_n_bits)
    nb = f2.f2_fit_workspace_bytes(model.num_ctx)
    ws, offd = f2.workspace(nb), torch.from_numpy(off).cuda()

    def call():
        assert f2.f2_fit_batch(rows, rows.numel(), offd, model, ws, nb) == f2.F2_OK
    return call, model


def encode_call(f2, model, ctx, x):
    """An encode of queries x [nq, stride] (device tensors) against a fitted model, ready to be called."""
    import torch
    nq, stride = x.shape
    words = torch.empty(nq, 2, dtype=torch.int64, device="cuda")
    qf = torch.empty(nq, dtype=torch.uint8, device="cuda")
    nb = f2.f2_encode_workspace_bytes(model, nq)
    ws = f2.workspace(nb)

    def call():
        assert f2.f2_encode_batch(model, ctx, x, stride, nq, words, qf, ws, nb) == f2.F2_OK
    return call
