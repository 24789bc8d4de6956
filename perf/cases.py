"""The calls that are timed: what a user of the learner has it do, through the package's entry points.

A user fits contexts (one, thousands, tens of thousands, or a few very wide ones), encodes query
batches against the fitted maps, groups an interleaved row stream before the fit, pools separately
fitted shards, builds fit rows from parsed values, and merges fields into encoded words.  Inputs,
output buffers, workspaces and (for the encodes) the fitted model are in hand before a call, as a
program that serves many calls keeps them; a pass is the library call or calls alone.

Training rows are odd-sized XORs of each context's own planted generators [x | 1 | y], so they are
consistent, span a planted subspace (0.7 of the width where the corpus statistics say so), and an
injected contradiction is a repeated row with one output bit flipped.  Queries are XORs of three
training feature vectors, a few with one bit flipped (mostly outside the span).
Every output is a bit string, a count or a flag, so results are compared exactly.
"""
import math

import numpy as np
import torch

from paper_2608_20532_amd import f2gpu

DEV = "cuda"


def listed():
    return [
        # one context learned and used at once, the smallest call: launches and latency
        {"name": "step_one", "kind": "step", "style": "uniform", "contexts": 1, "rows": 200, "queries": 1000, "stride": 1, "zipf": 0.0},
        # a target's mid-sized batch: widths 17-97, twice as many rows as columns
        {"name": "fit_4k", "kind": "fit", "style": "uniform", "contexts": 4096, "rows": 0},
        # a whole corpus: 80,000 contexts, mean width 41, log-normal row counts, 1% contradictory
        {"name": "fit_80k", "kind": "fit", "style": "corpus", "contexts": 80000, "rows": 0},
        # the widest contexts, full rank, twice as many rows as columns
        {"name": "fit_wide", "kind": "fit", "style": "dense", "contexts": 64, "width": 4095, "rows": 8192},
        # wide instruction forms as a corpus holds them: few distinct observations (rank far below the
        # width), learned and then used for a small batch of queries
        {"name": "step_sparse_wide", "kind": "step", "style": "sparse", "contexts": 96, "width": 1500, "rows": 0,
         "queries": 20000, "stride": 24, "zipf": 0.0},
        # re-encoding one binary: a million instructions over mid-sized maps, uniform contexts
        {"name": "encode_1m_uniform", "kind": "encode", "style": "uniform", "contexts": 4096, "rows": 0, "queries": 1000000, "stride": 2, "zipf": 0.0},
        # the same over a corpus of maps: the frequent contexts take most queries
        {"name": "encode_1m_corpus", "kind": "encode", "style": "corpus", "contexts": 80000, "rows": 0, "queries": 1000000, "stride": 4, "zipf": 1.1},
        # a corpus re-encoded in one batch, the largest call
        {"name": "encode_100m", "kind": "encode", "style": "corpus", "contexts": 80000, "rows": 0, "queries": 100000000, "stride": 4, "zipf": 1.1},
        # ingestion: the corpus's rows as they are gathered, mixed, grouped for the fit
        {"name": "group_7m", "kind": "group", "contexts": 80000, "rows": 7240070, "stride": 7},
        # shard models merged: three shards of each of 80,000 contexts
        {"name": "pool_80k", "kind": "pool", "pools": 80000, "shards": 3},
        # fit rows from five parsed values each
        {"name": "vectorize_7m", "kind": "vectorize", "rows": 7240070, "k": 5},
        # final words: a field XORed in, opaque bits restored
        {"name": "merge_100m", "kind": "merge", "words": 100000000, "shift": 105, "width": 17},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["fit", "fit", "wide", "encode", "encode", "encode", "step", "group", "pool", "vectorize", "merge"])
    style = rng.choice(["uniform", "corpus"])
    top = 4096 if style == "uniform" else 80000
    if kind == "fit":
        return {"kind": "fit", "style": style, "contexts": _log(rng, 1, top), "rows": 0}
    if kind == "wide":
        n = _log(rng, 512, 4095)
        return {"kind": "fit", "style": "dense", "contexts": _log(rng, 1, 64), "width": n, "rows": 2 * (n + 1) + rng.randrange(64)}
    if kind == "encode":
        return {"kind": "encode", "style": style, "contexts": _log(rng, 1, top), "rows": 0, "queries": _log(rng, 1000, 30000000),
                "stride": rng.randrange(2, 5) if style == "uniform" else rng.randrange(4, 6), "zipf": rng.choice([0.0, 1.1])}
    if kind == "step":
        if rng.random() < 0.5:
            return {"kind": "step", "style": style, "contexts": _log(rng, 1, top), "rows": 0, "queries": _log(rng, 500, 2000000),
                    "stride": 2 if style == "uniform" else 4, "zipf": 0.0}
        n = rng.randrange(600, 2000)
        return {"kind": "step", "style": "sparse", "contexts": _log(rng, 8, 128), "width": n, "rows": 0,
                "queries": _log(rng, 1000, 50000), "stride": (n + 63) // 64, "zipf": 0.0}
    if kind == "group":
        return {"kind": "group", "contexts": _log(rng, 1, 200000), "rows": _log(rng, 1000, 7000000), "stride": rng.randrange(3, 10)}
    if kind == "pool":
        return {"kind": "pool", "pools": _log(rng, 100, 80000), "shards": rng.randrange(2, 5)}
    if kind == "vectorize":
        return {"kind": "vectorize", "rows": _log(rng, 1000, 7000000), "k": rng.randrange(1, 9)}
    w = rng.randrange(1, 65)
    return {"kind": "merge", "words": _log(rng, 1000, 90000000), "shift": rng.randrange(0, 129 - w), "width": w}


# ---- inputs ----

def _shapes(style, C, rows, width, seed):
    """(n_bits, generators, rows) of each context: the case's own sizes, in an order of the seed's."""
    r = np.random.RandomState(20)
    if style == "uniform":  # one more input bit that is never set
        n = r.randint(16, 97, C) + 1
        g, m = n + 16, np.full(C, rows) if rows else 2 * n  # more generators than dimensions: they span them all
    elif style == "corpus":
        n = np.minimum(8 + r.geometric(1 / 33, C), 256)
        g, m = np.ceil(0.7 * n).astype(np.int64) + 1, np.clip(np.rint(np.exp(r.normal(math.log(30), 1.5, C))), 1, 4000)
    elif style == "dense":
        n = np.full(C, width)
        g, m = n + 64, np.full(C, rows)
    else:  # sparse: widths from just above 512, some tens of independent observations
        n = np.rint(np.exp(r.uniform(math.log(513), math.log(width), C)))
        g, m = np.clip(np.rint(np.exp(r.normal(math.log(24), 1.0, C))), 2, 400), np.clip(np.rint(np.exp(r.normal(math.log(120), 1.2, C))), 1, 4000)
    p = np.random.RandomState(seed % (1 << 32)).permutation(C)
    return n.astype(np.int64)[p], g.astype(np.int64)[p], m.astype(np.int64)[p]


def _case_shapes(case, seed):
    return _shapes(case["style"], case["contexts"], case["rows"], case.get("width", 0), seed)


def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return g


def _rand(g, *shape):
    return torch.randint(-2 ** 63, 2 ** 63 - 1, shape, generator=g, device=DEV, dtype=torch.int64)


def _dev(a, dtype=torch.int64):
    return torch.as_tensor(np.asarray(a)).to(DEV, dtype)


def _pick(g, lo, cnt):
    """A random entry of [lo, lo + cnt) for each element."""
    u = torch.rand(lo.shape, generator=g, device=DEV, dtype=torch.float64)
    return lo + torch.minimum((u * cnt).to(torch.int64), cnt - 1)


class _Rows:
    """Training rows: padded [R, F + 2] (features, then the output words), their contexts, and the packed buffer."""

    def __init__(self, style, n, gens, m, fam, seed):
        """Context c draws from the generators of family fam[c] (n and gens per context, equal within a family)."""
        g = _gen(seed)
        C = len(n)
        fams = int(fam.max()) + 1
        ng, nn = np.zeros(fams, np.int64), np.zeros(fams, np.int64)
        ng[fam], nn[fam] = gens, n
        F = int((n.max() + 64) // 64)
        goff = np.concatenate([[0], np.cumsum(ng)])
        gn = torch.repeat_interleave(_dev(nn), _dev(ng))
        w = torch.arange(F, device=DEV)
        bits = (gn[:, None] - (1 if style == "uniform" else 0) - 64 * w).clamp(0, 64)  # x bits below the width (or the unused one)
        mask = torch.where(bits >= 64, torch.full_like(bits, -1), (torch.ones_like(bits) << (bits & 63)) - 1)
        G = torch.cat([_rand(g, len(gn), F) & mask, _rand(g, len(gn), 2)], 1)
        G[torch.arange(len(gn), device=DEV), gn >> 6] |= torch.ones_like(gn) << (gn & 63)  # the constant
        ctx = torch.repeat_interleave(torch.arange(C, device=DEV), _dev(m))
        lo, cnt = _dev(goff[:-1][fam])[ctx], _dev(gens)[ctx]
        rows = G[_pick(g, lo, cnt)]
        for _ in range({"dense": 24, "uniform": 8}.get(style, 4)):
            rows ^= G[_pick(g, lo, cnt)]
        self.first = _dev(np.concatenate([[0], np.cumsum(m)]))
        self.m = _dev(m)
        if style in ("uniform", "corpus"):  # contradictions: a late row repeats an early one with an output bit flipped
            r = np.random.RandomState((seed + 1) % (1 << 32))
            hit = _dev(np.nonzero((r.rand(C) < (0.05 if style == "uniform" else 0.01)) & (m > 1))[0])
            src, dst = self.first[hit], self.first[hit + 1] - 1
            rows[dst] = rows[src]
            rows[dst, F] ^= 1 << 17
        self.n, self.F, self.C, self.rows, self.ctx = _dev(n), F, C, rows, ctx
        # packed: fw words, then the output words
        fw = (self.n[ctx] + 64) // 64
        keep = torch.cat([w < fw[:, None], torch.ones(len(ctx), 2, dtype=torch.bool, device=DEV)], 1)
        self.packed = rows[keep]
        W = (n + 64) // 64 + 2
        self.off_host = np.concatenate([[0], np.cumsum(m * W)])
        self.off = _dev(self.off_host)

    def queries(self, g, ctx, stride, out):
        """x words of one query per entry of ctx; a fraction out has one bit below the width flipped."""
        n, lo, cnt = self.n[ctx], self.first[ctx], self.m[ctx]
        x = self.rows[_pick(g, lo, cnt), :self.F]
        for _ in range(2):
            x ^= self.rows[_pick(g, lo, cnt), :self.F]
        i = torch.arange(len(ctx), device=DEV)
        x[i, n >> 6] ^= torch.ones_like(n) << (n & 63)  # the constant is not part of x
        bad = torch.nonzero(torch.rand(len(ctx), generator=g, device=DEV) < out)[:, 0]
        b = _pick(g, torch.zeros_like(bad), n[bad].clamp(min=1))
        x[bad, b >> 6] ^= torch.ones_like(b) << (b & 63)
        res = torch.zeros(len(ctx), stride, dtype=torch.int64, device=DEV)
        res[:, :min(stride, self.F)] = x[:, :stride]
        return res


def _fit_state(case, seed):
    n, gens, m = _case_shapes(case, seed)
    R = _Rows(case["style"], n, gens, m, np.arange(len(n)), seed)
    model = f2gpu.Model(n.astype(np.int32), device=DEV)
    nb = f2gpu.f2_fit_workspace_bytes(model.num_ctx)
    return R, {"case": case, "rows": R.packed, "off": R.off, "model": model, "ws": f2gpu.workspace(nb, DEV), "nb": nb}


def _call(status):
    if status != 0:
        raise RuntimeError(f2gpu.f2_status_string(status))


def _run_fit(s):
    _call(f2gpu.f2_fit_batch(s["rows"], s["rows"].numel(), s["off"], s["model"], s["ws"], s["nb"]))


def _add_queries(s, case, R, seed):
    g = _gen(seed + 7)
    Q, S, C = case["queries"], case["stride"], case["contexts"]
    if case["zipf"]:
        cdf = torch.cumsum(torch.arange(1, C + 1, device=DEV, dtype=torch.float64) ** -case["zipf"], 0)
        perm = torch.randperm(C, generator=g, device=DEV)
    s["ctx"] = torch.empty(Q, dtype=torch.int32, device=DEV)
    s["x"] = torch.empty(Q, S, dtype=torch.int64, device=DEV)
    for q0 in range(0, Q, 1 << 23):
        q = min(Q - q0, 1 << 23)
        u = torch.rand(q, generator=g, device=DEV, dtype=torch.float64)
        if case["zipf"]:
            ctx = perm[torch.searchsorted(cdf, u * cdf[-1]).clamp(max=C - 1)]
        else:
            ctx = (u * C).to(torch.int64).clamp(max=C - 1)
        s["ctx"][q0:q0 + q] = ctx
        s["x"][q0:q0 + q] = R.queries(g, ctx, S, 0.02)
    s["words"] = torch.zeros(Q, 2, dtype=torch.int64, device=DEV)
    s["qf"] = torch.zeros(Q, dtype=torch.uint8, device=DEV)
    s["enb"] = f2gpu.f2_encode_workspace_bytes(s["model"], Q)
    s["ews"] = f2gpu.workspace(s["enb"], DEV)


def _run_encode(s):
    c = s["case"]
    _call(f2gpu.f2_encode_batch(s["model"], s["ctx"], s["x"], c["stride"], c["queries"], s["words"], s["qf"], s["ews"], s["enb"]))
    return {"words": s["words"], "qflags": s["qf"]}


def _model_outputs(m, whole=True):
    out = {"pivots": m.pivots, "maps": m.maps, "rank": m.rank, "flags": m.ctx_flags, "contra": m.n_contra, "first": m.first_contra_row}
    if whole:
        out["basis"] = m.basis
    return out


def prepare(case, seed):
    kind = case["kind"]
    if kind in ("fit", "step", "encode"):
        R, s = _fit_state(case, seed)
        if kind != "fit":
            _add_queries(s, case, R, seed)
        if kind == "encode":
            _run_fit(s)
            del s["rows"], s["off"], s["ws"]
        return s
    g = _gen(seed)
    s = {"case": case}
    if kind == "group":
        C, R, S = case["contexts"], case["rows"], case["stride"]
        r = np.random.RandomState(seed % (1 << 32))
        n = np.minimum(8 + r.geometric(1 / 33, C), 64 * (S - 2) - 1).astype(np.int32)
        share = torch.cumsum(torch.exp(1.5 * torch.randn(C, generator=g, device=DEV, dtype=torch.float64)), 0)
        u = torch.rand(R, generator=g, device=DEV, dtype=torch.float64)
        ctx = torch.searchsorted(share, u * share[-1]).clamp(max=C - 1).to(torch.int32)
        ctx[torch.rand(R, generator=g, device=DEV) < 0.001] = -1  # observations of no known context
        nb = f2gpu.f2_group_workspace_bytes(C, R)
        s.update(ctx=ctx, rows=_rand(g, R, S), n=_dev(n, torch.int32), out=torch.zeros(R * S, dtype=torch.int64, device=DEV),
                 off=torch.zeros(C + 1, dtype=torch.int64, device=DEV), drop=torch.zeros(1, dtype=torch.int64, device=DEV),
                 nb=nb, ws=f2gpu.workspace(nb, DEV))
    elif kind == "pool":
        P, k = case["pools"], case["shards"]
        n, gens, m = (np.repeat(v, k) for v in _shapes("corpus", P, 0, 0, seed))
        m = np.maximum(m // k, 1)
        R = _Rows("shards", n, gens, m, np.repeat(np.arange(P), k), seed)
        members = f2gpu.fit(R.packed, R.off, n.astype(np.int32))
        pooled = f2gpu.Model(n[::k].astype(np.int32), device=DEV)
        nb = f2gpu.f2_pool_workspace_bytes(members, P)
        s.update(members=members, pooled=pooled, off=_dev(np.arange(P + 1) * k), ids=_dev(np.arange(P * k), torch.int32),
                 flags=torch.zeros(P, dtype=torch.int32, device=DEV), nb=nb, ws=f2gpu.workspace(nb, DEV))
    elif kind == "vectorize":
        R, k = case["rows"], case["k"]
        s.update(values=_rand(g, R, k), y=_rand(g, R, 2), keep=(-1 & (2 ** 64 - 1), ~(5 << 58) & (2 ** 64 - 1)),
                 out=torch.zeros(R, k + 3, dtype=torch.int64, device=DEV))
    else:
        Q = case["words"]
        s.update(words=_rand(g, Q, 2), field=_rand(g, Q), state=_rand(g, Q, 2), mask=(0, 5 << 58),
                 out=torch.zeros(Q, 2, dtype=torch.int64, device=DEV))
    return s


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "fit":
        _run_fit(s)
        # parity-check rows are a documented output too; a full-rank context has none (its area is scratch)
        out = _model_outputs(s["model"])
        if case["style"] != "dense":
            out["tables"] = s["model"].tables
        return out
    if kind == "step":
        _run_fit(s)
        enc = _run_encode(s)
        # a rank-deficient wide context leaves scratch past its basis rows: the queries' words show the basis there
        return {**_model_outputs(s["model"], case["style"] != "sparse"), **enc}
    if kind == "encode":
        return _run_encode(s)
    if kind == "group":
        _call(f2gpu.f2_group_rows(s["ctx"], s["rows"], case["stride"], case["rows"], s["n"], case["contexts"], s["out"],
                                  case["rows"] * case["stride"], s["off"], s["drop"], s["ws"], s["nb"]))
        return {"rows": s["out"], "off": s["off"], "dropped": s["drop"]}
    if kind == "pool":
        p = s["pooled"]
        _call(f2gpu.f2_pool_bases(s["members"], None, s["off"], s["ids"], s["ids"].numel(), p, s["flags"], s["ws"], s["nb"]))
        return {**_model_outputs(p), "tables": p.tables, "pool_flags": s["flags"]}
    if kind == "vectorize":
        _call(f2gpu.f2_vectorize_rows(s["values"], s["y"], case["rows"], case["k"], s["keep"], s["out"]))
        return s["out"]
    _call(f2gpu.f2_merge_words(s["words"], s["field"], case["shift"], case["width"], s["mask"], s["state"], case["words"], s["out"]))
    return s["out"]


# ---- what a pass cannot do without ----

def _fit_work(n, gens, m, offsets=True):
    """Rows, offsets and widths in; basis rows, pivots, maps and scalars out; 32-bit operations of the elimination."""
    W, r = (n + 64) // 64 + 2, np.minimum(np.minimum(gens, n + 1), m)
    b = 8 * (m * W).sum() + 12 * len(n) + (8 * r * W + 4 * r + 16 * (n + 1)).sum() + 20 * len(n)
    return float(b), float((2 * W * r * (r - 1)).sum())


def work(case):
    kind = case["kind"]
    if kind in ("fit", "step", "encode"):
        n, gens, m = _case_shapes(case, 1)
        b, f = _fit_work(n, gens, m) if kind != "encode" else (0.0, 0.0)
        if kind != "fit":
            Q = case["queries"]
            used = min(1.0, Q / len(n))
            b += Q * (4 + 8 * case["stride"] + 16 + 1) + used * 16.0 * float((n + 1).sum())
            f += Q * 4.0 * float(n.mean())
        return {"bytes": b, "flops": f}
    if kind == "group":
        # id, then a row's own words in and out (mean width 41: three words)
        S = case["stride"]
        W = float(np.mean((np.minimum(8 + np.random.RandomState(1).geometric(1 / 33, 4096), 64 * (S - 2) - 1) + 64) // 64 + 2))
        return {"bytes": case["rows"] * (4 + 16 * W) + 12 * case["contexts"], "flops": 0}
    if kind == "pool":
        n, gens, m = _shapes("corpus", case["pools"], 0, 0, 1)
        r = np.minimum(gens, np.maximum(m // case["shards"], 1)) * case["shards"]
        b, f = _fit_work(n, gens, r)
        return {"bytes": b, "flops": f}
    if kind == "vectorize":
        return {"bytes": case["rows"] * (8 * case["k"] + 16 + 8 * (case["k"] + 3)), "flops": 0}
    return {"bytes": case["words"] * (16 + 8 + 16 + 16), "flops": 0}


def tolerance(case):
    return "exact"


# ---- the same results from plain torch and Python integers ----

def _eliminate(rows, n, fw):
    """Streaming elimination of one context's rows (Python integers): basis {pivot: (features, word)}, contradictions."""
    order = list(range(n - 1, -1, -1)) + [n]  # x bits from the top, the constant last
    basis, contra, first = {}, 0, -1
    for i, (f, y) in enumerate(rows):
        for p, (bf, by) in basis.items():
            if f >> p & 1:
                f, y = f ^ bf, y ^ by
        if not f:
            if y:
                contra, first = contra + 1, i if first < 0 else first
            continue
        p = next(b for b in order if f >> b & 1)
        for k, (bf, by) in basis.items():
            if bf >> p & 1:
                basis[k] = (bf ^ f, by ^ y)
        basis[p] = (f, y)
    return [(p, *basis[p]) for p in order if p in basis], contra, first


def _words(v, k):
    return [((v >> (64 * i)) & (2 ** 64 - 1)) - ((v >> (64 * i + 63) & 1) << 64) for i in range(k)]


def _exact_fit(case, s):
    model = s["model"]
    rows, off = s["rows"].cpu().numpy().astype(np.uint64), s["off"].cpu().numpy()
    out = {k: torch.zeros_like(v, device="cpu") for k, v in _model_outputs(model).items()}
    for c, n in enumerate(int(v) for v in model.n_bits_host):
        fw = (n + 64) // 64
        seg = rows[off[c]:off[c + 1]].reshape(-1, fw + 2)
        val = [(sum(int(w) << (64 * i) for i, w in enumerate(r[:fw])), int(r[fw]) | int(r[fw + 1]) << 64) for r in seg]
        basis, contra, first = _eliminate(val, n, fw)
        for k, (p, f, y) in enumerate(basis):
            out["pivots"][model.piv_off_host[c] + k] = p
            b = int(model.basis_off_host[c]) + k * (fw + 2)
            out["basis"][b:b + fw + 2] = torch.tensor(_words(f, fw) + _words(y, 2))
            q = int(model.map_off_host[c]) + 2 * p
            out["maps"][q:q + 2] = torch.tensor(_words(y, 2))
        out["rank"][c], out["contra"][c], out["first"][c], out["flags"][c] = len(basis), contra, first, int(contra > 0)
    return out


def exact(case, seed):
    kind = case["kind"]
    if kind == "group":
        s = prepare(case, seed)
        ctx = torch.where(s["ctx"] < 0, case["contexts"], s["ctx"]).to(torch.int64)
        order = torch.sort(ctx, stable=True)[1]
        order = order[ctx[order] < case["contexts"]]
        W = ((s["n"].to(torch.int64) + 64) // 64 + 2)
        rows = s["rows"][order][torch.arange(case["stride"], device=DEV) < W[ctx[order]][:, None]]
        s["out"][:rows.numel()] = rows
        s["off"][1:] = torch.cumsum(torch.bincount(ctx, minlength=case["contexts"] + 1)[:-1] * W, 0)
        return {"rows": s["out"], "off": s["off"], "dropped": (ctx == case["contexts"]).sum().reshape(1)}
    if kind == "vectorize":
        s = prepare(case, seed)
        keep = torch.tensor([v - (v >> 63 << 64) for v in s["keep"]], device=DEV)
        return torch.cat([s["values"], torch.ones_like(s["y"][:, :1]), s["y"] & keep], 1)
    if kind == "merge":
        s = prepare(case, seed)
        w, a = case["width"], case["shift"]
        f = s["field"] if w == 64 else s["field"] & ((1 << w) - 1)
        lo = f << a if a < 64 else torch.zeros_like(f)
        hi = f << (a - 64) if a >= 64 else ((f >> 1) & (2 ** 63 - 1)) >> (63 - a)
        mask = torch.tensor([v - (v >> 63 << 64) for v in s["mask"]], device=DEV)
        return ((s["words"] ^ torch.stack([lo, hi], 1)) & ~mask) | (s["state"] & mask)
    if kind in ("fit", "step") and case["style"] in ("uniform", "corpus") and case["contexts"] <= 200:
        rest = ("tables",) if kind == "fit" else ("words", "qflags")
        return {**_exact_fit(case, _fit_state(case, seed)[1]), **dict.fromkeys(rest)}
    return None  # an elimination or encode in plain Python of these sizes takes far over 20 seconds
