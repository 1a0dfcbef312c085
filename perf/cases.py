"""The work that programs have this framework do, as measurable cases.

Every case is one call (or, for the stream, one round of requests) through the
public entry points of ``paper_1812_09141_amd.ssj`` on synthetic collections of
the three shapes that the repository's configurations stand for:

  * short: sets of about 12 tokens (lognormal, sigma 0.5, 2 to 200), Zipf(1.0);
  * long:  sets of about 130 tokens (lognormal, sigma 0.8, 10 to 2,000),
    Zipf(0.9) over 1,000,000 tokens;
  * heavy: Pareto(1.5) sizes from 3 to 5,000, Zipf(1.2) over 2,000,000 tokens.

Token ids ascend with document frequency, sets ascend by size (ties by their
first tokens).  A share ``dup`` of the sets are near-copies of other sets, as
collections that are joined in earnest hold them; random sets alone are hardly
ever similar.  Candidates come from the CPU prefix and length filter, as in the
repository's serving path.

The library returns similar pairs in no particular order, so a program that
compares or merges results orders them; ``run`` does that too where a case asks
for the pairs and not for their number (the library's output-count mode, which
is what the paper measured).  All outputs are
whole numbers, so there is nothing that a 64-bit computation would sharpen.
"""
import math

import numpy as np
import torch

from paper_1812_09141_amd import ssj
from ssj_inputs import filter as cfilter

DEV = "cuda:0"

# kind: (size law, Zipf exponent, token universe)
KINDS = {
    "short": (("lognormal", 12.0, 0.5, 2, 200), 1.0, 200_000),
    "long": (("lognormal", 130.0, 0.8, 10, 2_000), 0.9, 1_000_000),
    "heavy": (("pareto", 1.5, 3, 5_000), 1.2, 2_000_000),
}
MEAN = {"short": 12.0, "long": 130.0, "heavy": 8.4}
# prefix-filter candidates per pair of sets, by kind and threshold (measured)
DENSITY = {
    ("short", "3/5"): 3.1e-4, ("short", "7/10"): 6.2e-5, ("short", "4/5"): 1.1e-5, ("short", "9/10"): 1.0e-6,
    ("long", "7/10"): 2.5e-4, ("long", "4/5"): 3.0e-5,
    ("heavy", "3/4"): 6.8e-4, ("heavy", "4/5"): 4.2e-4,
}
# The plans that programs keep: what a new context has, and the three that the
# autotuner chose for the shapes (one thread per pair through the window ring;
# the same on a wider grid without the ring; long sets with a step budget).
PLANS = {
    "default": None,
    "ring": dict(inline_lanes=1, defer_from=5, staged=1),
    "wide": dict(inline_lanes=1, defer_from=5, wg_per_cu=12),
    "budget": dict(inline_lanes=1, defer_from=4, lanes=(4, 8, 16, 32, 64), spill_iters=32, spill_lanes=16,
                   wg_per_cu=6, staged=1),
}


def listed():
    base = dict(sim="jaccard", plan="default", positional=False, count=False, batches=0)
    return [
        # a lookup from an interactive program: some hundred candidates, how
        # many of them are similar
        dict(base, name="verify small", path="device", kind="short", sets=2_000, dup=0.1, t="4/5", cap=0, count=True),
        # candidates of a CPU filter in host memory, one synchronous call
        dict(base, name="verify host buffers", path="host", kind="short", sets=100_000, dup=0.02, t="7/10", cap=16384),
        # an offline sweep: four thresholds' candidates in one launch
        dict(base, name="verify four thresholds", path="batch", kind="short", sets=100_000, dup=0.005,
             t="3/5,7/10,4/5,9/10", cap=2048, plan="ring"),
        # a join of two collections that share many near-duplicates, by Cosine
        dict(base, name="verify two collections", path="rs", kind="short", sets=150_000, dup=0.3, t="3/5",
             cap=131072, sim="cosine"),
        # long sets: merges of many steps, a few very long ones among them
        dict(base, name="verify long sets", path="device", kind="long", sets=50_000, dup=0.02, t="7/10", cap=2048,
             plan="budget"),
        # the largest: Zipf-like sizes, 1.7e8 candidates, the count alone
        dict(base, name="verify heavy tail", path="device", kind="heavy", sets=500_000, dup=0.0, t="3/4", cap=0,
             count=True, plan="wide"),
        # the sweep's counts, with candidates grouped by probe set
        dict(base, name="verify grouped", path="groups", kind="short", sets=100_000, dup=0.005,
             t="3/5,7/10,4/5,9/10", cap=0, count=True, plan="ring"),
        # whole joins on the device: candidates and verification
        dict(base, name="join small", path="join_host", kind="short", sets=5_000, dup=0.1, t="7/10", cap=4096,
             positional=True),
        dict(base, name="join short sets", path="join", kind="short", sets=100_000, dup=0.02, t="3/5", cap=16384,
             positional=True),
        dict(base, name="join long sets", path="join", kind="long", sets=50_000, dup=0.02, t="7/10", cap=2048,
             positional=True),
        dict(base, name="join heavy tail", path="join", kind="heavy", sets=500_000, dup=0.0, t="3/4", cap=0,
             count=True),
        # serving: requests of very different sizes in flight together
        dict(base, name="stream of batches", path="stream", kind="short", sets=100_000, dup=0.02, t="3/5,4/5,9/10",
             cap=65536, batches=24),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: any path with any plan, sizes over the whole range."""
    path = rng.choice(["device", "host", "batch", "rs", "groups", "join", "join", "join_host", "candidates", "stream"])
    kind = rng.choice(["short", "short", "long", "heavy"])
    if path in ("batch", "groups", "stream"):
        kind = "short"
    most = {"short": 120_000, "long": 50_000, "heavy": 300_000}[kind]
    sets = _log_uniform(rng, {"short": 1_500, "long": 1_000, "heavy": 5_000}[kind], most)
    dup = rng.choice([0.02, 0.1, 0.3])
    if kind == "heavy":
        dup = 0.0  # its many sets of three common tokens are duplicates already
    c = dict(path=path, kind=kind, sets=sets, dup=dup, sim="jaccard", plan="default", positional=False,
             count=kind == "heavy", batches=0)
    if path in ("device", "batch", "rs", "groups", "join") and rng.random() < 0.5:
        c["count"] = True
    if path == "batch" or path == "groups":
        c["t"] = rng.choice(["3/5,7/10,4/5,9/10", "7/10,4/5", "3/5,9/10"])
    elif path == "stream":
        c["t"] = "3/5,4/5,9/10"
        c["batches"] = rng.randint(4, 24)
    else:
        c["t"] = rng.choice({"short": ["3/5", "7/10", "4/5", "9/10"], "long": ["7/10", "4/5"],
                             "heavy": ["3/4", "4/5"]}[kind])
    if path in ("join", "join_host", "candidates"):
        c["positional"] = rng.random() < 0.5
    else:
        c["plan"] = rng.choice(["default", "ring", "wide", "budget"])
    if path in ("device", "rs", "host") and kind != "heavy":
        c["sim"] = rng.choice(["jaccard", "cosine", "dice"] + (["overlap"] if kind == "short" else []))
    if path in ("host", "join_host") and kind == "heavy":
        c["path"] = "device" if path == "host" else "join"
    if path == "candidates":
        c["count"] = False
        if kind == "heavy":
            c["sets"] = min(c["sets"], 50_000)
        c["cap"] = 1 << max(10, math.ceil(math.log2(4 * _pairs(c, c["t"]) + 64)))
    elif c["count"]:
        c["cap"] = 0
    else:
        c["cap"] = 1 << max(10, math.ceil(math.log2(4 * (0.02 + dup) * sets * len(c["t"].split(",")))))
    return c


# ---------------------------------------------------------------------------
# Inputs, made on the GPU from the seed alone.

def _ratio(t):
    a, b = t.split("/")
    return int(a), int(b)


def _sizes(law, n, g):
    if law[0] == "lognormal":
        _, mean, sigma, lo, hi = law
        mu = math.log(mean) - sigma * sigma / 2.0
        x = torch.exp(mu + sigma * torch.randn(n, generator=g, device=DEV, dtype=torch.float64))
        return x.round().clamp(lo, hi).long()
    _, alpha, xm, hi = law
    u = 1.0 - torch.rand(n, generator=g, device=DEV, dtype=torch.float64)
    return (xm * u ** (-1.0 / alpha)).floor().clamp(xm, hi).long()


def _zipf(cdf, n, g):
    u = torch.rand(n, generator=g, device=DEV, dtype=torch.float64)
    return torch.searchsorted(cdf, u).clamp(max=cdf.numel() - 1)


def _within(start_of, idx):
    return torch.arange(idx.numel(), device=DEV) - start_of[idx]


def _starts(counts):
    s = torch.zeros(counts.numel() + 1, dtype=torch.int64, device=DEV)
    torch.cumsum(counts, 0, out=s[1:])
    return s


def collection(kind, n_sets, dup, seed):
    """CSR collection (offsets int64, tokens int32, host arrays)."""
    law, zipf_s, universe = KINDS[kind]
    g = torch.Generator(device=DEV)
    g.manual_seed(1_000_003 * seed + 17)
    cdf = torch.cumsum(torch.arange(1, universe + 1, device=DEV, dtype=torch.float64) ** (-zipf_s), 0)
    cdf /= cdf[-1].clone()
    n_base = max(1, round(n_sets * (1.0 - dup)))
    sizes = _sizes(law, n_base, g)
    # twice as many draws as wanted; a set keeps its first distinct ones
    m = 2 * sizes + 4
    idx = torch.repeat_interleave(torch.arange(n_base, device=DEV), m)
    tok = _zipf(cdf, idx.numel(), g)
    key, order = torch.sort((idx << 22) | tok, stable=True)
    first = torch.ones_like(key, dtype=torch.bool)
    first[1:] = key[1:] != key[:-1]
    keep = torch.sort(order[first]).values  # draw order
    idx, tok = idx[keep], tok[keep]
    st = _starts(torch.bincount(idx, minlength=n_base))
    keep = _within(st, idx) < sizes[idx]
    idx, tok = idx[keep], tok[keep]
    n_copy = n_sets - n_base
    if n_copy > 0:
        # near-copies: one token in ten replaced by a fresh draw
        src = torch.randint(0, n_base, (n_copy,), generator=g, device=DEV)
        cnt = torch.bincount(idx, minlength=n_base)
        st = _starts(cnt)
        ci = torch.repeat_interleave(torch.arange(n_copy, device=DEV), cnt[src])
        pos = _within(_starts(cnt[src]), ci)
        ct = tok[st[src][ci] + pos]
        fresh = torch.rand(ct.numel(), generator=g, device=DEV) < 0.1
        ct = torch.where(fresh, _zipf(cdf, ct.numel(), g), ct)
        key = torch.unique(torch.cat([(idx << 22) | tok, ((ci + n_base) << 22) | ct]))
        idx, tok = key >> 22, key & ((1 << 22) - 1)
    # token ids by ascending document frequency, tokens ascending in a set
    df = torch.bincount(tok, minlength=universe)
    occ = torch.nonzero(df).squeeze(1)
    new_id = torch.zeros(universe, dtype=torch.int64, device=DEV)
    new_id[occ[torch.sort(df[occ], stable=True).indices]] = torch.arange(occ.numel(), device=DEV)
    key = torch.sort((idx << 22) | new_id[tok]).values
    idx, tok = key >> 22, key & ((1 << 22) - 1)
    cnt = torch.bincount(idx, minlength=n_sets)
    st = _starts(cnt)
    # sets by size, then by their first two tokens
    t0 = tok[st[:-1]]
    t1 = tok[(st[:-1] + 1).clamp(max=tok.numel() - 1)]
    perm = torch.sort(t1, stable=True).indices
    perm = perm[torch.sort(t0[perm], stable=True).indices]
    perm = perm[torch.sort(cnt[perm], stable=True).indices]
    off = _starts(cnt[perm])
    j = torch.repeat_interleave(torch.arange(n_sets, device=DEV), cnt[perm])
    tokens = tok[st[perm][j] + _within(off, j)].int()
    return off.cpu().numpy(), tokens.cpu().numpy()


_contexts = {}


def _context(plan):
    """A program's context with its plan, kept for its life."""
    if plan not in _contexts:
        ctx = ssj.ssj_init(0, hbm_budget=16 << 30)
        if PLANS[plan] is not None:
            ssj.ssj_set_plan(ctx, ssj.make_plan(**PLANS[plan]))
        _contexts[plan] = ctx
    return _contexts[plan]


class Collection:
    """An uploaded collection, freed with its last user."""

    def __init__(self, ctx, off, tok):
        self.ctx, self.h = ctx, ssj.ssj_upload_collection(ctx, off, tok)

    def __del__(self, free=ssj.ssj_free_collection):
        free(self.ctx, self.h)


def _sim_threshold(case, t):
    """The threshold of the similarity function for a list filtered at t."""
    if case["sim"] == "overlap":
        return 8, 1
    return _ratio(t)


def _subset(off, tok, ids):
    cnt = np.diff(off)[ids]
    o = np.zeros(ids.shape[0] + 1, dtype=np.int64)
    np.cumsum(cnt, out=o[1:])
    at = np.repeat(off[:-1][ids] - o[:-1], cnt) + np.arange(o[-1])
    return o, tok[at]


def prepare(case, seed):
    ctx = _context(case["plan"])
    off, tok = collection(case["kind"], case["sets"], case["dup"], seed)
    s = {"case": case, "ctx": ctx}
    path, ts = case["path"], case["t"].split(",")
    thr = [_sim_threshold(case, t) for t in ts]
    s["thr"] = thr
    if path == "rs":
        even, odd = np.arange(0, case["sets"], 2), np.arange(1, case["sets"], 2)
        s["coll"], s["coll_s"] = Collection(ctx, *_subset(off, tok, even)), Collection(ctx, *_subset(off, tok, odd))
    else:
        s["coll"] = Collection(ctx, off, tok)
    cands = []
    if path not in ("join", "join_host", "candidates"):
        cands = [cfilter.candidates(off, tok, *_ratio(t)) for t in ts]
    if path == "rs":
        c = cands[0]
        a, b = c[c[:, 0] % 2 > c[:, 1] % 2][:, ::-1], c[c[:, 0] % 2 < c[:, 1] % 2]
        cands = [np.concatenate([a, b]) // 2]
    if path == "host":
        s["cands"] = [np.ascontiguousarray(cands[0])]
    elif path == "stream":
        # requests: whole stretches of a threshold's candidates, their sizes
        # from 1,000 to 1,000,000 pairs
        r = np.random.default_rng(seed)
        s["reqs"] = []
        for k in range(case["batches"]):
            c, t = cands[k % len(ts)], thr[k % len(ts)]
            n = min(int(math.exp(r.uniform(math.log(1e3), math.log(1e6)))), c.shape[0])
            at = int(r.integers(0, c.shape[0] - n + 1))
            s["reqs"].append((np.ascontiguousarray(c[at:at + n]), *t))
    elif path == "groups":
        s["cands"] = [tuple(torch.from_numpy(x).to(DEV) for x in ssj.groups_of(c)) for c in cands]
    else:
        s["cands"] = [torch.from_numpy(np.ascontiguousarray(c)).to(DEV) for c in cands]
    if path in ("device", "batch", "rs", "groups", "join", "candidates"):
        cap = case["cap"]
        s["count"] = torch.zeros(len(ts), dtype=torch.int64, device=DEV)
        s["out"] = torch.full((len(ts), cap, 2), -1, dtype=torch.int32, device=DEV) if cap else None
        outs = [s["out"][i] if cap else None for i in range(len(ts))]
        cnts = [s["count"][i:i + 1] for i in range(len(ts))]
        if path == "batch":
            s["reqs"] = [(c, *t, o, n, case["sim"]) for c, t, o, n in zip(s["cands"], thr, outs, cnts)]
        elif path == "groups":
            s["reqs"] = [(gr, si, *t, o, n, case["sim"]) for (gr, si), t, o, n in zip(s["cands"], thr, outs, cnts)]
    return s


def _ordered(pairs, cap):
    """Host pairs in order, in an array of the capacity."""
    out = np.full(cap, -1, dtype=np.int64)
    k = min(cap, pairs.shape[0])
    out[:k] = np.sort(np.ascontiguousarray(pairs).view(np.int64).ravel())[:k]
    return out


def run(s):
    case, ctx = s["case"], s["ctx"]
    path, h = case["path"], s["coll"].h
    if path == "host":
        tn, td = s["thr"][0]
        res = ssj.ssj_verify_sim(ctx, h, s["cands"][0], case["sim"], tn, td)
        return {"count": res.shape[0], "pairs": _ordered(res, case["cap"])}
    if path == "join_host":
        tn, td = s["thr"][0]
        res = ssj.ssj_join(ctx, h, tn, td, case["positional"])
        return {"count": res.shape[0], "pairs": _ordered(res, case["cap"])}
    if path == "stream":
        tickets = [ssj.ssj_stream_submit(ctx, h, c, tn, td) for c, tn, td in s["reqs"]]
        res = [ssj.ssj_stream_collect(ctx, t) for t in tickets]
        return {"counts": np.array([r.shape[0] for r in res]), "pairs": _ordered(np.concatenate(res), case["cap"])}
    out = s["out"][0] if s["out"] is not None else None
    tn, td = s["thr"][0]
    if path == "device":
        ssj.ssj_verify_device_sim(ctx, h, s["cands"][0], case["sim"], tn, td, out, s["count"])
    elif path == "rs":
        ssj.ssj_verify_rs_device(ctx, h, s["coll_s"].h, s["cands"][0], case["sim"], tn, td, out, s["count"])
    elif path == "batch":
        ssj.ssj_verify_batch_device(ctx, h, s["reqs"])
    elif path == "groups":
        ssj.ssj_verify_groups_batch_device(ctx, h, h, s["reqs"])
    elif path == "join":
        ssj.ssj_join_device(ctx, h, tn, td, case["positional"], out, s["count"])
    else:  # candidates, which come in order
        ssj.ssj_candidates_device(ctx, h, tn, td, case["positional"], out, s["count"])
        return {"count": s["count"], "pairs": s["out"]}
    if out is None:
        return {"count": s["count"]}
    # each request's pairs in order (unused room holds -1 and comes first)
    return {"count": s["count"], "pairs": torch.sort(s["out"].view(torch.int64), dim=1).values}


def _pairs(case, t):
    """Candidates that the prefix filter leaves at t, about."""
    return DENSITY[(case["kind"], t)] * case["sets"] ** 2 + 2.0 * case["dup"] * case["sets"]


def work(case):
    """Bytes of one pass: the tokens and set bounds once, the candidates where
    they are given, the results; a pair's decision is a handful of integer
    operations per token and no matrix work."""
    sets = case["sets"]
    b = 4.0 * MEAN[case["kind"]] * sets + 8.0 * sets
    pairs = sum(_pairs(case, t) for t in case["t"].split(","))
    if case["path"] == "stream":
        # 24 requests of about 145,000 pairs, fewer where a list is shorter
        pairs = sum(min(145e3, _pairs(case, t)) for t in case["t"].split(",")) * case["batches"] / 3.0
    if case["path"] == "rs":
        pairs /= 2.0
    if case["path"] == "candidates":
        b += 8.0 * pairs
    elif case["path"] not in ("join", "join_host"):
        b += (4.0 if case["path"] == "groups" else 8.0) * pairs
    if not case["count"]:
        b += 8.0 * case["dup"] * sets
    return {"bytes": b, "flops": 0.0}
