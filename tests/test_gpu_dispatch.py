"""Launches at the edges of the rules that pick their kernels and at the ends of
their workgroups: the longest pair just inside and just outside a deferred
class, step budgets at the longest merge, and batches that mix requests with
and without an output buffer, with more chunks than wavefronts of a workgroup;
against the oracle (whole numbers: no tolerance)."""
import os
import sys

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)

import oracle  # noqa: E402
from ssj_inputs import synth  # noqa: E402


@pytest.fixture(scope="module")
def S():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1812_09141_amd.ssj as ssj
    ssj.load_library()
    return ssj


@pytest.fixture(scope="module")
def ctx(S):
    c = S.ssj_init(0)
    yield c
    S.ssj_shutdown(c)


def _pairs(n, k, seed):
    return np.random.default_rng(seed).integers(0, n, (k, 2)).astype(np.int32)


@pytest.mark.parametrize("longest", [16, 17, 64, 65, 256, 257])
def test_longest_pair_at_a_class_bound(S, ctx, longest):
    # pairs of the two longest sets have 2 longest - 1 and 2 longest tokens:
    # 32 | 33, 128 | 129, 512 | 513 lie on either side of a bound
    rng = np.random.default_rng(700 + longest)
    base = np.sort(rng.choice(4 * longest, longest, replace=False))
    sets = [np.sort(rng.choice(base, size=int(rng.integers(max(1, longest // 2), longest)), replace=False)).tolist()
            for _ in range(150)]
    sets += [base.tolist(), base[1:].tolist(), base.tolist()]
    c = synth.collection_from_sets(sorted(sets, key=len))
    cand = _pairs(c.n_sets, 5000, 1)
    cand[:3] = [[c.n_sets - 1, c.n_sets - 2], [c.n_sets - 1, c.n_sets - 3], [c.n_sets - 3, c.n_sets - 2]]
    steps = 2 * ((longest + 3) // 4)  # window steps that no merge outruns
    h = S.ssj_upload_collection(ctx, c.offsets, c.tokens)
    try:
        for tn, td in [(1, 2), (9, 10)]:
            want = oracle.sort_pairs(oracle.select(c.offsets, c.tokens, cand, tn, td))
            for kw in [dict(defer_from=d, lanes=(4, 8, 16, 64, 256)) for d in range(6)] + \
                      [dict(defer_from=5, spill_iters=s, staged=g) for s in (steps - 1, steps) for g in (0, 1)]:
                print(f"longest {longest} t={tn}/{td} {kw}", flush=True)
                S.ssj_set_plan(ctx, S.make_plan(**kw))
                assert np.array_equal(oracle.sort_pairs(S.ssj_verify(ctx, h, cand, tn, td)), want)
    finally:
        S.ssj_free_collection(ctx, h)


@pytest.mark.parametrize("staged", [0, 1])
def test_batch_of_counts_and_pairs(S, ctx, staged):
    import torch
    c = synth.near_duplicate_collection(np.random.default_rng(5), n_base=80, copies=4, max_size=30, universe=300)
    S.ssj_set_plan(ctx, S.make_plan(defer_from=5, staged=staged, wg_per_cu=1))
    h = S.ssj_upload_collection(ctx, c.offsets, c.tokens)
    try:
        sizes = [1, 63, 64, 65, 0, 300, 5000, 200_000, 64, 1, 70_000]
        d_cnt = torch.full((len(sizes),), -7, dtype=torch.int64, device="cuda:0")
        reqs, want, outs = [], [], []
        for i, n in enumerate(sizes):
            cand = _pairs(c.n_sets, n, 40 + i)
            tn, td = [(1, 10), (1, 2), (0, 1)][i % 3]  # at 0 every pair passes: more than are staged
            want.append(oracle.sort_pairs(oracle.select(c.offsets, c.tokens, cand, tn, td)))
            out = None if i % 2 else torch.full((max(n, 1), 2), -1, dtype=torch.int32, device="cuda:0")
            outs.append(out)
            reqs.append((torch.from_numpy(cand).to("cuda:0"), tn, td, out, d_cnt[i:i + 1]))
        for _ in range(3):  # the counters return to zero after each launch
            d_cnt.fill_(-7)
            S.ssj_verify_batch_device(ctx, h, reqs)
            torch.cuda.synchronize()
            for i, w in enumerate(want):
                assert int(d_cnt[i].item()) == w.shape[0], i
                if outs[i] is not None:
                    assert np.array_equal(oracle.sort_pairs(outs[i][:w.shape[0]].cpu().numpy()), w), i
    finally:
        S.ssj_free_collection(ctx, h)


@pytest.mark.parametrize("longest", [400, 65535, 65536])
def test_cosine_at_the_threshold(S, ctx, longest):
    """Prefixes of one set: of n and o <= n tokens the similarity is sqrt(o / n),
    so o = n (t_num / t_den)^2 sits exactly at a threshold.  Sizes and threshold
    terms (in lowest terms) on both sides of what 64-bit arithmetic takes."""
    sims = [(3, 5), (60000, 100000), (1, 1), (181, 362), (32766, 32767), (32767, 32768), (32768, 32769),
            (19, 20), ((1 << 31) - 2, (1 << 31) - 1)]
    rng = np.random.default_rng(8)
    lens = {1, 2, 3, longest - 1, longest}
    for tn, td in sims:
        for n in {longest, longest - 1, 25 * (longest // 25), 4, int(rng.integers(10, longest))}:
            o = n * tn * tn // (td * td)
            lens |= {x for x in (n, o - 1, o, o + 1) if 1 <= x <= longest}
    lens = sorted(lens)
    c = synth.collection_from_sets([list(range(x)) for x in lens])
    r, s = np.tril_indices(c.n_sets, 0)
    cand = np.stack([r, s], axis=1).astype(np.int32)
    a, b = c.sizes()[r].astype(object), c.sizes()[s].astype(object)
    h = S.ssj_upload_collection(ctx, c.offsets, c.tokens)
    try:
        S.ssj_set_plan(ctx, S.make_plan(defer_from=3, lanes=(4, 8, 16, 64, 256)))
        for tn, td in sims:
            # the overlap of two prefixes is the shorter one: o^2 td^2 >= tn^2 n o
            keep = np.array([(y * td) ** 2 >= tn * tn * x * y for x, y in zip(a, b)], dtype=bool)
            print(f"cosine {tn}/{td}, {longest}: {int(keep.sum())} of {cand.shape[0]}", flush=True)
            got = oracle.sort_pairs(S.ssj_verify_sim(ctx, h, cand, "cosine", tn, td))
            assert np.array_equal(got, oracle.sort_pairs(cand[keep])), (tn, td)
    finally:
        S.ssj_free_collection(ctx, h)


@pytest.mark.parametrize("lanes", [4, 8, 16, 32, 64, 256])
def test_tiles_of_four_tokens_per_lane(S, ctx, lanes):
    """Set sizes around the tiles of the deferred kernel, overlaps counted exactly
    (Overlap thresholds at and above each pair's own), merged from the start and
    resumed after a step budget."""
    tile = 4 * min(lanes, 64)
    rng = np.random.default_rng(900 + lanes)
    universe = 6 * tile
    sets = []
    for n in (1, lanes, tile - 1, tile, tile + 1, 2 * tile - 1, 2 * tile, 2 * tile + 1, 3 * tile):
        n = min(n, universe)
        sets += [np.sort(rng.choice(universe, n, replace=False)).tolist() for _ in range(2)]
        sets.append(list(range(n)))                         # matches on every seam
        sets.append(list(range(universe - n, universe)))    # tails
    sets.append([0, (1 << 31) - 1])                         # the largest token
    sets.append([(1 << 31) - 1])
    c = synth.collection_from_sets(sorted(sets, key=len))
    r, s = np.tril_indices(c.n_sets, 0)
    cand = np.stack([r, s], axis=1).astype(np.int32)
    h = S.ssj_upload_collection(ctx, c.offsets, c.tokens)
    try:
        for plan in [dict(defer_from=0, lanes=(lanes,) * 5), dict(defer_from=5, spill_iters=1, spill_lanes=lanes)]:
            S.ssj_set_plan(ctx, S.make_plan(**plan))
            for k in (0, 1, 2, lanes, tile - 1, tile, tile + 1, 2 * tile, 3 * tile):
                want = oracle.sort_pairs(oracle.select(c.offsets, c.tokens, cand, k, 1, sim="overlap"))
                print(f"lanes {lanes} overlap {k}: {want.shape[0]}", flush=True)
                got = oracle.sort_pairs(S.ssj_verify_sim(ctx, h, cand, "overlap", k, 1))
                assert np.array_equal(got, want), (plan, k)
            for tn, td in [(1, 3), (4, 5)]:
                want = oracle.sort_pairs(oracle.select(c.offsets, c.tokens, cand, tn, td))
                assert np.array_equal(oracle.sort_pairs(S.ssj_verify(ctx, h, cand, tn, td)), want), (plan, tn, td)
    finally:
        S.ssj_free_collection(ctx, h)


def _similar_at(n, most, seed, step):
    """Sets of n tokens in pairs that share exactly k of them, k = 0, step, ..., n."""
    rng = np.random.default_rng(seed)
    sets = []
    for k in list(range(0, n, step)) + [n]:
        t = rng.choice(most, 2 * n - k, replace=False)
        sets += [np.sort(t[:n]).tolist(), np.sort(t[n - k:]).tolist()]
    return sets


@pytest.mark.parametrize("n, most", [(1, 2**31 - 1), (3, 60), (12, 2**31 - 1), (40, 10**6), (41, 2**31 - 1),
                                     (130, 10**6), (600, 5000)])
def test_signatures_keep_every_similar_pair(S, ctx, n, most):
    """Pairs of every overlap at the sizes where signatures are sparse, full and
    change their width, all pairs of the collection as candidates, under each
    rule and on both sides of the thresholds that long sets have them for."""
    sets = _similar_at(n, most, n, max(1, n // 25))
    c = synth.collection_from_sets(sorted(sets, key=len))
    r, s = np.tril_indices(c.n_sets, 0)
    cand = np.stack([r, s], axis=1).astype(np.int32)
    cand = np.tile(cand, (1 + 33_000 // cand.shape[0], 1))  # more chunks than launches without signatures have
    h = S.ssj_upload_collection(ctx, c.offsets, c.tokens)
    try:
        for plan in [{}, dict(inline_lanes=1, defer_from=5), dict(defer_from=5, spill_iters=2), dict(defer_from=5, staged=1),
                     dict(defer_from=5, hard_lanes=8)]:
            S.ssj_set_plan(ctx, S.make_plan(**plan))
            for sim, a, b in [("jaccard", 1, 3), ("jaccard", 33, 100), ("jaccard", 7, 10), ("jaccard", 1, 1),
                              ("dice", 1, 2), ("dice", 4, 5), ("cosine", 1, 2), ("cosine", 49999, 100000),
                              ("overlap", 1, 1), ("overlap", max(1, n // 2), 1), ("overlap", n, 1), ("overlap", 2**31 - 1, 1)]:
                want = oracle.sort_pairs(oracle.select(c.offsets, c.tokens, cand, a, b, sim=sim))
                got = oracle.sort_pairs(S.ssj_verify_sim(ctx, h, cand, sim, a, b))
                assert np.array_equal(got, want), (n, plan, sim, a, b)
                got = oracle.sort_pairs(S.ssj_verify_groups(ctx, h, h, *S.groups_of(cand), sim, a, b))
                assert np.array_equal(got, want), (n, plan, sim, a, b, "groups")
    finally:
        S.ssj_set_plan(ctx, S.make_plan())
        S.ssj_free_collection(ctx, h)


@pytest.mark.parametrize("n_r, n_s", [(12, 12), (12, 130), (130, 12), (130, 200)])
def test_signatures_of_two_collections(S, ctx, n_r, n_s):
    """Collections with equal and with different signatures."""
    rng = np.random.default_rng(n_r + n_s)
    base = np.sort(rng.choice(400, n_s, replace=False))
    def some(n, k):
        return [np.sort(rng.choice(base if i % 2 else 400, min(n, n_s if i % 2 else 400), replace=False)).tolist() for i in range(k)]
    cr, cs = (synth.collection_from_sets(sorted(x, key=len)) for x in (some(n_r, 40), some(n_s, 50)))
    cand = np.stack(np.meshgrid(np.arange(40), np.arange(50)), axis=-1).reshape(-1, 2).astype(np.int32)
    cand = np.tile(cand, (17, 1))
    hr, hs = (S.ssj_upload_collection(ctx, c.offsets, c.tokens) for c in (cr, cs))
    try:
        for sim, a, b in [("jaccard", 1, 4), ("jaccard", 2, 5), ("jaccard", 7, 10), ("cosine", 3, 5), ("dice", 3, 5), ("overlap", 9, 1)]:
            want = oracle.sort_pairs(oracle.select_rs(cr.offsets, cr.tokens, cs.offsets, cs.tokens, cand, a, b, sim=sim))
            assert np.array_equal(oracle.sort_pairs(S.ssj_verify_rs(ctx, hr, hs, cand, sim, a, b)), want), (sim, a, b)
    finally:
        S.ssj_free_collection(ctx, hr)
        S.ssj_free_collection(ctx, hs)


@pytest.mark.parametrize("n_groups, n_cand", [(1, 1), (1, 512 * 64), (2048, 512 * 64), (2048, 512 * 64 + 1),
                                              (2049, 512 * 64), (2048, 64), (3000, 2048), (1, 512 * 64 + 1)])
def test_small_grouped_launches_with_and_without_a_pre_pass(S, ctx, n_groups, n_cand):
    """Groups and chunks at the bounds up to which the workgroups find their
    groups themselves, with empty groups, and with malformed ends."""
    import torch
    rng = np.random.default_rng(n_cand)
    c = synth.collection_from_sets([np.sort(rng.choice(40, n, replace=False)).tolist()
                                    for n in np.sort(rng.integers(2, 20, 300))])
    probes = rng.integers(0, c.n_sets, n_groups).astype(np.int32)
    ends = np.sort(rng.integers(0, n_cand + 1, n_groups)).astype(np.int32)
    ends[-1] = n_cand
    groups = np.stack([probes, ends], axis=1)
    sids = rng.integers(0, c.n_sets, n_cand).astype(np.int32)
    flat = np.stack([np.repeat(probes, np.diff(ends, prepend=0)), sids], axis=1)
    h = S.ssj_upload_collection(ctx, c.offsets, c.tokens)
    try:
        for plan in [dict(defer_from=5), dict(defer_from=1), dict(inline_lanes=8, defer_from=5)]:
            S.ssj_set_plan(ctx, S.make_plan(**plan))
            want = oracle.sort_pairs(oracle.select(c.offsets, c.tokens, flat, 1, 3))
            got = oracle.sort_pairs(S.ssj_verify_groups(ctx, h, h, groups, sids, "jaccard", 1, 3))
            assert np.array_equal(got, want), plan
            d_s, d_n = torch.from_numpy(sids).cuda(), torch.zeros(1, dtype=torch.int64, device="cuda:0")
            for at, end in [(n_groups - 1, n_cand - 1), (n_groups // 2, n_cand + 1), (n_groups // 2, -1), (0, ends[0])]:
                bad = groups.copy()
                bad[at, 1] = end
                S.ssj_verify_groups_device(ctx, h, h, torch.from_numpy(bad).cuda(), d_s, "jaccard", 1, 3, None, d_n)
                torch.cuda.synchronize()
                assert int(d_n) == (want.shape[0] if end == ends[at] else -1), (plan, at, end)
    finally:
        S.ssj_set_plan(ctx, S.make_plan())
        S.ssj_free_collection(ctx, h)


def test_wide_signatures_at_the_scratch_of_the_allocation_free_call(S):
    """SSJ_NOALLOC_MAX_PAIRS pairs of long sets, whose queue then fills that
    call's scratch exactly, under a plan that queues nothing by itself; and a
    context that has never grown a queue, on a captured stream."""
    import torch
    rng = np.random.default_rng(12)
    base = np.sort(rng.choice(5000, 90, replace=False))
    sets = [np.sort(np.r_[rng.choice(base, 80, replace=False), 5000 + i]).tolist() if i % 2 else
            np.sort(rng.choice(5000, 80, replace=False)).tolist() for i in range(200)]
    c = synth.collection_from_sets(sorted(sets, key=len))
    n = 1 << 20
    cand = rng.integers(0, c.n_sets, (n, 2)).astype(np.int32)
    want = oracle.select(c.offsets, c.tokens, cand, 7, 10).shape[0]
    assert 0 < want < n
    ctx = S.ssj_init(0)
    try:
        S.ssj_set_plan(ctx, S.make_plan(inline_lanes=1, defer_from=5))
        h = S.ssj_upload_collection(ctx, c.offsets, c.tokens)
        d = torch.from_numpy(cand).cuda()
        count = torch.zeros(1, dtype=torch.int64, device="cuda:0")
        S.ssj_verify_device_noalloc(ctx, h, d, 7, 10, None, count)
        torch.cuda.synchronize()
        assert int(count) == want
        g, st = torch.cuda.CUDAGraph(), torch.cuda.Stream()
        with torch.cuda.graph(g, stream=st):
            S.ssj_verify_device(ctx, h, d, 7, 10, None, count, stream=st)
        for _ in range(3):
            count.zero_()
            torch.cuda.synchronize()
            g.replay()
            torch.cuda.synchronize()
            assert int(count) == want
        S.ssj_verify_device(ctx, h, d, 7, 10, None, count)
        torch.cuda.synchronize()
        assert int(count) == want
        del g
    finally:
        S.ssj_shutdown(ctx)


@pytest.mark.parametrize("n", [1, 64 * 4, 64 * 4 + 1, 128 * 4 * 64 - 64, 128 * 4 * 64, 128 * 4 * 64 + 1])
def test_the_end_of_small_launches(S, ctx, n):
    """Launches of one request and of five, with pairs and with counts alone,
    around the grid up to which a workgroup ends with one atomic per request;
    an id out of range is the error of its request alone, and leaves nothing."""
    import torch
    rng = np.random.default_rng(n)
    c = synth.collection_from_sets([np.sort(rng.choice(30, k, replace=False)).tolist() for k in np.sort(rng.integers(2, 15, 200))])
    sizes = [n, 0, max(1, n // 3), 65, n - n // 3]
    cands = [rng.integers(0, c.n_sets, (k, 2)).astype(np.int32) for k in sizes]
    want = [oracle.sort_pairs(oracle.select(c.offsets, c.tokens, k, 1, 2)) for k in cands]
    h = S.ssj_upload_collection(ctx, c.offsets, c.tokens)
    try:
        for plan in [dict(inline_lanes=1, defer_from=5), dict(inline_lanes=8, defer_from=5)]:
            S.ssj_set_plan(ctx, S.make_plan(**plan))
            for some in ([0], [0, 1, 2], [4, 3, 2, 1, 0], [3, 3, 3, 3]):
                for bad in (None, 0, len(some) - 1, None):
                    d_cand, out, count = [], [], []
                    for at, k in enumerate(some):
                        x = cands[k].copy()
                        if at == bad and len(x):
                            x[-1, 1] = c.n_sets
                        d_cand.append(torch.from_numpy(x).cuda())
                        out.append(torch.empty((max(len(x), 1), 2), dtype=torch.int32, device="cuda:0") if at % 2 == 0 else None)
                        count.append(torch.full((1,), -7, dtype=torch.int64, device="cuda:0"))
                    S.ssj_verify_batch_device(ctx, h, [(a, 1, 2, o, m) for a, o, m in zip(d_cand, out, count)])
                    torch.cuda.synchronize()
                    for at, k in enumerate(some):
                        m = int(count[at])
                        if at == bad and len(cands[k]):
                            assert m == -1
                        else:
                            assert m == len(want[k]), (plan, some, bad, at)
                            if out[at] is not None:
                                assert np.array_equal(oracle.sort_pairs(out[at][:m].cpu().numpy()), want[k])
    finally:
        S.ssj_set_plan(ctx, S.make_plan())
        S.ssj_free_collection(ctx, h)


@pytest.mark.parametrize("left", [0, 1, 31, 32, 33, 64])
def test_long_sets_where_signatures_leave_many_pairs(S, ctx, left):
    """Chunks of long sets of which left of 64 pairs are similar: lists of a few
    pairs and of enough to be merged where they are found, pairs shorter and longer
    than the launch merges there (a sixteenth of its chunks), results with and
    without an output buffer, flat and grouped."""
    import torch
    rng = np.random.default_rng(60 + left)
    sets, sim = [], []
    for k in range(60):  # two similar sets of 48 tokens, now and then of 60 or 300
        m = 300 if k % 12 == 5 else 60 if k % 4 == 3 else 48
        base = np.sort(rng.choice(6000, m + 4, replace=False))
        for _ in range(2):
            sets.append(np.sort(rng.choice(base, m, replace=False)).tolist())
    order = np.argsort([len(x) for x in sets], kind="stable")
    where = np.empty(120, dtype=np.int64)
    where[order] = np.arange(120)
    c = synth.collection_from_sets([sets[i] for i in order])
    assert c.n_tokens > 40 * c.n_sets
    sim = np.stack([where[1::2], where[::2]], axis=1).astype(np.int32)
    h = S.ssj_upload_collection(ctx, c.offsets, c.tokens)
    try:
        # merged where they are: none; none; up to 262 tokens; up to 625
        for chunks in (60, 2_000, 4_200, 10_000):
            cand = rng.integers(0, c.n_sets, (chunks, 64, 2)).astype(np.int32)
            cand[:, :left] = sim[rng.integers(0, 60, (chunks, left))]
            cand = cand.reshape(-1, 2)[:-7 if left == 33 else None]
            for sim_, tn, td in [("jaccard", 7, 10), ("cosine", 4, 5)]:
                want = oracle.sort_pairs(oracle.select(c.offsets, c.tokens, cand, tn, td, sim=sim_))
                assert want.shape[0] >= left * chunks * 0.9
                for plan in [dict(), dict(defer_from=5), dict(defer_from=5, staged=1, wg_per_cu=12),
                             dict(defer_from=4, spill_iters=32)]:
                    S.ssj_set_plan(ctx, S.make_plan(**plan))
                    print(f"left {left} chunks {chunks} {sim_} {plan}", flush=True)
                    got = oracle.sort_pairs(S.ssj_verify_sim(ctx, h, cand, sim_, tn, td))
                    assert np.array_equal(got, want)
                    d, n = torch.from_numpy(cand).cuda(), torch.zeros(1, dtype=torch.int64, device="cuda:0")
                    S.ssj_verify_device_sim(ctx, h, d, sim_, tn, td, None, n)
                    assert int(n) == want.shape[0]
                if chunks in (60, 4_200):
                    got = oracle.sort_pairs(S.ssj_verify_groups(ctx, h, h, *S.groups_of(cand), sim_, tn, td))
                    assert np.array_equal(got, want)
    finally:
        S.ssj_set_plan(ctx, S.make_plan())
        S.ssj_free_collection(ctx, h)


def _one_kernel(S, ctx, run):
    """Whether the launches of run have no second kernel."""
    S.ssj_timing_enable(ctx, 1)
    S.ssj_timing_read(ctx, reset=True)
    try:
        run()
        return S.ssj_timing_read(ctx, reset=True)[1] == 0.0
    finally:
        S.ssj_timing_enable(ctx, 0)


@pytest.mark.parametrize("longest", [64, 65, 256, 257])
def test_long_class_bounds_under_the_plan(S, ctx, longest):
    """Sets of more than 40 tokens on average at thresholds below half of them, so
    that launches run as their plan says: the longest pair on either side of a
    class bound (128 | 129, 512 | 513) and budgets at the longest merge."""
    rng = np.random.default_rng(800 + longest)
    base = np.sort(rng.choice(4 * longest, longest, replace=False))
    sets = [np.sort(rng.choice(base, size=int(rng.integers(max(1, longest // 2), longest)), replace=False)).tolist()
            for _ in range(100)]
    sets += [np.sort(rng.choice(4 * longest, int(rng.integers(longest // 2, longest)), replace=False)).tolist()
             for _ in range(50)]
    sets += [base.tolist(), base[1:].tolist(), base.tolist()]
    c = synth.collection_from_sets(sorted(sets, key=len))
    assert c.n_tokens > 40 * c.n_sets
    cand = _pairs(c.n_sets, 5000, 1)
    cand[:3] = [[c.n_sets - 1, c.n_sets - 2], [c.n_sets - 1, c.n_sets - 3], [c.n_sets - 3, c.n_sets - 2]]
    steps = 2 * ((longest + 3) // 4)  # window steps that no merge outruns
    last = int(np.searchsorted([32, 128, 512, 2048], 2 * longest))  # the class of the longest pair
    h = S.ssj_upload_collection(ctx, c.offsets, c.tokens)
    try:
        for sim, tn, td in [("jaccard", 1, 4), ("jaccard", 1, 10), ("overlap", longest // 5, 1), ("cosine", 2, 5)]:
            want = oracle.sort_pairs(oracle.select(c.offsets, c.tokens, cand, tn, td, sim=sim))
            assert 0 < want.shape[0] < cand.shape[0]
            for kw in [dict(defer_from=d, lanes=(4, 8, 16, 64, 256)) for d in range(6)] + \
                      [dict(defer_from=5, spill_iters=s, staged=g) for s in (1, steps - 1, steps) for g in (0, 1)]:
                print(f"longest {longest} {sim} {tn}/{td} {kw}", flush=True)
                S.ssj_set_plan(ctx, S.make_plan(**kw))
                got = []
                one = _one_kernel(S, ctx, lambda: got.append(S.ssj_verify_sim(ctx, h, cand, sim, tn, td)))
                assert np.array_equal(oracle.sort_pairs(got[0]), want)
                assert one == (kw.get("spill_iters", 0) in (0, steps) and last < kw["defer_from"])
    finally:
        S.ssj_set_plan(ctx, S.make_plan())
        S.ssj_free_collection(ctx, h)


@pytest.mark.parametrize("t", [(3, 10), (1, 4), (1, 10)])
def test_long_near_duplicates_under_every_plan(S, ctx, t):
    """Thousands of passing long pairs (10 to 600 tokens) at thresholds below half
    of a mean set: every long-set plan with its own kernel, queues and resumed
    merges, which higher thresholds leave to the signatures' mode."""
    from test_gpu_parity import LONG_PLANS
    from ssj_inputs import filter as cfilter
    rng = np.random.default_rng(31)
    c = synth.near_duplicate_collection(rng, n_base=1500, copies=3, max_size=600, universe=1_000_000,
                                        change_frac=0.08, min_size=10, zipf_s=0.9)
    cand = np.concatenate([cfilter.candidates(c.offsets, c.tokens, 7, 10), _pairs(c.n_sets, 60_000, 9)])
    want = oracle.sort_pairs(oracle.select(c.offsets, c.tokens, cand, *t))
    assert 1000 < want.shape[0] < cand.shape[0]
    h = S.ssj_upload_collection(ctx, c.offsets, c.tokens)
    try:
        for name, plan in LONG_PLANS:
            print(f"long near-dup t={t} {name} n={cand.shape[0]}", flush=True)
            # (None: a new context's plan)
            S.ssj_set_plan(ctx, S.make_plan(**(plan or dict(defer_from=3, lanes=(4, 16, 64, 256, 256)))))
            got = []
            one = _one_kernel(S, ctx, lambda: got.append(S.ssj_verify(ctx, h, cand, *t)))
            assert np.array_equal(oracle.sort_pairs(got[0]), want), name
            assert one == (name in ("inline-16", "inline-64", "staged")), name
            got = oracle.sort_pairs(S.ssj_verify_groups(ctx, h, h, *S.groups_of(cand), "jaccard", *t))
            assert np.array_equal(got, want), name
    finally:
        S.ssj_set_plan(ctx, S.make_plan())
        S.ssj_free_collection(ctx, h)


@pytest.mark.parametrize("staged", [0, 1])
def test_batch_of_counts_and_pairs_of_long_sets(S, ctx, staged):
    """A batch that mixes requests with and without an output buffer on sets of
    more than 40 tokens, where a staged plan has the window ring."""
    import torch
    c = synth.near_duplicate_collection(np.random.default_rng(5), n_base=80, copies=4, max_size=120, min_size=50,
                                        universe=4000)
    assert c.n_tokens > 40 * c.n_sets
    S.ssj_set_plan(ctx, S.make_plan(defer_from=5, staged=staged, wg_per_cu=1))
    h = S.ssj_upload_collection(ctx, c.offsets, c.tokens)
    try:
        sizes = [1, 63, 64, 65, 0, 300, 5000, 200_000, 64, 1, 70_000]
        d_cnt = torch.full((len(sizes),), -7, dtype=torch.int64, device="cuda:0")
        reqs, want, outs = [], [], []
        for i, n in enumerate(sizes):
            cand = _pairs(c.n_sets, n, 40 + i)
            tn, td = [(1, 10), (1, 4), (0, 1)][i % 3]  # at 0 every pair passes: more than are staged
            want.append(oracle.sort_pairs(oracle.select(c.offsets, c.tokens, cand, tn, td)))
            out = None if i % 2 else torch.full((max(n, 1), 2), -1, dtype=torch.int32, device="cuda:0")
            outs.append(out)
            reqs.append((torch.from_numpy(cand).to("cuda:0"), tn, td, out, d_cnt[i:i + 1]))
        for _ in range(3):
            d_cnt.fill_(-7)
            assert _one_kernel(S, ctx, lambda: S.ssj_verify_batch_device(ctx, h, reqs))
            torch.cuda.synchronize()
            for i, w in enumerate(want):
                assert int(d_cnt[i].item()) == w.shape[0], i
                if outs[i] is not None:
                    assert np.array_equal(oracle.sort_pairs(outs[i][:w.shape[0]].cpu().numpy()), w), i
    finally:
        S.ssj_set_plan(ctx, S.make_plan())
        S.ssj_free_collection(ctx, h)


@pytest.mark.parametrize("extra", [0, 1])
@pytest.mark.parametrize("n, most", [(1, 2**31 - 1), (3, 60), (12, 2**31 - 1), (40, 10**6)])
def test_narrow_signatures_of_large_launches(S, ctx, n, most, extra):
    """Pairs of every overlap in lists of 4,096 chunks, which go without narrow
    signatures, and of one pair more, of one collection and of two, flat and grouped."""
    sets = _similar_at(n, most, n + 50, max(1, n // 25))
    c = synth.collection_from_sets(sorted(sets, key=len))
    o = synth.collection_from_sets(sorted(sets[::2] + sets[:5], key=len))
    r, s = np.tril_indices(c.n_sets, 0)
    cand = np.stack([r, s], axis=1).astype(np.int32)
    cand = np.resize(cand, (4096 * 64 + extra, 2))
    cand = cand[np.argsort(cand[:, 0], kind="stable")]
    two = np.stack([cand[:, 0], cand[:, 1] % o.n_sets], axis=1)
    h, ho = (S.ssj_upload_collection(ctx, x.offsets, x.tokens) for x in (c, o))
    try:
        for sim, a, b in [("jaccard", 1, 3), ("jaccard", 7, 10), ("jaccard", 1, 1), ("dice", 1, 2), ("cosine", 1, 2),
                          ("cosine", 49999, 100000), ("overlap", max(1, n // 2), 1), ("overlap", 2**31 - 1, 1)]:
            want = oracle.sort_pairs(oracle.select(c.offsets, c.tokens, cand, a, b, sim=sim))
            want2 = oracle.sort_pairs(oracle.select_rs(c.offsets, c.tokens, o.offsets, o.tokens, two, a, b, sim=sim))
            for plan in [dict(defer_from=3, lanes=(4, 16, 64, 256, 256)), dict(defer_from=5),
                         dict(defer_from=5, spill_iters=2), dict(defer_from=5, hard_lanes=8)]:
                print(f"n {n} + {extra} {sim} {a}/{b} {plan}: {want.shape[0]}", flush=True)
                S.ssj_set_plan(ctx, S.make_plan(**plan))
                assert np.array_equal(oracle.sort_pairs(S.ssj_verify_sim(ctx, h, cand, sim, a, b)), want)
                assert np.array_equal(oracle.sort_pairs(S.ssj_verify_rs(ctx, h, ho, two, sim, a, b)), want2)
            got = oracle.sort_pairs(S.ssj_verify_groups(ctx, h, h, *S.groups_of(cand), sim, a, b))
            assert np.array_equal(got, want)
    finally:
        S.ssj_set_plan(ctx, S.make_plan())
        S.ssj_free_collection(ctx, h)
        S.ssj_free_collection(ctx, ho)
