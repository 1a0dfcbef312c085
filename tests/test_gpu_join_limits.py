"""Whole joins at the limits of the path that takes them: thousands of equal
sets beside many other sizes at thresholds near 1, on both sides of the number
of prefix entries up to which the host does not wait for the meetings; more
meetings than the join's own path takes; and prefixes that are refused.  The
similar pairs are known from how the sets are made (whole numbers: no
tolerance)."""
import os
import sys

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)


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


def _csr(sizes, tokens):
    off = np.zeros(len(sizes) + 1, dtype=np.int64)
    np.cumsum(sizes, out=off[1:])
    assert off[-1] == tokens.shape[0]
    return off, tokens.astype(np.int32)


def _copies(copies, size, others, singles=0):
    """copies equal sets of size tokens, and besides them sets without a partner:
    one of every size in others, and single tokens."""
    n0 = max(size, 1)
    parts, at = [], n0 + singles
    if singles:
        parts += [([1], np.array([n0 + i])) for i in range(singles)]
    body = [(np.full(copies, size), np.tile(np.arange(size), copies))]
    for k in others:
        parts.append(([k], np.arange(at, at + k)))
        at += k
    lo = [p for p in parts if p[0][0] < size]
    hi = [p for p in parts if p[0][0] >= size]
    all_ = lo + body + hi
    return _csr(np.concatenate([p[0] for p in all_]), np.concatenate([p[1] for p in all_])), len(lo)


def _count(S, ctx, h, tn, td, out=None):
    import torch
    n = torch.full((1,), -7, dtype=torch.int64, device="cuda:0")
    S.ssj_join_device(ctx, h, tn, td, True, out, n)
    torch.cuda.synchronize()
    return int(n)


# (copies, their size, other sizes, single tokens, threshold): 14,000, 21,000,
# 52,414, 25,600 and 65,536 prefix entries at t = 1 and near it, 65,537 and 71,000
@pytest.mark.parametrize("copies, size, others, singles, t", [
    (12_000, 1, range(2, 2002), 0, (1, 1)), (20_000, 10, range(11, 1011), 0, (1, 1)),
    (50_000, 1, range(2, 301), 0, (19, 20)), (25_000, 7, range(8, 601), 0, (99, 100)),
    (40_000, 3, range(4, 504), 25_036, (1, 1)), (40_000, 3, range(4, 504), 25_037, (1, 1)),
    (25_000, 2, range(3, 1003), 45_000, (1, 1))])
def test_equal_sets_beside_many_sizes(S, ctx, copies, size, others, singles, t):
    import torch
    (off, tok), first = _copies(copies, size, others, singles)
    want = copies * (copies - 1) // 2
    print(f"{copies} copies of {size}, {len(others)} sizes, {singles} singles, t={t}: {want}", flush=True)
    h = S.ssj_upload_collection(ctx, off, tok)
    try:
        assert _count(S, ctx, h, *t) == want
        with pytest.raises(S.SsjError) as e:
            S.ssj_join(ctx, h, *t, out_cap=1000)
        assert e.value.code == S.SSJ_ETRUNC and e.value.n == want
        if want < 100_000_000:  # the pairs themselves: every one of the copies, once
            out = torch.empty((want, 2), dtype=torch.int32, device="cuda:0")
            assert _count(S, ctx, h, *t, out) == want
            r, s = out[:, 0].long() - first, out[:, 1].long() - first
            assert bool((s >= 0).all()) and bool((r > s).all()) and bool((r < copies).all())
            key = torch.sort(r * copies + s).values
            assert bool((key[1:] != key[:-1]).all())
    finally:
        S.ssj_free_collection(ctx, h)


def test_more_meetings_than_the_join_takes(S, ctx):
    """66,000 sets that share their first token, sizes in no order: 2,177,967,000
    meetings, which are left to candidates and their verification."""
    rng = np.random.default_rng(31)
    n = 66_000
    sizes = rng.integers(2, 42, n)
    kind = rng.integers(0, 150, n)  # equal size and kind: equal sets
    off = np.zeros(n + 1, dtype=np.int64)
    np.cumsum(sizes, out=off[1:])
    at = np.arange(off[-1]) - np.repeat(off[:-1], sizes)
    tok = np.where(at == 0, 0, np.repeat(1 + 100 * kind, sizes) + at)
    _, c = np.unique(sizes * 1000 + kind, return_counts=True)
    h = S.ssj_upload_collection(ctx, off, tok.astype(np.int32))
    try:
        want = int((c.astype(np.int64) * (c - 1) // 2).sum())
        assert _count(S, ctx, h, 1, 1) == want
        assert S.ssj_join(ctx, h, 1, 1).shape[0] == want
    finally:
        S.ssj_free_collection(ctx, h)


def test_prefixes_that_too_many_sets_share_are_refused(S, ctx):
    """530,000 sets of 74 sizes share their first token: 2,194,787,975 pieces of
    64 list entries, above the 2^31 that a join takes, though at t = 1
    only sets of one size meet.  With half of the sets it is taken."""
    for n, refused in [(530_000, True), (265_000, False)]:
        sizes = np.sort(2 + np.arange(n) % 74)
        off = np.zeros(n + 1, dtype=np.int64)
        np.cumsum(sizes, out=off[1:])
        at = np.arange(off[-1]) - np.repeat(off[:-1], sizes)
        tok = np.where(at == 0, 0, np.repeat(1 + 100 * (np.arange(n) // 2), sizes) + at)  # pairs of neighbours
        key = sizes * n + np.arange(n) // 2
        want = int((key[1:] == key[:-1]).sum())
        h = S.ssj_upload_collection(ctx, off, tok.astype(np.int32))
        try:
            if refused:
                with pytest.raises(S.SsjError) as e:
                    S.ssj_join(ctx, h, 1, 1)
                assert e.value.code == S.SSJ_ENOMEM
                with pytest.raises(S.SsjError) as e:
                    _count(S, ctx, h, 1, 1)
                assert e.value.code == S.SSJ_ENOMEM
            else:
                assert _count(S, ctx, h, 1, 1) == want
                assert S.ssj_join(ctx, h, 1, 1).shape[0] == want
        finally:
            S.ssj_free_collection(ctx, h)


def test_short_device_memory_leaves_a_join_to_the_candidates(S):
    """45,000 sets that share their first token, sizes in no order, and an output
    for as many pairs as they meet, with 4 GiB of the device left: neither 8 GiB
    for the 1.0e9 meetings' pairs nor a failure; with memory the same result."""
    import torch
    rng = np.random.default_rng(32)
    n = 45_000
    sizes = rng.integers(2, 42, n)
    kind = rng.integers(0, 400, n)  # equal size and kind: equal sets
    off = np.zeros(n + 1, dtype=np.int64)
    np.cumsum(sizes, out=off[1:])
    at = np.arange(off[-1]) - np.repeat(off[:-1], sizes)
    tok = np.where(at == 0, 0, np.repeat(1 + 100 * kind, sizes) + at)
    _, c = np.unique(sizes * 1000 + kind, return_counts=True)
    want = int((c.astype(np.int64) * (c - 1) // 2).sum())
    ctx = S.ssj_init(0)
    try:
        h = S.ssj_upload_collection(ctx, off, tok.astype(np.int32))
        torch.cuda.empty_cache()
        rest = torch.empty(torch.cuda.mem_get_info()[0] - (4 << 30), dtype=torch.uint8, device="cuda:0")
        got = S.ssj_join(ctx, h, 1, 1, out_cap=1 << 30)
        assert got.shape[0] == want
        del rest
        torch.cuda.empty_cache()
        again = S.ssj_join(ctx, h, 1, 1, out_cap=1 << 30)
        key = [np.sort(x[:, 0].astype(np.int64) << 32 | x[:, 1]) for x in (got, again)]
        assert np.array_equal(*key)
        for x in key[:1]:
            assert (x[1:] != x[:-1]).all()
        assert (sizes[got[:, 0]] == sizes[got[:, 1]]).all() and (kind[got[:, 0]] == kind[got[:, 1]]).all()
        assert S.ssj_join(ctx, h, 1, 1).shape[0] == want
    finally:
        S.ssj_shutdown(ctx)
