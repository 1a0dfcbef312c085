"""The self-join on the device at the sizes where its kernels can go wrong:
collections whose set sizes do not ascend with the id (no table of first
entries), probes of exactly 63 to 65 meetings and lists that fill more than one
work unit, merges that outrun the step budget, sets of one token, results
around the output's capacity; against the oracle on the CPU filter's
candidates (whole numbers: no tolerance)."""
import os
import sys

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)

import oracle  # noqa: E402
from ssj_inputs import filter as cfilter  # noqa: E402
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


def _shuffled(c, seed):
    perm = np.random.default_rng(seed).permutation(c.n_sets)
    return synth.collection_from_sets([c.set(int(i)).tolist() for i in perm])


def _collection(name):
    rng = np.random.default_rng(4100)
    if name in ("near duplicates", "near duplicates, sizes shuffled"):
        c = synth.near_duplicate_collection(rng, n_base=150, copies=4, max_size=60, universe=700)
        return c if name == "near duplicates" else _shuffled(c, 1)
    if name == "lists of 64 to 66 sets":
        # token k is shared by 64 + k % 3 sets, every set has a token of its own too
        sets = []
        for k in range(12):
            sets += [sorted([k, 100 + 70 * k + i]) for i in range(64 + k % 3)]
        return synth.collection_from_sets(sorted(sets, key=len))
    if name == "one long list":
        # 700 sets share their first token: 244,650 meetings of 11 groups
        return synth.collection_from_sets([[0, 1 + i, 2000 + i // 7, 3000 + i // 7] for i in range(700)])
    if name == "long merges":
        # near-copies of sets of 300 to 2,000 tokens, of which the first 40 differ
        sets = []
        for b in range(6):
            n = (300, 301, 640, 999, 1500, 2000)[b]
            body = np.sort(rng.choice(np.arange(5000, 12000), n, replace=False))
            for v in range(4):
                drop = rng.random(n) < 0.03
                head = np.sort(rng.choice(5000, 8 * v, replace=False))
                sets.append(np.concatenate([head, body[~drop]]).tolist())
        return synth.collection_from_sets(sorted(sets, key=len))
    if name == "single tokens":
        return synth.collection_from_sets([[int(t)] for t in rng.integers(0, 9, 200)])
    raise KeyError(name)


@pytest.mark.parametrize("name", ["near duplicates", "near duplicates, sizes shuffled", "lists of 64 to 66 sets",
                                  "one long list", "long merges", "single tokens"])
def test_join_equals_the_oracle(S, ctx, name):
    import torch
    c = _collection(name)
    h = S.ssj_upload_collection(ctx, c.offsets, c.tokens)
    try:
        for tn, td in [(1, 4), (1, 2), (7, 10), (9, 10), (1, 1)]:
            # the filter's own collections are ordered by size: all pairs where this one is not
            if np.all(np.diff(c.sizes()) >= 0):
                cand = cfilter.candidates(c.offsets, c.tokens, tn, td)
            else:
                r, s = np.tril_indices(c.n_sets, -1)
                cand = np.stack([r, s], axis=1).astype(np.int32)
            want = oracle.sort_pairs(oracle.select(c.offsets, c.tokens, cand, tn, td))
            k = want.shape[0]
            print(f"{name} t={tn}/{td}: {k}", flush=True)
            for positional in (False, True):
                assert np.array_equal(oracle.sort_pairs(S.ssj_join(ctx, h, tn, td, positional)), want)
            # capacities just below and at the result, and the count alone
            d_cnt = torch.zeros(1, dtype=torch.int64, device="cuda:0")
            for cap in {max(k - 1, 0), k, 0}:
                d_out = torch.full((cap + 1, 2), -1, dtype=torch.int32, device="cuda:0")
                S.ssj_join_device(ctx, h, tn, td, True, d_out[:cap] if cap else None, d_cnt)
                torch.cuda.synchronize()
                assert int(d_cnt.item()) == k
                got = d_out.cpu().numpy()
                assert (got[cap] == -1).all()
                if cap == k and k:
                    assert np.array_equal(oracle.sort_pairs(got[:k]), want)
            if k > 1:
                with pytest.raises(S.SsjError) as e:
                    S.ssj_join(ctx, h, tn, td, True, out_cap=k - 1)
                assert e.value.code == S.SSJ_ETRUNC and e.value.n == k
    finally:
        S.ssj_free_collection(ctx, h)
