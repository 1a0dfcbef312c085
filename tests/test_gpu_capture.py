"""Calls on a stream that is being captured: a captured launch holds only
scratch that its plan uses by itself, so that a larger call between capture and
replay takes nothing from under it; a plan's merge states are left out where no
call has made room for them; whole joins are refused."""
import ctypes
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


class Graph:
    """The work that calls enqueue on a stream of its own, as a graph."""

    def __init__(self):
        import torch
        self.hip = ctypes.CDLL("libamdhip64.so")
        self.stream = torch.cuda.Stream()
        self.st = ctypes.c_void_p(self.stream.cuda_stream)
        self.graph, self.exe = ctypes.c_void_p(), ctypes.c_void_p()

    def capture(self, call):
        assert self.hip.hipStreamBeginCapture(self.st, 2) == 0  # relaxed
        try:
            call(self.stream)
        finally:
            assert self.hip.hipStreamEndCapture(self.st, ctypes.byref(self.graph)) == 0

    def nodes(self):
        n = ctypes.c_size_t()
        assert self.hip.hipGraphGetNodes(self.graph, None, ctypes.byref(n)) == 0
        return n.value

    def replay(self):
        if not self.exe:
            assert self.hip.hipGraphInstantiate(ctypes.byref(self.exe), self.graph, None, None, 0) == 0
        assert self.hip.hipGraphLaunch(self.exe, self.st) == 0
        self.stream.synchronize()

    def close(self):
        if self.exe:
            self.hip.hipGraphExecDestroy(self.exe)
        if self.graph:
            self.hip.hipGraphDestroy(self.graph)


def _long_sets(n=300):
    rng = np.random.default_rng(12)
    base = np.sort(rng.choice(5000, 90, replace=False))
    sets = [np.sort(np.r_[rng.choice(base, 80, replace=False), 5000 + i]).tolist() if i % 2 else
            np.sort(rng.choice(5000, 80, replace=False)).tolist() for i in range(n)]
    return synth.collection_from_sets(sorted(sets, key=len)), rng


@pytest.mark.parametrize("grouped", [False, True])
@pytest.mark.parametrize("plan, kernels", [(dict(defer_from=5), 1), (dict(defer_from=5, staged=1), 1),
                                           (dict(defer_from=2), 2), (dict(defer_from=5, spill_iters=2), 2)])
def test_replays_after_a_larger_call(S, plan, kernels, grouped):
    """Long sets at a threshold for which eager launches queue their pairs: a
    plan that queues nothing is captured as one kernel without a queue, and its
    replays after a larger call, and that call's, are right."""
    import torch
    c, rng = _long_sets()
    few = rng.integers(0, c.n_sets, (20_000, 2)).astype(np.int32)
    few = few[np.argsort(few[:, 0], kind="stable")]
    many = rng.integers(0, c.n_sets, (300_000, 2)).astype(np.int32)
    want = [oracle.select(c.offsets, c.tokens, x, 7, 10).shape[0] for x in (few, many)]
    assert 0 < want[0] < few.shape[0]
    ctx = S.ssj_init(0)
    g = Graph()
    try:
        S.ssj_set_plan(ctx, S.make_plan(**plan))
        h = S.ssj_upload_collection(ctx, c.offsets, c.tokens)
        n, n2 = (torch.zeros(1, dtype=torch.int64, device="cuda:0") for _ in range(2))
        d, d2 = torch.from_numpy(few).cuda(), torch.from_numpy(many).cuda()
        gr, si = (torch.from_numpy(x).cuda() for x in S.groups_of(few))

        def call(stream=None):
            if grouped:
                S.ssj_verify_groups_device(ctx, h, h, gr, si, "jaccard", 7, 10, None, n, stream=stream)
            else:
                S.ssj_verify_device(ctx, h, d, 7, 10, None, n, stream=stream)

        call()
        torch.cuda.synchronize()
        assert int(n) == want[0]
        n.zero_()
        g.capture(call)
        if kernels == 1:
            assert g.nodes() == 1
            S.ssj_verify_device(ctx, h, d2, 7, 10, None, n2)  # grows what launches queue in
            torch.cuda.synchronize()
            assert int(n2) == want[1]
        assert g.nodes() == kernels
        for _ in range(3):
            n.zero_()
            torch.cuda.synchronize()
            g.replay()
            assert int(n) == want[0]
            call()
            torch.cuda.synchronize()
            assert int(n) == want[0]
    finally:
        g.close()
        S.ssj_shutdown(ctx)


def test_a_budget_plan_captured_without_its_states(S):
    """Warmed up where long sets queue whole pairs, captured where merges are cut
    off: they restart, with no allocation in between."""
    import torch
    c, rng = _long_sets()
    cand = rng.integers(0, c.n_sets, (20_000, 2)).astype(np.int32)
    want = oracle.select(c.offsets, c.tokens, cand, 3, 10).shape[0]
    assert 0 < want < cand.shape[0]
    ctx = S.ssj_init(0)
    g = Graph()
    try:
        S.ssj_set_plan(ctx, S.make_plan(defer_from=5, spill_iters=2, spill_lanes=16))
        h = S.ssj_upload_collection(ctx, c.offsets, c.tokens)
        n = torch.zeros(1, dtype=torch.int64, device="cuda:0")
        d = torch.from_numpy(cand).cuda()
        S.ssj_verify_device(ctx, h, d, 7, 10, None, n)
        torch.cuda.synchronize()
        free = torch.cuda.mem_get_info()[0]
        g.capture(lambda stream: S.ssj_verify_device(ctx, h, d, 3, 10, None, n, stream=stream))
        assert torch.cuda.mem_get_info()[0] == free
        for _ in range(3):
            n.zero_()
            torch.cuda.synchronize()
            g.replay()
            assert int(n) == want
            S.ssj_verify_device(ctx, h, d, 3, 10, None, n)
            torch.cuda.synchronize()
            assert int(n) == want
    finally:
        g.close()
        S.ssj_shutdown(ctx)


def test_joins_are_not_captured(S):
    """A join small enough to run without waiting for its totals, with all its
    scratch made, is refused on a stream being captured; nothing is enqueued and
    the context goes on."""
    import torch
    c = synth.near_duplicate_collection(np.random.default_rng(3), n_base=100, copies=3, max_size=20, universe=300)
    ctx = S.ssj_init(0)
    g = Graph()
    try:
        h = S.ssj_upload_collection(ctx, c.offsets, c.tokens)
        n = torch.zeros(1, dtype=torch.int64, device="cuda:0")
        S.ssj_join_device(ctx, h, 7, 10, True, None, n)
        torch.cuda.synchronize()
        want = int(n)
        assert want > 0

        def call(stream):
            with pytest.raises(S.SsjError) as e:
                S.ssj_join_device(ctx, h, 7, 10, True, None, n, stream=stream)
            assert e.value.code == S.SSJ_EINVAL

        g.capture(call)
        assert g.nodes() == 0
        n.zero_()
        S.ssj_join_device(ctx, h, 7, 10, True, None, n)
        torch.cuda.synchronize()
        assert int(n) == want
    finally:
        g.close()
        S.ssj_shutdown(ctx)
