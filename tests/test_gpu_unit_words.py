"""A context's own words in the arena's first unit do not depend on what the
arena held when it was created: the arena is filled with set bits after
creation, then the context's first call is one that takes tickets (a small
job's roots, count or labels; a large bank's selection).  Every call is made
three times and checked against the CPU oracle, also with the first one
captured into a graph."""
import numpy as np
import pytest
import torch

import oracle
from tests.gpu_util import arena, dev, host, log, u64, zeros_u64

pytestmark = pytest.mark.gpu

SIZES = [5, 3 * 64 * 4096 + 17, 9 * 4096, 31]  # groups of one and of several tiles, buffers of one and of several groups


@pytest.fixture(scope="module")
def pcs():
    import paper_2607_21686_amd as P
    return P


def fresh(pcs, stream=None):
    ar = arena(32 << 20)
    ctx = pcs.Context(ar, stream=stream) if stream else pcs.Context(ar)
    ar.fill_(0xFF)
    torch.cuda.synchronize()
    return ctx


def job(seed):
    rng = np.random.default_rng(seed)
    bufs = [rng.integers(0, 256, size=k, dtype=np.uint8) for k in SIZES]
    return bufs, [dev(b) for b in bufs]


@pytest.mark.parametrize("first", ["fingerprint", "checkpoint", "distance", "verify"])
def test_first_call_of_a_small_job(pcs, first):
    log("unit words", first)
    bufs, d = job(len(first))
    h, r, s = oracle.fingerprint(bufs)
    cpb = [oracle.chunk_count(b.size) for b in bufs]
    words = oracle.bitmap_words(cpb)
    ctx = fresh(pcs)
    plan = [pcs.flat(t) for t in d]
    for turn in range(3):
        H, R, S = zeros_u64(h.size), zeros_u64(len(bufs)), zeros_u64(1)
        if first == "fingerprint":
            ctx.fingerprint(plan, H, R, S)
        elif first == "checkpoint":
            ctx.delete(ctx.checkpoint(plan, hash=True, chunk_hashes=H, roots=R, session_root=S))
        elif first == "distance":
            ref = torch.from_numpy(h.view(np.int64).copy()).cuda()
            ref[turn] += 1
            assert ctx.distance(ref, plan) == 1 / h.size
        else:
            ctx.set_timing(True)  # a timed checkpoint takes no tickets
            snap = ctx.checkpoint(plan, hash=True)
            ctx.set_timing(False)
            back = [torch.zeros_like(t) for t in d]
            bad, lab = zeros_u64(words), torch.full((len(bufs),), 9, dtype=torch.uint8, device="cuda")
            ctx.restore_verify(snap, [pcs.flat(t) for t in back], bad, lab)
            assert not u64(bad)[:words].any() and not host(lab).any()
            assert all(np.array_equal(host(t), b) for t, b in zip(back, bufs))
            ctx.delete(snap)
        if first in ("fingerprint", "checkpoint"):
            assert np.array_equal(u64(H)[:h.size], h) and np.array_equal(u64(R), r) and int(u64(S)[0]) == s
    ctx.close()


def test_first_call_of_a_large_selection(pcs):
    log("unit words, selection")
    n, keep = 40_000, 9_999
    scores = np.random.default_rng(5).standard_normal(n).astype(np.float32)
    ctx = fresh(pcs)
    sc = torch.from_numpy(scores).cuda()
    want = oracle.bank_select(scores, keep)
    for turn in range(3):
        kept = torch.full((keep,), -1, dtype=torch.int32, device="cuda")
        ctx.bank_shrink([], sc, keep, kept)
        assert np.array_equal(kept.cpu().numpy(), want)
    ctx.close()


def test_first_call_captured(pcs):
    log("unit words, captured")
    bufs, d = job(77)
    h, r, s = oracle.fingerprint(bufs)
    side = torch.cuda.Stream()
    ctx = fresh(pcs, side)
    plan = [pcs.flat(t) for t in d]
    H, R, S = zeros_u64(h.size), zeros_u64(len(bufs)), zeros_u64(1)

    def check():
        assert np.array_equal(u64(H)[:h.size], h) and np.array_equal(u64(R), r) and int(u64(S)[0]) == s
        for t in (H, R, S):
            t.zero_()
        torch.cuda.synchronize()

    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        ctx.fingerprint(plan, H, R, S)
    for _ in range(3):
        graph.replay()
        check()
        ctx.fingerprint(plan, H, R, S)  # eager, on the same context and stream
        check()
    ctx.close()
