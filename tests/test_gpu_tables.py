"""Both sides of what a job's argument tables hold (96 buffers, 16 rings in
more than one piece) through every call that reads them: fingerprints, a
fingerprinted checkpoint, plain and verified restores, an incremental
checkpoint with a few dirty chunks, classification and distance; buffers are
ragged, some empty.  And windows whose chunks span many pieces in jobs of
whole-group tiles, which take each granule's address from the geometry.
Everything against the CPU oracle, exactly."""
import numpy as np
import pytest
import torch

import oracle
import workloads as W
from tests.gpu_util import arena, dev, host, log, u64, zeros_u64

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pcs():
    import paper_2607_21686_amd as P
    return P


def check_all_calls(pcs, srcs, dsts, logical, changed, after):
    """srcs(live=True) / dsts(): descriptors; logical(): the oracle's bytes of
    each buffer; changed(): modifies a few chunks of the live state; after():
    the destinations' bytes, as logical() gives them."""
    ctx = pcs.Context(arena(512 << 20))
    bufs = logical()
    h, r, s = oracle.fingerprint(bufs)
    n, T = len(bufs), h.size
    cpb = [oracle.chunk_count(b.size) for b in bufs]

    def outs():
        return zeros_u64(T), zeros_u64(n), zeros_u64(1)

    def same(o, h, r, s):
        assert np.array_equal(u64(o[0])[:h.size], h)
        assert np.array_equal(u64(o[1]), r)
        assert int(u64(o[2])[0]) == s

    for call in (ctx.fingerprint, ctx.fingerprint_noalloc):
        o = outs()
        call(srcs(), *o)
        same(o, h, r, s)
    o = outs()
    full = ctx.checkpoint(srcs(), hash=True, chunk_hashes=o[0], roots=o[1], session_root=o[2])
    same(o, h, r, s)
    plain = ctx.checkpoint(srcs())
    old = o[0].clone()
    assert ctx.distance(old, srcs()) == 0.0
    changed()
    bufs2 = logical()
    h2, r2, s2 = oracle.fingerprint(bufs2)
    dirty = int((h != h2).sum())
    assert ctx.distance(old, srcs()) == dirty / T
    o = outs()
    inc = ctx.checkpoint(srcs(), parent=full, chunk_hashes=o[0], roots=o[1], session_root=o[2])
    same(o, h2, r2, s2)
    assert ctx.info(inc)["dirty_chunks"] == dirty
    words = oracle.bitmap_words(cpb)
    for snap, want in ((full, bufs), (plain, bufs), (inc, bufs2)):
        ctx.restore(snap, dsts())
        assert all(np.array_equal(a, b) for a, b in zip(after(), want))
    for snap, want in ((inc, bufs2), (full, bufs)):
        bad, lab = zeros_u64(words), torch.full((n,), 7, dtype=torch.uint8, device="cuda")
        bad.fill_(-1)
        ctx.restore_verify(snap, dsts(), bad, lab)
        assert all(np.array_equal(a, b) for a, b in zip(after(), want))
        assert not u64(bad)[:words].any() and not host(lab).any()
    gh = torch.stack([old[:T], o[0][:T], old[:T]])
    bm, lab = zeros_u64(words), torch.full((n,), 7, dtype=torch.uint8, device="cuda")
    ctx.classify(gh, 3, cpb, bm, lab)
    obm, olab = oracle.classify(np.stack([h, h2, h]), cpb)
    assert np.array_equal(u64(bm)[:words], obm) and np.array_equal(host(lab), olab)
    ctx.close()


@pytest.mark.parametrize("nbuf", [1, 63, 64, 65, 95, 96, 97])
@pytest.mark.parametrize("large", [False, True])
def test_flat_buffers(pcs, nbuf, large):
    rng = np.random.default_rng([nbuf, large])
    top = (60 << 20) // nbuf if large else 200_000
    sizes = [int(rng.integers(1, top)) for _ in range(nbuf)]
    sizes[0] = top if large else 5
    for i in range(7, nbuf, 13):
        sizes[i] = 0
    if nbuf > 1:
        sizes[-1] = 0 if nbuf % 2 else 33
    log("tables flat", nbuf, "large" if large else "small")
    bufs = [rng.integers(0, 256, size=k, dtype=np.uint8) for k in sizes]
    live = [dev(b) if b.size else torch.zeros(16, dtype=torch.uint8, device="cuda") for b in bufs]
    back = [torch.zeros_like(t) for t in live]

    def changed():
        for i in range(0, nbuf, 5):
            if sizes[i]:
                for at in {0, sizes[i] // 2, sizes[i] - 1}:
                    live[i][at] += 1

    check_all_calls(pcs, lambda: [pcs.flat(t, k) for t, k in zip(live, sizes)],
                    lambda: [pcs.flat(t, k) for t, k in zip(back, sizes)],
                    lambda: [host(t)[:k] for t, k in zip(live, sizes)], changed,
                    lambda: [host(t)[:k] for t, k in zip(back, sizes)])


def rings_case(pcs, geoms, heads2):
    """Rings, with a flat buffer first and between them."""
    rng = np.random.default_rng([len(geoms), geoms[0].outer])
    mem = [rng.integers(0, 256, size=g.ring_bytes, dtype=np.uint8) for g in geoms]
    live = [dev(m) for m in mem]
    back = [torch.zeros_like(t) for t in live]
    flat_live, flat_back = dev(rng.integers(0, 256, size=70_001, dtype=np.uint8)), torch.zeros(70_001, dtype=torch.uint8, device="cuda")
    to = [g.with_head(h) for g, h in zip(geoms, heads2)]

    def descs(ts, gs, flat):
        d = [pcs.flat(flat)]
        for t, g in zip(ts, gs):
            d.append(pcs.ring(t, g.outer, g.capacity, g.row_bytes, g.head, g.window, g.outer_stride))
        return d + [pcs.flat(flat, 16) if flat is flat_live else pcs.flat(tail_back)]

    tail_back = torch.zeros(16, dtype=torch.uint8, device="cuda")

    def windows(ts, gs):
        return [oracle.ring_window(host(t), g.outer, g.outer_stride, g.capacity, g.row_bytes, g.head, g.window)
                for t, g in zip(ts, gs)]

    def changed():
        for t, g in zip(live, geoms):
            t[g.head * g.row_bytes] += 1           # the first window byte
            t[(g.outer - 1) * g.outer_stride + (g.head + g.window - 1) % g.capacity * g.row_bytes] += 1

    check_all_calls(pcs, lambda: descs(live, geoms, flat_live), lambda: descs(back, to, flat_back),
                    lambda: [host(flat_live)] + windows(live, geoms) + [host(flat_live)[:16]], changed,
                    lambda: [host(flat_back)] + windows(back, to) + [host(tail_back)])


@pytest.mark.parametrize("nring", [1, 7, 8, 9, 15, 16, 17])
def test_rings(pcs, nring):
    log("tables rings", nring)
    # (every window wraps, so that each ring is one of the rings the tables count)
    shapes = [(3, 700, 2048, 500), (2, 100, 48, 99), (1, 9, 4096, 5), (64, 40, 256, 33), (5, 64, 1008, 64)]
    geoms, heads2 = [], []
    for i in range(nring):
        outer, cap, row, win = shapes[i % len(shapes)]
        geoms.append(W.Ring(outer, cap, row, win, cap - 1 - i % 3, cap * row + 16 * (i % 2)))
        heads2.append((3 + 5 * i) % cap)
    rings_case(pcs, geoms, heads2)


@pytest.mark.parametrize("outer,cap,row,win", [(32000, 90, 16, 80), (700, 70, 1024, 48), (9, 265, 1024, 257),
                                               (150, 265, 1024, 257)])
def test_many_pieces_in_whole_group_tiles(pcs, outer, cap, row, win):
    """More than 128 groups of windows whose pieces are shorter than a chunk
    (16-byte rows: up to eight pieces a chunk; 1 KiB rows wrapping after one).
    The last two: tiles in which one chunk of three pieces stands among whole
    ones, in eighths of groups and in whole groups."""
    log("tables many pieces", outer, cap, row, win)
    rings_case(pcs, [W.Ring(outer, cap, row, win, cap - 1)], [cap - 2])


@pytest.mark.parametrize("nring", [9, 16])
def test_rings_take_no_arena_space(pcs, nring):
    """Up to 16 wrapped rings (one per layer and K or V, say) travel in the
    kernel arguments: they restore, plain and verified, from an arena with no
    free unit, and their allocation-free fingerprint stages nothing, so it
    can be captured."""
    log("tables rings, full arena", nring)
    rng = np.random.default_rng(nring)
    g = W.Ring(1, 70, 1008, 64, 60)
    side = torch.cuda.Stream()
    ctx = pcs.Context(arena(8 << 20), stream=side)
    live = [dev(rng.integers(0, 256, size=g.ring_bytes, dtype=np.uint8)) for _ in range(nring)]
    back = [torch.zeros_like(t) for t in live]
    torch.cuda.synchronize()

    def descs(ts):
        return [pcs.ring(t, g.outer, g.capacity, g.row_bytes, g.head, g.window) for t in ts]

    def windows(ts):
        return [oracle.ring_window(host(t), g.outer, g.outer_stride, g.capacity, g.row_bytes, g.head, g.window) for t in ts]

    want = windows(live)
    h, r, s = oracle.fingerprint(want)
    words = oracle.bitmap_words([oracle.chunk_count(b.size) for b in want])
    snap = ctx.checkpoint(descs(live), hash=True)
    one = [pcs.flat(live[0], 16)]
    with pytest.raises(pcs.PcsError):
        while True:
            ctx.checkpoint(one)
    assert ctx.arena_stats()["free"] == 0
    ctx.restore(snap, descs(back))
    assert all(np.array_equal(a, b) for a, b in zip(windows(back), want))
    for t in back:
        t.zero_()
    torch.cuda.synchronize()
    bad, lab = zeros_u64(words), torch.full((nring,), 7, dtype=torch.uint8, device="cuda")
    torch.cuda.synchronize()
    ctx.restore_verify(snap, descs(back), bad, lab)
    assert all(np.array_equal(a, b) for a, b in zip(windows(back), want))
    assert not u64(bad)[:words].any() and not host(lab).any()
    H, R, S = zeros_u64(h.size), zeros_u64(nring), zeros_u64(1)
    torch.cuda.synchronize()
    plan = pcs.BufArray(descs(live))
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        ctx.fingerprint_noalloc(plan, H, R, S)
    for _ in range(3):
        for t in (H, R, S):
            t.zero_()
        torch.cuda.synchronize()
        graph.replay()
        assert np.array_equal(u64(H)[:h.size], h) and np.array_equal(u64(R), r) and int(u64(S)[0]) == s
        ctx.restore(snap, descs(back))  # eager work of the context between replays
    ctx.close()
