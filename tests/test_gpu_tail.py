"""Small jobs whose 8-chunk tiles finish them in the same launch: buffer and
session roots (fingerprints, fingerprinted checkpoints), the count of a
distance and the labels of a verified restore, at the edges of a tile (8
chunks), a group (64) and the job (128 groups), of one to 96 buffers, several
times in a row on one context (the tickets must come back to zero), against the
CPU oracle.  A job with an empty buffer takes launches of their own and gives
the same."""
import numpy as np
import pytest
import torch

import oracle
from tests.gpu_util import arena, dev, host, log, u64, zeros_u64

pytestmark = pytest.mark.gpu

C, GROUP = 4096, 64 * 4096
JOBS = {
    "one byte": [1], "one tile": [8 * C], "tile + 1": [8 * C + 1], "7 tiles": [56 * C - 3], "group": [GROUP],
    "group + 1": [GROUP + 1], "2 groups": [2 * GROUP], "64 groups": [64 * GROUP], "65 groups": [65 * GROUP - 9],
    "128 groups": [128 * GROUP], "2 x 64 groups": [64 * GROUP, 63 * GROUP + 77],
    "96 tiny": [1 + 37 * i for i in range(96)], "96 ragged": [(i % 9) * 8 * C + 1 + i for i in range(96)],
    "65 buffers": [C * (1 + i % 20) for i in range(65)], "mixed": [5, 3 * GROUP + 17, 9 * C, 40 * GROUP, 31],
    "with an empty one": [5, 0, GROUP, 9 * C],
}


@pytest.fixture(scope="module")
def pcs():
    import paper_2607_21686_amd as P
    return P


@pytest.mark.parametrize("name", list(JOBS))
def test_tail(pcs, name):
    sizes = JOBS[name]
    rng = np.random.default_rng(len(name) + len(sizes))
    bufs = [rng.integers(0, 256, size=k, dtype=np.uint8) for k in sizes]
    log("tail", name)
    h, r, s = oracle.fingerprint(bufs)
    n, T, cpb = len(bufs), h.size, [oracle.chunk_count(k) for k in sizes]
    words = oracle.bitmap_words(cpb)
    ar = arena(256 << 20)
    ctx = pcs.Context(ar)
    d = [dev(b) if b.size else torch.zeros(16, dtype=torch.uint8, device="cuda") for b in bufs]
    plan = pcs.BufArray([pcs.flat(t, k) for t, k in zip(d, sizes)])
    back = [torch.zeros_like(t) for t in d]
    dst = pcs.BufArray([pcs.flat(t, k) for t, k in zip(back, sizes)])
    ref = None
    for turn in range(3):
        H, R, S = zeros_u64(T), zeros_u64(n), zeros_u64(1)
        if turn == 1:
            ctx.fingerprint(plan, H, R)       # no session root: buffers finish alone
        elif turn == 2:
            ctx.fingerprint(plan, None, None, S)
        else:
            ctx.fingerprint(plan, H, R, S)
        if turn != 2:
            assert np.array_equal(u64(H)[:T], h) and np.array_equal(u64(R), r)
        if turn != 1:
            assert int(u64(S)[0]) == s
        H, R, S = zeros_u64(T), zeros_u64(n), zeros_u64(1)
        snap = ctx.checkpoint(plan, hash=True, chunk_hashes=H, roots=R, session_root=S)
        assert np.array_equal(u64(H)[:T], h) and np.array_equal(u64(R), r) and int(u64(S)[0]) == s
        ref = H if ref is None else ref
        # Distance: a few chunks changed in the reference.
        assert ctx.distance(ref, plan) == 0.0
        hit = sorted({0, T // 2, T - 1})
        other = ref.clone()
        other[hit] += 1
        assert ctx.distance(other, plan) == len(hit) / T
        assert ctx.distance(torch.zeros_like(ref) if 0 not in h else other, plan) == (1.0 if 0 not in h else len(hit) / T)
        # Verified restore: clean, then with the first byte of the first and
        # the last chunk's slot flipped.
        addr, nbytes = ctx.view(snap)
        for flips in ([], [0, nbytes - C]):
            for at in set(flips):
                ar[addr - ar.data_ptr() + at] ^= 1
            bad, lab = zeros_u64(words), torch.full((n,), 9, dtype=torch.uint8, device="cuda")
            bad.fill_(-1)
            for t in back:
                t.zero_()
            ctx.restore_verify(snap, dst, bad, lab)
            got = [host(t)[:k] for t, k in zip(back, sizes)]
            obm, olab = oracle.classify(np.stack([h, oracle.fingerprint(got)[0]]), cpb)
            assert np.array_equal(u64(bad)[:words], obm) and np.array_equal(host(lab), olab)
            assert int(olab.sum()) == (0 if not flips else len({0, max(i for i, k in enumerate(sizes) if k)}))
        ctx.delete(snap)
    ctx.close()


@pytest.mark.parametrize("name", ["96 ragged", "2 x 64 groups", "mixed"])
def test_tail_beside_a_busy_stream(pcs, name):
    """The same hand-over between workgroups while another stream keeps the CUs,
    caches and memory busy: every root, count and label of forty turns."""
    sizes = JOBS[name]
    rng = np.random.default_rng(len(name))
    bufs = [rng.integers(0, 256, size=k, dtype=np.uint8) for k in sizes]
    log("tail beside a busy stream", name)
    h, r, s = oracle.fingerprint(bufs)
    n, T, cpb = len(bufs), h.size, [oracle.chunk_count(k) for k in sizes]
    words = oracle.bitmap_words(cpb)
    turns = 40
    side, load = torch.cuda.Stream(), torch.cuda.Stream()
    d = [dev(b) for b in bufs]
    back = [torch.zeros_like(t) for t in d]
    ref = torch.from_numpy(h.view(np.int64).copy()).cuda()
    ref[T // 2] += 1
    big = torch.zeros(1 << 30, dtype=torch.uint8, device="cuda")
    ar, ar2 = arena(256 << 20), arena((1 << 30) + (64 << 20))
    R = torch.zeros((2 * turns, n), dtype=torch.int64, device="cuda")
    S = torch.zeros((2 * turns, 1), dtype=torch.int64, device="cuda")
    bad = torch.full((turns, words), -1, dtype=torch.int64, device="cuda")
    lab = torch.full((turns, n), 9, dtype=torch.uint8, device="cuda")
    torch.cuda.synchronize()
    ctx, other = pcs.Context(ar, stream=side), pcs.Context(ar2, stream=load)
    plan = pcs.BufArray([pcs.flat(t, k) for t, k in zip(d, sizes)])
    dst = pcs.BufArray([pcs.flat(t, k) for t, k in zip(back, sizes)])
    for i in range(turns):
        other.delete(other.checkpoint([pcs.flat(big)], hash=True))
        ctx.fingerprint(plan, None, R[2 * i], S[2 * i])
        snap = ctx.checkpoint(plan, hash=True, roots=R[2 * i + 1], session_root=S[2 * i + 1])
        ctx.restore_verify(snap, dst, bad[i], lab[i])
        ctx.delete(snap)
        if i % 8 == 0:
            assert ctx.distance(ref, plan) == 1 / T
    torch.cuda.synchronize()
    assert (R.cpu().numpy().view(np.uint64) == r).all() and (S.cpu().numpy().view(np.uint64) == s).all()
    assert not bad.any() and not lab.any()
    assert all(np.array_equal(host(t)[:k], b) for t, k, b in zip(back, sizes, bufs))
    ctx.close()
    other.close()
