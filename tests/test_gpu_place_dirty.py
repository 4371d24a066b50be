"""Slot placement and dirty copy outside the two-launch incremental path (jobs
with device tables, more than 4096 groups, or an arena too small for the worst
case, where the host places the slots): stored bytes, stored counts and
restores against the CPU oracle, for dirty chunks that fill a few groups, lie
far apart, are every chunk, none, or the very first and last."""
import numpy as np
import pytest
import torch

import oracle
from tests.gpu_util import arena, dev, host, log, u64, zeros_u64

pytestmark = pytest.mark.gpu

C, GROUP = 4096, 64 * 4096
JOBS = {
    "65 groups, host placed": [64 * GROUP - 5, 3],
    "67 groups with empty buffers, host placed": [0, 65 * GROUP, 0, GROUP + 9, 0],
    "300 groups, host placed": [297 * GROUP + 5 * C + 77, 2 * GROUP + 1],
    "97 buffers, device tables": [(i * 37 % 90) * C + 1 + i for i in range(97)],
    "97 buffers, device tables, host placed": [(i * 53 % 70) * C + 9 for i in range(97)],
    "4100 groups": [4098 * GROUP + 7 * C, 100 * C + 3],
}
PATTERNS = {
    "few groups": lambda T: np.arange(T)[-(T // 40 + 1):],
    "far apart": lambda T: np.arange(0, T, 193),
    "every": lambda T: np.arange(T),
    "none": lambda T: np.arange(0),
    "first and last": lambda T: np.array(sorted({0, T - 1})),
    "every other group": lambda T: np.arange(T)[np.arange(T) // 64 % 2 == 0],
}


@pytest.fixture(scope="module")
def pcs():
    import paper_2607_21686_amd as P
    return P


@pytest.mark.parametrize("name", list(JOBS))
def test_place_dirty(pcs, name):
    sizes = JOBS[name]
    rng = np.random.default_rng(len(name))
    cur = [rng.integers(0, 256, size=k, dtype=np.uint8) for k in sizes]
    cpb = [oracle.chunk_count(k) for k in sizes]
    where = [(b, i) for b, k in enumerate(cpb) for i in range(k)]
    T, state = len(where), sum(cpb) * C
    tight = name.endswith("host placed")
    ctx = pcs.Context(arena((2 if tight else 3) * state + (64 << 20)))
    d = [dev(b) if b.size else torch.zeros(16, dtype=torch.uint8, device="cuda") for b in cur]
    descs = lambda ts: [pcs.flat(t, k) for t, k in zip(ts, sizes)]
    st = oracle.Store()
    par, opar = ctx.checkpoint(descs(d), hash=True), st.checkpoint(cur)
    if tight:  # fill the arena up to the worst case: with its own metadata the call no longer fits it
        fill = ctx.arena_stats()["largest_free"] - state
        ctx.checkpoint([pcs.flat(torch.zeros(fill, dtype=torch.uint8, device="cuda"))])
        assert ctx.arena_stats()["largest_free"] <= state
    for label, pick in PATTERNS.items():
        log("place dirty", name, label)
        now = [b.copy() for b in cur]
        for g in pick(T):
            b, i = where[g]
            now[b][i * C] ^= 0x41
        for t, b in zip(d, now):
            if b.size:
                t.copy_(torch.from_numpy(b))
        H, R, S = zeros_u64(T), zeros_u64(len(sizes)), zeros_u64(1)
        if tight and label == "every":
            with pytest.raises(pcs.PcsError):
                ctx.checkpoint(descs(d), parent=par, chunk_hashes=H, roots=R, session_root=S)
            continue
        snap = ctx.checkpoint(descs(d), parent=par, chunk_hashes=H, roots=R, session_root=S)
        osnap = st.checkpoint(now, opar)
        h, r, s = oracle.fingerprint(now)
        assert np.array_equal(u64(H)[:T], h) and np.array_equal(u64(R), r) and int(u64(S)[0]) == s
        want = st.payload(osnap)
        assert ctx.info(snap)["dirty_chunks"] == len(pick(T)) and ctx.info(snap)["stored_bytes"] == want.size
        pay = torch.empty(max(1, want.size), dtype=torch.uint8, device="cuda")
        ctx.payload(snap, pay)
        assert np.array_equal(host(pay)[:want.size], want)
        back = [torch.zeros_like(t) for t in d]
        ctx.restore(snap, descs(back))
        assert all(np.array_equal(host(t)[:k], b) for t, k, b in zip(back, sizes, now))
        ctx.delete(snap)
    ctx.close()
