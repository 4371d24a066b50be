"""Entry moves of a bank shrink at the edges of their work items: every
granule size (16 to 1 bytes, what the entry size and the addresses allow),
entries laid end to end (at most 4096 granules) and cut into slices (more),
counts on both sides of a 1024-granule item, in place and out of place, parts
that move nothing between parts that do; and the multi-workgroup selection
where its buckets and ties are uneven.  Bytes and indices are compared with
the CPU oracle exactly."""
import numpy as np
import pytest
import torch

import oracle
from tests.gpu_util import arena, dev, host, log

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pcs():
    import paper_2607_21686_amd as P
    return P


# entry bytes of the parts, entries, kept
CASES = [
    ([1], 5000, 1023), ([1], 5000, 1025), ([2], 3000, 1024), ([28], 513, 146), ([28], 513, 147),
    ([24], 700, 341), ([24, 3, 1, 16, 2], 700, 342),
    ([4096 * 16], 9, 4), ([4097 * 16], 9, 4), ([4096], 9, 5), ([4097], 9, 5), ([4098 * 4, 7, 4096 * 8], 12, 7),
    ([199680, 28], 21, 3), ([16], 40000, 1), ([48, 6], 40000, 39999),
]


@pytest.mark.parametrize("inplace", [False, True])
@pytest.mark.parametrize("sizes,n,keep", CASES)
def test_moves_match_oracle(pcs, sizes, n, keep, inplace):
    rng = np.random.default_rng([n, keep, len(sizes)])
    parts = [rng.integers(0, 256, n * eb, dtype=np.uint8) for eb in sizes]
    scores = rng.standard_normal(n).astype(np.float32)
    want_kept, want = oracle.bank_shrink(list(zip(parts, sizes)), scores, keep)
    log("moves", sizes, n, keep, "in place" if inplace else "out of place")
    ctx = pcs.Context(arena(64 << 20))
    srcs = [dev(p) for p in parts]
    dsts = [None if inplace else torch.zeros(keep * eb, dtype=torch.uint8, device="cuda") for eb in sizes]
    kept = torch.zeros(keep, dtype=torch.int32, device="cuda")
    ctx.bank_shrink([(a, d, eb) for a, d, eb in zip(srcs, dsts, sizes)], torch.from_numpy(scores).cuda(), keep, kept)
    assert np.array_equal(host(kept).view(np.uint32), want_kept)
    for a, d, eb, w in zip(srcs, dsts, sizes, want):
        got = host(a if d is None else d)[:keep * eb]
        assert np.array_equal(got, np.asarray(w).reshape(-1)[:keep * eb])
    ctx.close()


@pytest.mark.parametrize("offset,eb", [(8, 24), (4, 24), (2, 24), (1, 24), (16, 1000)])
def test_moves_follow_the_source_alignment(pcs, offset, eb):
    """The granule is what the source address allows too."""
    n, keep = 900, 333
    rng = np.random.default_rng([offset, eb])
    bank = rng.integers(0, 256, n * eb, dtype=np.uint8)
    scores = rng.standard_normal(n).astype(np.float32)
    _, (want,) = oracle.bank_shrink([(bank, eb)], scores, keep)
    ctx = pcs.Context(arena(8 << 20))
    whole = torch.zeros(n * eb + offset, dtype=torch.uint8, device="cuda")
    src = whole[offset:]
    src.copy_(dev(bank))
    dst = torch.zeros(keep * eb, dtype=torch.uint8, device="cuda")
    ctx.bank_shrink([(src, dst, eb)], torch.from_numpy(scores).cuda(), keep)
    assert np.array_equal(host(dst), np.asarray(want).reshape(-1)[:keep * eb])
    ctx.close()


@pytest.mark.parametrize("kind", ["ties", "one bucket", "last bit", "both signs", "extremes"])
@pytest.mark.parametrize("n", [32769, 100003])
def test_large_selection_buckets(pcs, n, kind):
    """Five calls in a row on one context (the selection's words must come
    back to zero), keeping one, some, all but one and all entries."""
    rng = np.random.default_rng([n, len(kind)])
    s = {"ties": lambda: np.zeros(n, np.float32),
         "one bucket": lambda: (1.0 + rng.integers(0, 4096, n) * 2.0 ** -23).astype(np.float32),
         "last bit": lambda: rng.integers(0, 2, n).astype(np.uint32).view(np.float32),
         "both signs": lambda: rng.standard_normal(n).astype(np.float32),
         "extremes": lambda: rng.choice(np.array([np.nan, np.inf, -np.inf, -0.0, 0.0, 3e38], np.float32), n)}[kind]()
    ctx = pcs.Context(arena(8 << 20))
    sd = torch.from_numpy(s).cuda()
    for keep in (1, 7, n // 3, n - 1, n):
        want, _ = oracle.bank_shrink([], s, keep)
        kept = torch.zeros(keep, dtype=torch.int32, device="cuda")
        ctx.bank_shrink([], sd, keep, kept)
        assert np.array_equal(host(kept).view(np.uint32), want), (kind, keep)
    ctx.close()


@pytest.mark.parametrize("n", [3, 255, 257, 1023, 1024, 1025, 1027, 4095, 4097, 8192, 8193, 16384, 16385, 32767, 32768])
def test_one_workgroup_selection(pcs, n):
    """Both sides of the sizes where the workgroup has 256 and 1024 lanes and a lane
    holds 1, 2, 4 and 8 groups of scores, at every alignment of the first one, with many ties."""
    rng = np.random.default_rng(n)
    s = np.round(rng.standard_normal(n + 3) * 50).astype(np.float32)
    ctx = pcs.Context(arena(4 << 20))
    sd = torch.from_numpy(s).cuda()
    for off in range(4):
        view = sd[off:off + n]
        for keep in (1, n // 2, n - 1):
            want, _ = oracle.bank_shrink([], s[off:off + n], keep)
            kept = torch.zeros(keep, dtype=torch.int32, device="cuda")
            ctx.bank_shrink([], view, keep, kept)
            assert np.array_equal(host(kept).view(np.uint32), want), (off, keep)
    ctx.close()


@pytest.mark.parametrize("low_bits", [0, 9, 20], ids=["ties", "10-bit buckets", "21-bit buckets"])
@pytest.mark.parametrize("n", [1, 5, 512, 1024, 4097, 32768])
def test_selection_of_whole_buckets(pcs, n, low_bits):
    """Runs of up to 32 scores that share every key bit above `low_bits`, so
    that a run is kept whole, all but one, or with one more: the search ends
    after its first, second or last pass, and the ranges before and after the
    whole groups take part."""
    rng = np.random.default_rng([n, low_bits])
    run = min(32, n)
    top = (np.arange(n) // run).astype(np.uint32) << np.uint32(max(low_bits, 11))
    key = (np.uint32(0x3F800000) + top) | rng.integers(0, 1 << low_bits, n).astype(np.uint32)
    s = np.concatenate([np.zeros(3, np.float32), rng.permutation(key).astype(np.uint32).view(np.float32)])
    ctx = pcs.Context(arena(4 << 20))
    sd = torch.from_numpy(s).cuda()
    for off in range(4):
        m = min(n, s.size - off)
        for keep in sorted({min(max(k, 1), m) for k in (run - 1, run, run + 1, m // 2 // run * run, m)}):
            want, _ = oracle.bank_shrink([], s[off:off + m], keep)
            kept = torch.zeros(keep, dtype=torch.int32, device="cuda")
            ctx.bank_shrink([], sd[off:off + m], keep, kept)
            assert np.array_equal(host(kept).view(np.uint32), want), (off, keep)
    ctx.close()
