// pcs_layout.h -- descriptors and constants shared by the host runtime and
// the gfx950 kernels of libpcs: plain structs with fixed layouts, no HIP.
// Internal to the library (not part of the C ABI).
#pragma once

#include <stddef.h>
#include <stdint.h>

namespace pcs {

constexpr uint64_t kChunk = 4096;       // fingerprint and snapshot granule (bytes)
constexpr uint32_t kGroupChunks = 64;   // chunks per work group and per bitmap word

// A maximal physically contiguous piece of a buffer's logical byte stream:
// logical bytes [lstart, next run's lstart) live at addr onwards.  A flat
// buffer is one run; a ring window is at most two runs per ring (before and
// after the wrap), merged where physically adjacent.  (Kernels compute these
// pieces, see Geom; the list is what that is checked against.)
struct Run {
    uint64_t lstart;
    uint64_t addr;
};

constexpr uint64_t chunks_of(uint64_t nbytes) { return nbytes / kChunk + (nbytes % kChunk != 0); }

// Where a buffer's logical bytes lie.  Flat (win == 0): at addr onwards.
// Ring: `win` logical bytes per ring, ring o at addr + o * stride; the first
// `first` bytes of a ring's window start `head` bytes into it, the rest at
// its beginning.  inv_win = 1 / win.
struct Geom {
    uint64_t addr;
    uint64_t nbytes;
    uint64_t win, first, head, stride;
    double inv_win;
};
// Physical address of logical byte L < nbytes, and the bytes from L to the
// end of its physically contiguous piece.
struct Where {
    uint64_t addr, left;
};
// The ring number comes from a multiplication by inv_win: it is below 2^30
// (a descriptor's limit on rings), so the product is off by less than 2^-20
// and its floor by at most one, which the remainder shows.  Kernels compute
// addresses this way instead of searching a table of pieces: a search costs a
// dependent load a step, and a table of many rings does not fit the kernel
// arguments.
struct RingAt {
    uint64_t base, r;  // the ring's address; the byte's place in its window
};
constexpr RingAt ring_at(const Geom &g, uint64_t L)
{
    uint64_t o = (uint64_t)((double)L * g.inv_win);
    int64_t rem = (int64_t)(L - o * g.win);
    if (rem < 0) {
        --o;
        rem += (int64_t)g.win;
    } else if ((uint64_t)rem >= g.win) {
        ++o;
        rem -= (int64_t)g.win;
    }
    return RingAt{g.addr + o * g.stride, (uint64_t)rem};
}
constexpr Where locate(const Geom &g, uint64_t L)
{
    if (g.win == 0) return Where{g.addr + L, g.nbytes - L};
    const RingAt p = ring_at(g, L);
    return p.r < g.first ? Where{p.base + g.head + p.r, g.first - p.r} : Where{p.base + (p.r - g.first), g.win - p.r};
}

// Where one chunk's bytes lie: byte x (x < len) is at (x < split ? a1 : a2)
// + x when the chunk spans at most two pieces (it straddles a ring's wrap, or
// the end of one ring's window and the start of the next); a1 = 0 marks a
// chunk of more pieces (rows shorter than a chunk), located per access.
// Piece boundaries are 16-byte aligned, so no 16-byte granule crosses one.
// slot: the chunk's 4096-byte snapshot slot (pack, restore; the kernels' own).
struct ChunkLoc {
    uint64_t a1, a2, slot;
    uint32_t split, len;
};
constexpr ChunkLoc chunk_loc(const Geom &g, uint64_t chunk)
{
    const uint64_t cb = chunk * kChunk, rest = g.nbytes - cb;
    ChunkLoc l{0, 0, 0, 0, (uint32_t)(rest < kChunk ? rest : kChunk)};
    if (g.win == 0) {
        l.a1 = l.a2 = g.addr + cb;
        l.split = l.len;
        return l;
    }
    const RingAt p = ring_at(g, cb);
    const bool before = p.r < g.first;  // in the part of the window before the wrap
    const uint64_t a1 = before ? p.base + g.head + p.r : p.base + (p.r - g.first);
    const uint64_t left = before ? g.first - p.r : g.win - p.r;
    if (l.len <= left) {
        l.a1 = l.a2 = a1;
        l.split = l.len;
        return l;
    }
    // The buffer goes on after this piece: past the wrap, or in the next ring
    // (derived, not located anew, which every lane of a tile would wait for).
    const bool wraps = before && g.first < g.win;
    const uint64_t next = wraps ? p.base : p.base + g.stride + g.head, left2 = wraps ? g.win - g.first : g.first;
    if (l.len - left <= left2) {
        l.a1 = a1;
        l.split = (uint32_t)left;
        l.a2 = next - left;  // byte `split` of the chunk is the second piece's first byte
    }
    return l;
}

// One buffer of a job.  Every kernel grids over 64-chunk groups of one
// buffer; group_begin is this buffer's first group in the job.
struct JobBuf {
    Geom g;
    uint32_t chunk_begin;     // first chunk of this buffer in job-wide chunk order
    uint32_t group_begin;     // first 64-chunk group of this buffer in the job
    uint64_t payload;         // device address of chunk 0's 4096-byte slot (pack dst, restore src)
    uint64_t manifest;        // restore: device address of uint64 arena offsets, one per chunk
                              // incremental pack: where this buffer's new manifest entries go
    uint64_t hash_dst[2];     // device addresses of chunk 0's fingerprint outputs (0 = none)
    uint64_t root_dst[2];     // device addresses of the root outputs (0 = none)
    uint64_t parent_hash;     // incremental: device address of the parent's chunk-0 fingerprint;
                              // verified restore: of the snapshot's stored chunk-0 fingerprint
    uint64_t parent_chunks;   // incremental: chunks the parent held for this buffer
    uint64_t parent_manifest; // incremental: parent's manifest entries (0 if the parent is full)
    uint64_t parent_slot0;    // incremental, full parent: arena offset of the parent's chunk-0 slot
    constexpr uint64_t nchunks() const { return chunks_of(g.nbytes); }
};

// A list reduced by the Merkle kernel: values [begin, begin + count) of the
// input array; the root goes to dst[0] / dst[1] (0 = none) and scratch[idx].
struct MerkleList {
    uint64_t begin;
    uint64_t count;
    uint64_t dst[2];
};

// Where a launch finds its buffer table.
//   DevTables: in device memory (staged per call), with a group map that
//              gives each group its buffer; any job.
//   ArgTables: carried in the kernel arguments themselves (nothing staged);
//              jobs of at most kArgBufs buffers, kArgRings of them rings, and
//              one session where fingerprints are written.  A workgroup reads
//              the whole table with a few vector loads, one round trip to
//              memory, and finds its buffer with a ballot.
constexpr uint32_t kArgBufs = 96, kArgRings = 16;
// Small jobs (at most kSmallJobGroups groups) are cut into kSmallTiles
// sub-tiles per group, so that a few groups still spread over many CUs.
// Fingerprint and pack tiles then write one Merkle node per sub-tile (an
// aligned 8-chunk subtree, which the Merkle lists reduce like group nodes).
// Smaller tiles do not pay: a tile's fingerprint is bounded by one chunk's
// XXH64 chain (128 dependent rounds per accumulator), which 8-chunk tiles
// overlap with their loads.
constexpr uint64_t kSmallJobGroups = 128;
constexpr uint32_t kSmallTiles = 8;
inline uint32_t tile_split(uint64_t ngroups) { return ngroups <= kSmallJobGroups ? kSmallTiles : 1; }

// Tile order of the tile kernels: the tile workgroup b of a launch of nb
// workgroups takes.  The dispatcher deals a launch's workgroups to the eight
// XCDs in turn (workgroup b runs on XCD b mod 8), so the tiles are handed
// out XCD by XCD:
//   - below kXcdBlockJobs tiles: XCD x works through the x-th contiguous
//     eighth of the job in order, entered at a point staggered by x/8 of its
//     length (wrapping), so that the eight streams do not walk over the same
//     memory channels in step;
//   - from kXcdBlockJobs tiles: blocks of kXcdBlock consecutive tiles are
//     dealt to the XCDs in turn, so every XCD streams through every part of
//     the job and none is left with a stretch of memory that happens to be
//     slower; the tail of fewer than eight blocks keeps the launch order.
// A bijection of [0, nb).  (constexpr: callable from host and device code.)
constexpr uint32_t kXcds = 8, kXcdBlock = 512, kXcdBlockJobs = 16384;
constexpr uint32_t xcd_tile_of(uint32_t b, uint32_t nb)
{
    const uint32_t x = b % kXcds, i = b / kXcds;
    if (nb >= kXcdBlockJobs) {
        const uint32_t full = nb / (kXcds * kXcdBlock);  // whole rounds of blocks
        if (b >= full * kXcds * kXcdBlock) return b;
        return ((i / kXcdBlock) * kXcds + x) * kXcdBlock + i % kXcdBlock;
    }
    const uint32_t per = nb / kXcds, rem = nb % kXcds;
    const uint32_t n = per + (x < rem ? 1u : 0u);  // tiles of XCD x (>= 1 when workgroup b exists)
    return x * per + (x < rem ? x : rem) + (i + x * (n / kXcds)) % n;
}

// Words of the arena's first unit, which the library keeps (byte offsets).
// Bump: two bump words of incremental slot placement and a call's payload
// top.  Select: tickets and the first histogram of a large bank's selection,
// cleared by the context's first call that takes tickets and zero between calls
// from then on (the launch that uses them clears them again).
constexpr uint64_t kUnitBump = 0;
constexpr uint64_t kUnitSelect = 64;
constexpr uint32_t kSelectTickets = 4, kSelectFirstBuckets = 256;
constexpr uint64_t kUnitSelectBytes = 4 * (kSelectTickets + kSelectFirstBuckets);
// Tail: tickets of the tile launches that finish their own job (TailWords),
// the same.
constexpr uint64_t kUnitTail = 2048 - 8 * 64;

// Tickets of a small job whose 8-chunk tiles finish it (all zero between
// launches): one per group, 16 bytes apart, one per buffer, one for the job.
struct TailWords {
    uint64_t job;
    uint32_t pad[30];
    uint32_t buf[96];
    uint32_t group[kSmallJobGroups][4];
};
static_assert(kUnitTail + sizeof(TailWords) <= 4096 && kUnitTail % 128 == 0, "the tickets lie in the arena's first unit");

struct DevTables {
    const JobBuf *bufs;
    const uint32_t *map;  // each group's buffer
    uint32_t nbuf;
    uint32_t pad;
};

// JobBuf packed for the kernel arguments.  What a job lays out linearly
// (fingerprints, manifests, roots) is a base plus an index; aux depends on
// what the job does:
//   pack:            device address of chunk 0's slot
//   restore, verify: the same, or the address of the buffer's manifest
//                    entries with kAuxManifest set
//   diff:            parent's first chunk | parent's chunks << 32
struct ArgBuf {
    uint64_t addr;
    uint64_t nbytes;
    uint32_t chunk_begin, group_begin;
    uint64_t aux;
};
constexpr uint64_t kAuxManifest = 1;
struct ArgRing {
    uint64_t win, first, head, stride;
    double inv_win;
};
struct ArgTables {
    uint32_t nbuf, nring;
    uint64_t hash[2];          // chunk fingerprints of chunk i: hash + 8 i (0 = none)
    uint64_t root[2];          // root of buffer b: root + 8 b (0 = none)
    uint64_t sroot[2];         // session root (0 = none)
    uint64_t manifest;         // diff: new manifest entry of chunk i: manifest + 8 i
    uint64_t parent_hash;      // diff: parent's chunk i; verify: stored fingerprint of chunk i
    uint64_t parent_manifest;  // diff: parent's manifest (0 if the parent is full)
    uint64_t parent_slot0;     // diff, full parent: arena offset of its chunk 0's slot
    uint64_t tail;             // sub-tiles that finish their job: device address of the TailWords (0: they do not)
    uint64_t tail_scratch;     // roots: a value per group, then one per buffer
    uint64_t tail_count;       // diff: where the number of set mask bits goes (mapped host memory)
    uint64_t tail_labels;      // verify: a byte per buffer
    uint8_t ring_buf[kArgRings];  // the buffer of each ring
    ArgRing rings[kArgRings];
    ArgBuf bufs[kArgBufs];
};
// Kernel arguments are limited to 4 KiB; a launch passes one ArgTables and at
// most a few pointers and sizes besides.
static_assert(kArgBufs <= 256, "a buffer number fits in ring_buf");
static_assert(sizeof(ArgTables) + 224 <= 4096, "argument tables must fit in the kernel arguments");

// The Merkle list of a buffer of a job in the argument tables: one value per
// tile (`tiles` of them to a group), or, once its aligned blocks of 64 are
// reduced (pre), one per block; and its items, the blocks of 64 a wavefront
// reduces at once.
constexpr uint64_t merkle_values(uint64_t nchunks, uint32_t tiles, bool pre)
{
    const uint64_t per = kGroupChunks / tiles, n = nchunks / per + (nchunks % per != 0);
    return pre ? n / 64 + (n % 64 != 0) : n;
}
constexpr uint32_t merkle_items(uint64_t values) { return (uint32_t)(values / 64 + (values % 64 != 0)); }
constexpr uint32_t merkle_item_values(uint64_t values, uint32_t item)
{
    const uint64_t left = values - 64ull * item;
    return left < 64 ? (uint32_t)left : 64;
}

// Buffer lists of a Merkle launch that hold more than kMerkleLdsValues
// values (a buffer of more than 1 GiB): when at most kLongLists of them, a
// grid-wide pass reduces their aligned 64-value blocks first,
// one wavefront each, into the list's first scratch level (at the list's own
// offset), and the per-list reduction starts from there.  Block b of the
// pass belongs to list j when block_begin[j] <= b < block_begin[j + 1].
constexpr uint64_t kMerkleLdsValues = 4096;
constexpr uint32_t kLongLists = 4;  // more long lists reduce in parallel, one workgroup each, anyway
struct LongLists {
    uint32_t n;
    uint32_t pad;
    uint64_t begin[kLongLists];
    uint64_t count[kLongLists];
    uint64_t block_begin[kLongLists + 1];
};

// The entry moves of a bank shrink, every part in one launch.  Part p moves
// the kept entries of entry_bytes eb from src to dst (stage: in place, the
// staging area for entries the compaction would overwrite before reading
// them; 0 out of place) in granules of 1 << gl bytes (16 to 1, what the
// addresses and eb allow).  Its work items, kMoveItem granules each, are
// [item_begin[p], item_begin[p + 1]): move_slices() slices of every kept
// entry, or, for entries of at most kMoveStreamGranules granules, slices of
// all kept entries laid end to end, so that a slice holds several entries
// and no lane idles on a short one.
constexpr uint32_t kMoveLanes = 256, kMoveUnroll = 4;
constexpr uint32_t kMoveItem = kMoveLanes * kMoveUnroll;
constexpr uint64_t kMoveStreamGranules = 4 * kMoveItem;
struct ShrinkPart {
    uint64_t src, dst, stage;
    uint64_t eb;
    uint32_t gl, pad;
};
// Slices per entry (0: the part's entries are laid end to end).
constexpr uint64_t move_slices(uint64_t gpe)
{
    return gpe <= kMoveStreamGranules ? 0 : gpe / kMoveItem + (gpe % kMoveItem != 0);
}
// Work items of a part that moves `keep` entries of gpe granules.
constexpr uint64_t move_items(uint64_t keep, uint64_t gpe)
{
    const uint64_t spe = move_slices(gpe), all = keep * gpe;
    return spe ? keep * spe : all / kMoveItem + (all % kMoveItem != 0);
}
constexpr uint32_t kShrinkParts = 64;
struct ShrinkParts {
    uint32_t n;
    uint32_t pad;
    uint64_t items;
    uint64_t item_begin[kShrinkParts];  // parts past n begin at `items`
    ShrinkPart p[kShrinkParts];
};
static_assert(sizeof(ShrinkParts) + 64 <= 4096, "shrink parts must fit in the kernel arguments");

}  // namespace pcs
