// Host-only test of the address arithmetic the kernels use (pcs_layout.h:
// locate, chunk_loc) against the piece list of the same descriptor
// (pcs_host.h: describe), and of the Merkle-item and move-item rules.
#include <cinttypes>
#include <cstdio>
#include <cstdlib>
#include <random>

#include "../../paper_2607_21686_amd/csrc/pcs_host.h"

using namespace pcs;

#define CHECK(x)                                                        \
    do {                                                                \
        if (!(x)) {                                                     \
            printf("%s:%d: %s\n", __FILE__, __LINE__, #x);              \
            exit(1);                                                    \
        }                                                               \
    } while (0)

static pcs_buf ring(uint64_t ptr, uint64_t outer, uint64_t cap, uint64_t row, uint64_t head, uint64_t window,
                    uint64_t stride)
{
    pcs_buf b{};
    b.ptr = ptr;
    b.kind = PCS_RING;
    b.row_bytes = row;
    b.capacity = cap;
    b.head = head;
    b.window = window;
    b.outer = outer;
    b.outer_stride = stride;
    return b;
}

// Every byte of every piece's ends, and every chunk's description.
static void check_against_runs(const pcs_buf &b)
{
    Layout lay;
    std::vector<Run> rs;
    std::string why;
    CHECK(describe(b, 0, &lay, &rs, &why) == PCS_OK);
    CHECK(lay.geom.nbytes == lay.nbytes);
    CHECK(lay.nruns == rs.size());
    if (!lay.nbytes) return;
    for (size_t k = 0; k < rs.size(); ++k) {
        const uint64_t end = k + 1 < rs.size() ? rs[k + 1].lstart : lay.nbytes;
        for (uint64_t L : {rs[k].lstart, rs[k].lstart + 1, (rs[k].lstart + end) / 2, end - 1}) {
            if (L >= end) continue;
            const Where w = locate(lay.geom, L);
            CHECK(w.addr == rs[k].addr + (L - rs[k].lstart));
            CHECK(w.left == end - L);
        }
    }
    size_t k = 0;
    for (uint64_t c = 0; c < lay.nchunks; ++c) {
        const ChunkLoc l = chunk_loc(lay.geom, c);
        const uint64_t cb = c * kChunk;
        CHECK(l.len == std::min<uint64_t>(kChunk, lay.nbytes - cb));
        while (k + 1 < rs.size() && rs[k + 1].lstart <= cb) ++k;
        const auto end = [&](size_t j) { return j + 1 < rs.size() ? rs[j + 1].lstart : lay.nbytes; };
        if (cb + l.len <= end(k)) {
            CHECK(l.split == l.len && l.a1 == rs[k].addr + (cb - rs[k].lstart));
        } else if (cb + l.len <= end(k + 1)) {
            CHECK(l.a1 == rs[k].addr + (cb - rs[k].lstart));
            CHECK(l.split == end(k) - cb);
            CHECK(l.a2 + l.split == rs[k + 1].addr);
        } else {
            CHECK(l.a1 == 0);
        }
    }
}

static void test_rings(uint64_t seed)
{
    std::mt19937_64 rng(seed);
    for (int it = 0; it < 6000; ++it) {
        const uint64_t row = 16 * (1 + rng() % (it % 3 ? 20 : 400));
        const uint64_t cap = 1 + rng() % 60, head = rng() % cap, window = rng() % (cap + 1);
        const uint64_t outer = rng() % 40;
        const uint64_t stride = cap * row + 16 * (rng() % 3 == 0 ? 0 : rng() % 5);
        check_against_runs(ring(16 * (1 + rng() % (1u << 20)), outer, cap, row, head, window, stride));
    }
    // Full windows, one-row windows, one ring.
    for (uint64_t outer : {1, 2, 7})
        for (uint64_t window : {1, 63, 64})
            for (uint64_t head : {0, 1, 63}) check_against_runs(ring(4096, outer, 64, 48, head, window, 64 * 48));
}

// Rings too many or too large to list: the address from 128-bit arithmetic.
static void test_large(uint64_t seed)
{
    std::mt19937_64 rng(seed);
    for (int it = 0; it < 200000; ++it) {
        const uint64_t outer = 1 + rng() % (1ULL << (1 + rng() % 30));
        const uint64_t row = 16 * (1 + rng() % 4096), cap = 1 + rng() % (1ULL << (rng() % 20));
        const uint64_t head = rng() % cap, window = 1 + rng() % cap, stride = cap * row + 16 * (rng() % 3);
        unsigned __int128 extent = (unsigned __int128)outer * stride;
        if (extent >> 57) continue;
        const pcs_buf b = ring(16 * (1 + rng() % (1u << 20)), outer, cap, row, head, window, stride);
        Layout lay;
        std::string why;
        CHECK(describe(b, 0, &lay, nullptr, &why) == PCS_OK);
        for (int q = 0; q < 6; ++q) {
            const uint64_t o = q == 0 ? outer - 1 : q == 1 ? 0 : rng() % outer;
            const uint64_t t = q % 3 == 0 ? 0 : q % 3 == 1 ? window - 1 : rng() % window;
            const uint64_t x = rng() % 2 ? row - 1 : 0;
            const uint64_t L = (o * window + t) * row + x;
            CHECK(locate(lay.geom, L).addr == b.ptr + o * stride + ((head + t) % cap) * row + x);
        }
    }
}

// A part's work items cover its granules once: slices of entries, or slices
// of all entries laid end to end.
static void test_move_items()
{
    for (uint64_t gpe : {1ull, 7ull, 1023ull, 1024ull, 1025ull, 4095ull, 4096ull, 4097ull, 12480ull, 1ull << 33})
        for (uint64_t keep : {1ull, 3ull, 146ull, 1024ull, 50000ull}) {
            const uint64_t spe = move_slices(gpe), items = move_items(keep, gpe);
            if (gpe > kMoveStreamGranules) {
                CHECK(spe * kMoveItem >= gpe && (spe - 1) * kMoveItem < gpe && items == keep * spe);
            } else {
                CHECK(spe == 0 && items * kMoveItem >= keep * gpe && (items - 1) * kMoveItem < keep * gpe);
            }
        }
}

// A promote-odd tree over v, level by level.
static uint64_t node(uint64_t l, uint64_t r) { return (l ^ 0x9E3779B97F4A7C15ull) * 3 + (r + 1) * 0xC2B2AE3D27D4EB4Full; }
static uint64_t tree(std::vector<uint64_t> v)
{
    while (v.size() > 1) {
        for (size_t i = 0; 2 * i < v.size(); ++i) v[i] = 2 * i + 1 < v.size() ? node(v[2 * i], v[2 * i + 1]) : v[2 * i];
        v.resize((v.size() + 1) / 2);
    }
    return v[0];
}

// A list reduced item by item, as the argument-table kernels do it (the first
// level of long lists apart, more than 64 items in blocks of their own), has
// the root of the whole tree.
static std::vector<uint64_t> by_items(const std::vector<uint64_t> &v)
{
    std::vector<uint64_t> part;
    for (uint32_t k = 0; k < merkle_items(v.size()); ++k) {
        const auto at = v.begin() + 64ull * k;
        part.push_back(tree(std::vector<uint64_t>(at, at + merkle_item_values(v.size(), k))));
    }
    return part;
}
static void test_merkle_items()
{
    for (uint64_t blocks : {1ull, 2ull, 63ull, 64ull, 65ull, 4095ull, 4096ull, 4097ull, 262144ull})
        for (int64_t d : {-65, -63, -1, 0, 1, 62})
            for (uint32_t tiles : {1u, kSmallTiles}) {
                const uint64_t values = 64 * blocks + (uint64_t)d;
                if (values == 0 || values >> 40 || values > 1ull << 24) continue;
                const uint64_t per = kGroupChunks / tiles;
                CHECK(merkle_values(values * per, tiles, false) == values);
                CHECK(merkle_values(values * per - per + 1, tiles, false) == values);
                std::vector<uint64_t> v(values);
                for (uint64_t i = 0; i < values; ++i) v[i] = i * 0xD1B54A32D192ED03ull + blocks;
                const uint64_t want = tree(v);
                for (bool pre : {false, true}) {
                    std::vector<uint64_t> list = v;
                    if (pre) list = by_items(v);
                    CHECK(list.size() == merkle_values(values * per, tiles, pre));
                    std::vector<uint64_t> part = by_items(list);
                    if (part.size() > 4096) continue;  // beyond one workgroup: such a list has its first level done
                    if (part.size() > 64) part = by_items(part);
                    CHECK(part.size() <= 64);
                    CHECK(tree(part) == want);
                }
            }
}

int main()
{
    test_rings(1);
    test_large(2);
    test_move_items();
    test_merkle_items();
    printf("ok\n");
    return 0;
}
