// pcs_kernels.hip -- gfx950 (CDNA4) kernels of libpcs: chunked XXH64 with a
// Merkle combine, fused pack + fingerprint, scatter restore, incremental
// dirty-chunk packing and cross-replay classification.
//
// Work decomposition shared by every kernel: a job is a table of buffers,
// each cut into 4096-byte chunks, and the chunks of one buffer into aligned
// groups of 64.  One workgroup handles one group (in a job of at most 128
// groups, an eighth of one); it finds its buffer through a group-to-buffer
// map (written by k_stage with the tables) when the tables live in device
// memory, or with one vector load and a ballot when a job carries its tables
// in the kernel arguments (nothing staged).  Where a ring buffer's bytes lie
// follows from its shape, head and row by arithmetic; no table of runs is
// stored.  Groups never straddle buffers, so a group's 64 chunk fingerprints reduce to one Merkle node
// inside the workgroup (a promote-odd tree over n leaves splits into aligned
// 64-leaf subtrees), and a group is exactly one word of the classification
// bitmap.
//
// Memory traffic is 16-byte vector loads and stores throughout.  Nothing
// here is a contraction, so no MFMA is used; the hash is 64-bit integer
// multiply work on the vector ALU.
#include <hip/hip_ext.h>

#include <algorithm>
#include <type_traits>

#include "pcs_device.h"

// Device scratch of the allocation-free entry point (pcs_fingerprint_noalloc):
// descriptor tables, the group map and the Merkle levels of one call.  Every
// GPU the library runs on holds its own copy until the process ends.  In host
// code this name is a host-side stand-in, never a device address: host code
// uses only the per-device address that static_scratch_address returns.
static __device__ __align__(256) uint8_t scratch[pcs::kStaticScratchBytes];

namespace pcs {

hipError_t static_scratch_address(uint64_t *addr)
{
    void *p = nullptr;
    const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    *addr = e == hipSuccess ? (uint64_t)p : 0;
    return e;
}

namespace {

// Timing events for the next kernel launch, set by the runtime around one
// launcher call while dispatch timing is on: that launch stamps `start` when
// its kernel begins and `stop` when it ends (the dispatch's own timestamps,
// so queueing and launch overhead are not counted).  Other launches take the
// plain launch path.
thread_local hipEvent_t t_start = nullptr, t_stop = nullptr;
thread_local bool t_used = false;

template <class K, class... Args>
void run_kernel(K kernel, dim3 grid, dim3 block, hipStream_t s, Args... args)
{
    if (!t_start) {
        hipLaunchKernelGGL(kernel, grid, block, 0, s, args...);
        return;
    }
    hipExtLaunchKernelGGL(kernel, grid, block, 0, s, t_start, t_stop, 0, args...);
    t_start = t_stop = nullptr;
    t_used = true;
}

// XXH64 primes (xxHash specification).
constexpr uint64_t P1 = 0x9E3779B185EBCA87ULL;
constexpr uint64_t P2 = 0xC2B2AE3D27D4EB4FULL;
constexpr uint64_t P3 = 0x165667B19E3779F9ULL;
constexpr uint64_t P4 = 0x85EBCA77C2B2AE63ULL;
constexpr uint64_t P5 = 0x27D4EB2F165667C5ULL;

__device__ __forceinline__ uint64_t umin(uint64_t a, uint64_t b) { return a < b ? a : b; }

// 64-bit rotate left by 0 < r < 32: two v_alignbit_b32.
__device__ __forceinline__ uint64_t rotl(uint64_t x, int r)
{
    const uint32_t lo = (uint32_t)x, hi = (uint32_t)(x >> 32);
    const uint32_t nhi = __builtin_amdgcn_alignbit(hi, lo, 32 - r);
    const uint32_t nlo = __builtin_amdgcn_alignbit(lo, hi, 32 - r);
    return ((uint64_t)nhi << 32) | nlo;
}

// Accumulator step: add lane * P2, rotate left 31, multiply by P1.
__device__ __forceinline__ uint64_t xround(uint64_t acc, uint64_t lane)
{
    acc += lane * P2;
    acc = rotl(acc, 31);
    return acc * P1;
}

// The same with lane * P2 already formed.
__device__ __forceinline__ uint64_t xstep(uint64_t acc, uint64_t scaled)
{
    return rotl(acc + scaled, 31) * P1;
}

__device__ __forceinline__ uint64_t avalanche(uint64_t h)
{
    h ^= h >> 33;
    h *= P2;
    h ^= h >> 29;
    h *= P3;
    h ^= h >> 32;
    return h;
}

// XXH64 (seed 0) of the empty input: the short-input start value, length 0,
// no tail, avalanche.
__device__ __forceinline__ uint64_t empty_hash() { return avalanche(P5); }

// XXH64 (seed 0) of the 16 bytes le64(l) || le64(r): the Merkle node.
__device__ __forceinline__ uint64_t node_hash(uint64_t l, uint64_t r)
{
    uint64_t acc = P5 + 16;
    acc ^= xround(0, l);
    acc = rotl(acc, 27) * P1 + P4;
    acc ^= xround(0, r);
    acc = rotl(acc, 27) * P1 + P4;
    return avalanche(acc);
}

// A 64-bit DPP move (CTL below 0x100: a permutation of each lane quad, two
// bits per lane; 0x100 + n: from n lanes above within a row of 16).
template <int CTL>
__device__ __forceinline__ uint64_t dpp64(uint64_t v)
{
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)v, CTL, 0xF, 0xF, false);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(v >> 32), CTL, 0xF, 0xF, false);
    return ((uint64_t)hi << 32) | lo;
}

__device__ __forceinline__ uint32_t lane_word(uint32_t v, uint32_t lane)
{
    return (uint32_t)__builtin_amdgcn_readlane((int)v, (int)lane);
}
__device__ __forceinline__ uint64_t lane_word(uint64_t v, uint32_t lane)
{
    return ((uint64_t)lane_word((uint32_t)(v >> 32), lane) << 32) | lane_word((uint32_t)v, lane);
}

// The value 16 lanes above (S = 16: in lanes 0-15 and 32-47) or 32 lanes
// above (S = 32: in lanes 0-31).
template <int S>
__device__ __forceinline__ uint64_t row_swap(uint64_t v)
{
    const uint32_t lo = (uint32_t)v, hi = (uint32_t)(v >> 32);
    if constexpr (S == 16) {
        const auto a = __builtin_amdgcn_permlane16_swap(lo, lo, false, false);
        const auto b = __builtin_amdgcn_permlane16_swap(hi, hi, false, false);
        return ((uint64_t)b[1] << 32) | a[1];
    } else {
        const auto a = __builtin_amdgcn_permlane32_swap(lo, lo, false, false);
        const auto b = __builtin_amdgcn_permlane32_swap(hi, hi, false, false);
        return ((uint64_t)b[1] << 32) | a[1];
    }
}

// The value S lanes above (S a power of two), in the lanes l with
// l mod 2 S < S; other lanes get something else.  DPP moves and row swaps: none
// waits on the LDS path as a shuffle does.
template <int S>
__device__ __forceinline__ uint64_t from_above(uint64_t v)
{
    if constexpr (S == 1) return dpp64<0xF5>(v);
    else if constexpr (S == 2) return dpp64<0xAA>(v);
    else if constexpr (S == 4) return dpp64<0x104>(v);
    else if constexpr (S == 8) return dpp64<0x108>(v);
    else return row_swap<S>(v);
}

// Promote-odd Merkle reduction of m values of one wavefront (m wave-uniform,
// at most 2^LEVELS): value i lies in lane S * i.  A level's node stays in the
// lane of its left child, so nothing is compacted; the root is valid in
// lane 0.
template <int S, int LEVELS>
__device__ __forceinline__ uint64_t wave_merkle(uint64_t v, uint32_t m)
{
    if constexpr (LEVELS > 0) {
        if (m <= 1) return v;
        const uint64_t right = from_above<S>(v);
        const uint32_t i = (threadIdx.x & 63) / S;
        if (i + 1 < m) v = node_hash(v, right);  // lanes of odd i compute a value nothing reads
        return wave_merkle<2 * S, LEVELS - 1>(v, (m + 1) / 2);
    }
    return v;
}

// Four such reductions at once: value i of list q (n[q] of them, at most 64)
// is lane i of v[q]; the root of list q ends in lane q.  A level halves the
// lanes a list needs, so the first two levels interleave the lists (0 and 1
// in even and odd lanes, then all four) and the rest run on all of them: 7
// nodes per lane where four reductions one after another take 24.  (n by
// value: a choice between array elements would put the array in memory.)
__device__ __forceinline__ uint64_t wave_merkle4(const uint64_t (&v)[4], uint32_t n0, uint32_t n1, uint32_t n2,
                                                 uint32_t n3)
{
    const uint32_t lane = threadIdx.x & 63;
    const uint32_t even_n = (lane & 2) ? n2 : n0, odd_n = (lane & 2) ? n3 : n1;
    uint64_t w[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const uint64_t a = v[2 * h], b = v[2 * h + 1];
        const uint64_t below = dpp64<0xA0>(b), above = dpp64<0xF5>(a);  // (moved before any lane branches)
        const bool odd = lane & 1;
        const uint64_t left = odd ? below : a, right = odd ? b : above;
        w[h] = (lane | 1) < (odd ? (h ? n3 : n1) : (h ? n2 : n0)) ? node_hash(left, right) : left;
    }
    const uint64_t below = dpp64<0x44>(w[1]), above = dpp64<0xEE>(w[0]);
    const bool second = lane & 2;
    const uint64_t left = second ? below : w[0], right = second ? w[1] : above;
    uint32_t m = (((lane & 1) ? odd_n : even_n) + 1) >> 1;
    uint32_t i = lane >> 2;  // this lane's node of list lane & 3
    uint64_t r = 2 * i + 1 < m ? node_hash(left, right) : left;
    const auto level = [&](uint64_t above) {  // lanes of even i; the others compute a value nothing reads
        m = (m + 1) >> 1;
        if (i + 1 < m) r = node_hash(r, above);
        i >>= 1;
    };
    level(from_above<4>(r));
    level(from_above<8>(r));
    level(from_above<16>(r));
    level(from_above<32>(r));
    return r;
}

// The tile a workgroup takes (xcd_tile_of).  Measured on MI355X against the
// plain blockIdx order: pack + fingerprint of a 512 MiB ring window 204 ->
// 190-198 us, restore 189 -> 180-185 us; on the 1024-session batch the fused
// kernel 11.5 -> 10.9-11.0 ms in every input placement tried, where
// contiguous eighths alone gave 11.45 ms in some.
__device__ __forceinline__ uint32_t xcd_tile() { return xcd_tile_of(blockIdx.x, gridDim.x); }

// Device addresses arrive as integers; casting them to the global address
// space makes the compiler emit global_* (not flat_*) memory instructions.
typedef uint32_t v4u32 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(1))) v4u32 g_v4u32;
typedef __attribute__((address_space(1))) uint64_t g_u64;
typedef __attribute__((address_space(1))) uint32_t g_u32;
typedef __attribute__((address_space(1))) uint16_t g_u16;
typedef __attribute__((address_space(1))) uint8_t g_u8;

__device__ __forceinline__ uint4 load16(uint64_t a)
{
    const v4u32 v = *(const g_v4u32 *)a;
    return make_uint4(v.x, v.y, v.z, v.w);
}
__device__ __forceinline__ void store16(uint64_t a, uint4 v)
{
    const v4u32 w = {v.x, v.y, v.z, v.w};
    *(g_v4u32 *)a = w;
}

// Streaming (nontemporal) forms for bulk state that is touched once per call.
__device__ __forceinline__ uint4 load16_nt(uint64_t a)
{
    const v4u32 v = __builtin_nontemporal_load((const g_v4u32 *)a);
    return make_uint4(v.x, v.y, v.z, v.w);
}
__device__ __forceinline__ void store16_nt(uint64_t a, uint4 v)
{
    const v4u32 w = {v.x, v.y, v.z, v.w};
    __builtin_nontemporal_store(w, (g_v4u32 *)a);
}

// Bytes [0, n) of a granule from `a` (n < 16), zero above: in-bounds reads only.
__device__ uint4 load_partial(uint64_t a, uint32_t n)
{
    uint32_t w[4] = {0, 0, 0, 0};
    const g_u8 *p = (const g_u8 *)a;
    for (uint32_t k = 0; k < n; ++k) w[k >> 2] |= (uint32_t)p[k] << (8 * (k & 3));
    return make_uint4(w[0], w[1], w[2], w[3]);
}

__device__ void store_partial(uint64_t a, uint4 v, uint32_t n)
{
    g_u8 *p = (g_u8 *)a;
    const uint32_t w[4] = {v.x, v.y, v.z, v.w};
    for (uint32_t k = 0; k < n; ++k) p[k] = (uint8_t)(w[k >> 2] >> (8 * (k & 3)));
}

// Inclusive prefix sum across the 64 lanes of a wavefront, in DPP moves (no
// LDS round trips): shifts by 1, 2, 4 and 8 lanes within each row of 16
// lanes, then row 0's total (lane 15) into row 1 and row 2's into row 3
// (row_bcast:15), then rows 0-1's total (lane 31) into rows 2 and 3
// (row_bcast:31).  A lane whose source lies outside its row, or a row the
// row mask leaves out, adds 0 (the `old` operand).
__device__ __forceinline__ uint32_t wave_incl_scan(uint32_t x)
{
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x111, 0xF, 0xF, false);  // row_shr:1
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x112, 0xF, 0xF, false);  // row_shr:2
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x114, 0xF, 0xF, false);  // row_shr:4
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x118, 0xF, 0xF, false);  // row_shr:8
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x142, 0xA, 0xF, false);  // row_bcast:15
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x143, 0xC, 0xF, false);  // row_bcast:31
    return x;
}

// Values that pass between workgroups of one launch go through these, or
// through agent-scope atomics, and nothing else does: an agent-scope access
// goes to memory, past the eight XCDs' L2 caches, which are not coherent with
// one another.  What orders them is the ticket: a wavefront waits until its own
// stores have reached memory (vmcnt) before the ticket is taken for it, and
// loads what the others left only after it has seen the last ticket.  So the
// tickets need no release or acquire of their own, which would write back and
// invalidate a whole L2 each time (1024 workgroups taking one: 24 us with,
// 14 us without; at one ticket per eight workgroups 16 us against none
// measurable).
template <class V>
__device__ __forceinline__ void agent_store(V *p, V v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <class V>
__device__ __forceinline__ V agent_load(const V *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// Adds to a ticket word for one lane, after this wavefront's stores have
// reached memory; the word's value before.
template <class V>
__device__ __forceinline__ V take_ticket(V *word, V add)
{
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    const V n = __hip_atomic_fetch_add(word, add, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    asm volatile("" ::: "memory");
    return n;
}
// True in every lane of the last of `of` wavefronts to get here; the ticket
// is then back at zero.
__device__ __forceinline__ bool last_wavefront(uint32_t *ticket, uint32_t of)
{
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    uint32_t last = 0;
    if ((threadIdx.x & 63) == 0) {
        last = take_ticket(ticket, 1u) + 1 == of;
        if (last) agent_store(ticket, 0u);
    }
    return __builtin_amdgcn_readfirstlane(last) != 0;
}
// The same for whole workgroups (every thread calls it).
__device__ __forceinline__ bool last_workgroup(uint32_t *ticket, uint32_t of, uint32_t *flag)
{
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (threadIdx.x == 0) {
        *flag = take_ticket(ticket, 1u) + 1 == of;
        if (*flag) agent_store(ticket, 0u);
    }
    __syncthreads();
    return *flag != 0;
}

// ---------------------------------------------------------------- job tables

// Stages a job's tables for the kernels that follow on the stream: copies
// n16 16-byte units from mapped host memory to device memory, and one lane
// per group writes the map entry of its buffer.  The map part starts from
// group counts on the host side of the link, so a wavefront takes one buffer
// at a time (two reads over the link) and fills that buffer's entries.
// Workgroups [0, copy_blocks) copy, the rest map.  One launch where a copy
// and a map launch took two (2.9 + 3.2 us and the gap between them).
constexpr uint32_t kStageLanes = 256, kStageUnits = 4 * kStageLanes;
__global__ __launch_bounds__(kStageLanes) void k_stage(uint64_t host, uint64_t dev, uint64_t n16, uint32_t copy_blocks,
                                                       const JobBuf *__restrict__ host_bufs, uint32_t nbuf,
                                                       uint32_t *__restrict__ map)
{
    const uint32_t t = threadIdx.x;
    if (blockIdx.x < copy_blocks) {
        const uint64_t u0 = (uint64_t)blockIdx.x * kStageUnits + t;
        uint4 v[4];
#pragma unroll
        for (uint32_t k = 0; k < 4; ++k)
            if (u0 + k * kStageLanes < n16) v[k] = load16(host + 16 * (u0 + k * kStageLanes));
#pragma unroll
        for (uint32_t k = 0; k < 4; ++k)
            if (u0 + k * kStageLanes < n16) store16(dev + 16 * (u0 + k * kStageLanes), v[k]);
        return;
    }
    const uint32_t b = (blockIdx.x - copy_blocks) * (kStageLanes / 64) + (t >> 6);
    if (b >= nbuf) return;
    const uint64_t first = host_bufs[b].group_begin, chunks = host_bufs[b].nchunks();
    const uint64_t n = chunks / kGroupChunks + (chunks % kGroupChunks != 0);
    for (uint64_t i = t & 63; i < n; i += 64) map[first + i] = b;
}

// What a tile kernel needs of one buffer, in registers of the wavefront that
// asked (the same in every lane).
struct TileBuf {
    Geom g;
    uint64_t nchunks, chunk_begin, group_begin;
    uint64_t slots;        // device address of chunk 0's slot (pack, restore)
    uint64_t slot_list;    // restore: address of its manifest entries (0: slots are contiguous)
    uint64_t hash[2];      // addresses of chunk 0's fingerprint outputs
    uint64_t parent_hash;  // diff, verify: address of the fingerprint chunk 0 is compared with
    uint64_t parent_chunks, manifest, parent_manifest, parent_slot0;  // diff
    uint32_t index;
};

// Group G's buffer, read by a whole wavefront (CPW: the chunks of the
// kernel's tiles).
template <int MODE, int CPW>
__device__ __forceinline__ TileBuf tile_buf(const DevTables &tab, uint64_t G)
{
    TileBuf b;
    b.index = __builtin_amdgcn_readfirstlane(tab.map[G]);
    const JobBuf &jb = tab.bufs[b.index];
    b.g = jb.g;
    b.nchunks = jb.nchunks();
    b.chunk_begin = jb.chunk_begin;
    b.group_begin = jb.group_begin;
    b.slots = jb.payload;
    b.slot_list = MODE == kModeVerify ? jb.manifest : 0;
    b.hash[0] = jb.hash_dst[0];
    b.hash[1] = jb.hash_dst[1];
    b.parent_hash = jb.parent_hash;
    b.parent_chunks = jb.parent_chunks;
    b.manifest = jb.manifest;
    b.parent_manifest = jb.parent_manifest;
    b.parent_slot0 = jb.parent_slot0;
    return b;
}

// The argument tables in a wavefront's registers: lane l holds buffers l and
// 64 + l % 32 and ring l % 16.  A search, one dependent load a step and several
// more for the chosen entry, took 5,700 cycles of an 8-chunk tile's 20,000.
static_assert(kArgBufs == 96 && kArgRings == 16, "lanes of ArgLanes");
struct ArgLanes {
    ArgBuf lo, hi;
    ArgRing ring;
    uint32_t ring_buf;
    uint64_t valid_lo, valid_hi, rings;  // ballots
    __device__ __forceinline__ explicit ArgLanes(const ArgTables &t)
    {
        const uint32_t lane = threadIdx.x & 63;
        lo = t.bufs[lane];
        hi = t.bufs[64 + (lane & 31)];
        ring = t.rings[lane & 15];
        ring_buf = t.ring_buf[lane & 15];
        valid_lo = __ballot(lane < t.nbuf);
        valid_hi = __ballot(lane < 32 && 64 + lane < t.nbuf);
        rings = __ballot(lane < t.nring);
    }
    // Asks for every field to be in its register here, so that all loads are in
    // flight together and a workgroup learns its buffer in one round trip to
    // memory.  The compiler on its own moves the loads of a chosen entry's fields
    // behind the choice, a second round trip: 32 MiB ring windows restored in
    // 12.4 us and fingerprinted in 16.0, with this 12.1 and 15.7.  (Not for
    // classification, which needs few fields: 6.6 against 7.5 us there.)
    __device__ __forceinline__ void hold()
    {
        asm volatile("" : "+v"(lo.addr), "+v"(lo.nbytes), "+v"(lo.chunk_begin), "+v"(lo.group_begin), "+v"(lo.aux),
                          "+v"(hi.addr), "+v"(hi.nbytes), "+v"(hi.chunk_begin), "+v"(hi.group_begin), "+v"(hi.aux));
        asm volatile("" : "+v"(ring.win), "+v"(ring.first), "+v"(ring.head), "+v"(ring.stride), "+v"(ring.inv_win),
                          "+v"(ring_buf));
    }
    // The buffer of group G: the last one that begins at or before it (an
    // empty buffer begins where the next one does and loses).
    __device__ __forceinline__ uint32_t find(uint64_t G) const
    {
        const uint64_t a = __ballot(lo.group_begin <= G) & valid_lo, b = __ballot(hi.group_begin <= G) & valid_hi;
        return (uint32_t)(__popcll(a) + __popcll(b)) - 1;
    }
    __device__ __forceinline__ ArgBuf buf(uint32_t i) const
    {
        const uint32_t l = i & 63;
        ArgBuf r;
        if (i < 64) {
            r.addr = lane_word(lo.addr, l);
            r.nbytes = lane_word(lo.nbytes, l);
            r.chunk_begin = lane_word(lo.chunk_begin, l);
            r.group_begin = lane_word(lo.group_begin, l);
            r.aux = lane_word(lo.aux, l);
        } else {
            r.addr = lane_word(hi.addr, l);
            r.nbytes = lane_word(hi.nbytes, l);
            r.chunk_begin = lane_word(hi.chunk_begin, l);
            r.group_begin = lane_word(hi.group_begin, l);
            r.aux = lane_word(hi.aux, l);
        }
        return r;
    }
    __device__ __forceinline__ Geom geom(uint32_t i, const ArgBuf &b) const
    {
        Geom g{b.addr, b.nbytes, 0, 0, 0, 0, 0};
        const uint64_t m = __ballot(ring_buf == i) & rings;
        if (m) {
            const uint32_t l = (uint32_t)__builtin_ctzll(m);
            g.win = lane_word(ring.win, l);
            g.first = lane_word(ring.first, l);
            g.head = lane_word(ring.head, l);
            g.stride = lane_word(ring.stride, l);
            g.inv_win = __longlong_as_double((long long)lane_word((uint64_t)__double_as_longlong(ring.inv_win), l));
        }
        return g;
    }
};
// A job of one buffer in whole-group tiles reads that entry alone, by scalar
// loads: a launch of few rounds shows the difference (fingerprints of 128 / 200
// MiB 31.2 / 48.4 -> 30.4 / 47.1 us, packs of 200 MiB 82.0 -> 81.0).  8-chunk tiles
// gain nothing from it, and with several buffers the question costs 0.2 us or so.
template <int MODE, int CPW>
__device__ __forceinline__ TileBuf tile_buf(const ArgTables &tab, uint64_t G)
{
    TileBuf b;
    ArgBuf a;
    if (CPW == kGroupChunks && tab.nbuf == 1) {
        a = tab.bufs[0];
        b.index = 0;
        b.g = Geom{a.addr, a.nbytes, 0, 0, 0, 0, 0};
        if (tab.nring) {
            const ArgRing &r = tab.rings[0];
            b.g = Geom{a.addr, a.nbytes, r.win, r.first, r.head, r.stride, r.inv_win};
        }
    } else {
        ArgLanes lanes(tab);
        lanes.hold();
        b.index = lanes.find(G);
        a = lanes.buf(b.index);
        b.g = lanes.geom(b.index, a);
    }
    b.nchunks = chunks_of(a.nbytes);
    b.chunk_begin = a.chunk_begin;
    b.group_begin = a.group_begin;
    const bool listed = MODE == kModeVerify && (a.aux & kAuxManifest);
    b.slots = listed ? 0 : a.aux;
    b.slot_list = listed ? a.aux & ~kAuxManifest : 0;
    b.hash[0] = tab.hash[0] ? tab.hash[0] + 8 * b.chunk_begin : 0;
    b.hash[1] = tab.hash[1] ? tab.hash[1] + 8 * b.chunk_begin : 0;
    const uint64_t pb = MODE == kModeDiff ? (uint32_t)a.aux : b.chunk_begin;
    b.parent_hash = tab.parent_hash + 8 * pb;
    b.parent_chunks = a.aux >> 32;
    b.manifest = tab.manifest ? tab.manifest + 8 * b.chunk_begin : 0;
    b.parent_manifest = tab.parent_manifest ? tab.parent_manifest + 8 * pb : 0;
    b.parent_slot0 = tab.parent_slot0 + pb * kChunk;
    return b;
}

// A tile's setup, by the first wavefront of a workgroup: its buffer, then
// lane c describes chunk c of the tile (CPW chunks, `part` of its group).
// The others read from LDS after a barrier what the tile needs: each field is
// written on its own, and the geometry only for a tile with a chunk of more
// than two pieces, so that few registers are live at once (all at once they
// cost the 1024-lane hash tiles their second workgroup per CU).
struct TileInfo {
    uint64_t c0;  // the tile's first chunk
    uint32_t nv;  // its chunks (0: the buffer's last group ends before this tile)
    bool many;    // a chunk of it spans more than two pieces
    bool ragged;  // its last chunk ends inside a granule
    uint32_t buf, group_begin;  // the buffer, its first group and its chunks
    uint64_t nchunks;
    uint64_t hash[2], parent_hash, parent_chunks, manifest, parent_manifest, parent_slot0;
    Geom g;
};
template <int MODE, int CPW, class Tab>
__device__ __forceinline__ void tile_setup(const Tab &tab, uint64_t G, uint32_t part, uint64_t arena_base,
                                           TileInfo *info, ChunkLoc *loc)
{
    const uint32_t t = threadIdx.x;
    if (t < 64) {
        const TileBuf b = tile_buf<MODE, CPW>(tab, G);
        const uint64_t c0 = (G - b.group_begin) * kGroupChunks + part * CPW;
        const uint32_t nv = c0 < b.nchunks ? (uint32_t)umin(CPW, b.nchunks - c0) : 0;
        bool pieces = false;
        if (t < CPW) {
            ChunkLoc l{0, 0, 0, 0, 0};
            if (t < nv) {
                l = chunk_loc(b.g, c0 + t);
                pieces = l.a1 == 0;
                if (MODE == kModeVerify && b.slot_list) l.slot = arena_base + ((const g_u64 *)b.slot_list)[c0 + t];
                else if (MODE == kModePack || MODE == kModeVerify) l.slot = b.slots + (c0 + t) * kChunk;
            }
            loc[t] = l;
        }
        const auto put = [&](uint64_t *field, uint64_t v) {
            if (t == 0) *field = v;
            __builtin_amdgcn_sched_barrier(0);
        };
        put(&info->c0, c0);
        if (t == 0) info->nv = nv;
        put(&info->hash[0], b.hash[0]);
        put(&info->hash[1], b.hash[1]);
        if (MODE == kModeDiff || MODE == kModeVerify) put(&info->parent_hash, b.parent_hash);
        if (MODE == kModeDiff) {
            put(&info->parent_chunks, b.parent_chunks);
            put(&info->manifest, b.manifest);
            put(&info->parent_manifest, b.parent_manifest);
            put(&info->parent_slot0, b.parent_slot0);
        }
        const bool many = __any(pieces);
        if (t == 0) {
            info->many = many;
            info->buf = b.index;
            info->group_begin = (uint32_t)b.group_begin;
            info->nchunks = b.nchunks;
            info->ragged = (b.g.nbytes & 15) != 0 && c0 + nv == b.nchunks;
        }
        if (many) {
            put(&info->g.addr, b.g.addr);
            put(&info->g.nbytes, b.g.nbytes);
            put(&info->g.win, b.g.win);
            put(&info->g.first, b.g.first);
            put(&info->g.head, b.g.head);
            put(&info->g.stride, b.g.stride);
            if (t == 0) info->g.inv_win = b.g.inv_win;
        }
    }
    __syncthreads();
}

// ---------------------------------------------------------------- fingerprint

// Waits for every load (and store) this wavefront has in flight.  k_copy puts
// it where a prefetched slice is first needed, before the step's stores: their
// number varies by lane, so left to itself the compiler waits for all memory
// operations at each later use, that is for each store before the next store
// and for all of them before the next slice's loads.  In k_copy at 100 / 128 /
// 256 MiB packs went from 41.1 / 47.0 / 82.7 to 35.3 / 41.7 / 79.2 us and
// restores from 40.1 / 48.2 / 89.5 to 37.6 / 45.2 / 87.6.  The fused pack
// (hash_tile) keeps the compiler's waits: there the same wait cost 348 -> 357
// us at 1 GiB, where the stores' own waits pace the write-back.
__device__ __forceinline__ void wait_loads() { __builtin_amdgcn_s_waitcnt(0x0F70); }  // vmcnt(0)

// U granules of a lane, granule k at at[k]: its 16 bytes at offset x of a chunk
// of len[k] bytes, zero past the chunk's end.  Every whole granule's load is
// issued before the rare partial ones, which wait byte by byte (ragged: there
// is one in the tile; decided per granule, each load waited for the last).
template <int U>
__device__ __forceinline__ void load_granules(const uint64_t (&at)[U], const uint32_t (&len)[U], uint32_t x, bool ragged,
                                              uint4 (&r)[U])
{
#pragma unroll
    for (int k = 0; k < U; ++k) {
        r[k] = make_uint4(0, 0, 0, 0);
        if (x + 16 <= len[k]) r[k] = load16_nt(at[k]);
    }
    if (ragged) {
#pragma unroll
        for (int k = 0; k < U; ++k)
            if (x < len[k] && x + 16 > len[k]) r[k] = load_partial(at[k], len[k] - x);
    }
}

// Where byte x (x < l.len, a multiple of 16) of a tile's chunk c lies, in a tile
// that has a chunk of more than two pieces: from the chunk's description, or,
// for such a chunk itself, from the geometry.
__device__ __forceinline__ uint64_t granule_at(const TileInfo &info, const ChunkLoc &l, uint32_t c, uint32_t x)
{
    if (x >= l.len) return 0;
    if (l.a1) return (x < l.split ? l.a1 : l.a2) + x;
    return locate(info.g, (info.c0 + c) * kChunk + x).addr;
}

// First-round stagger.  The workgroups of a launch's first round (one per CU)
// all start together and then move their slices in step: every CU reads the
// same offsets within its chunks at the same moment.  In jobs of a few
// rounds this costs the first two rounds about a fifth of their speed
// (per-workgroup timelines on MI355X, 512 MiB pack + fingerprint: 25 against
// 21 us per group; jobs of 768 MiB and more do not show it).  Holding the
// first-round workgroups back by 0..7 phases of stg.ticks of the constant
// real-time counter (phase = position within the XCD, mod 8) spreads them
// over most of a group's duration; later workgroups start whenever a CU
// frees up and need no stagger.  The wait is also bounded by a spin count,
// so it ends even if the counter stood still.
__device__ __forceinline__ void stagger_start(const Stagger &stg)
{
    if (stg.ticks == 0 || blockIdx.x >= stg.first_round) return;
    const uint64_t wait = (uint64_t)((blockIdx.x / kXcds) % kStaggerPhases) * stg.ticks;
    const uint64_t t0 = __builtin_amdgcn_s_memrealtime();
    for (uint32_t spin = 0; spin < kStaggerMaxSpins && __builtin_amdgcn_s_memrealtime() - t0 < wait; ++spin)
        __builtin_amdgcn_s_sleep(2);
}

// N stripes of one accumulator's chain, the lane words (already multiplied by
// P2) 32 bytes apart in LDS: the next B are loaded while B are consumed, so
// the chain waits on its own arithmetic alone (28 cycles a round measured
// with the words in registers; 64 when each group of eight reads waited).  A
// loop, not unrolled: unrolled, the compiler moves all N loads up front and
// out of registers.
template <int N>
__device__ __forceinline__ uint64_t chain(uint64_t va, const uint8_t *p)
{
    constexpr int B = 16;
    static_assert(N % (2 * B) == 0, "whole pairs of batches");
    uint64_t d[B], e[B];
#pragma unroll
    for (int i = 0; i < B; ++i) d[i] = *reinterpret_cast<const uint64_t *>(p + 32 * i);
#pragma unroll 1
    for (int s = 0; s < N; s += 2 * B, p += 64 * B) {
#pragma unroll
        for (int i = 0; i < B; ++i) e[i] = *reinterpret_cast<const uint64_t *>(p + 32 * (B + i));
#pragma unroll
        for (int i = 0; i < B; ++i) va = xstep(va, d[i]);
        if (s + 2 * B < N) {
#pragma unroll
            for (int i = 0; i < B; ++i) d[i] = *reinterpret_cast<const uint64_t *>(p + 32 * (2 * B + i));
        }
#pragma unroll
        for (int i = 0; i < B; ++i) va = xstep(va, e[i]);
    }
    return va;
}

// What the 8-chunk tiles of a small job in the argument tables do at their
// end, so that no launch has to follow them (tab.tail): the last tile of a
// group to finish, then the last group of a buffer, then the last buffer of the
// job, each by the first wavefront of its workgroup.  A step up costs a
// round trip or two to memory (about 1.5 us); the launch it saves took 4 us and
// the gap before it.  Needs every buffer non-empty: an empty one has no tile.
//
// Roots: `node`, in lane 0, is the tile's.
__device__ __forceinline__ void tail_roots(const ArgTables &tab, const TileInfo &info, uint64_t *nodes, uint32_t tile_id,
                                           uint64_t node)
{
    TailWords *w = (TailWords *)tab.tail;
    uint64_t *group_nodes = (uint64_t *)tab.tail_scratch, *buf_roots = group_nodes + gridDim.x / kSmallTiles;
    const uint32_t lane = threadIdx.x & 63, G = tile_id / kSmallTiles, b = info.buf;
    const uint64_t left = info.nchunks - (uint64_t)(G - info.group_begin) * kGroupChunks;
    const uint32_t nt = ((uint32_t)umin(left, kGroupChunks) + 7) / 8;
    const uint32_t ng = (uint32_t)((info.nchunks + kGroupChunks - 1) / kGroupChunks);
    // n values of a list of at most 128, as the wavefront's root.
    const auto reduce = [&](const uint64_t *p, uint32_t n) {
        uint64_t v = wave_merkle<1, 6>(lane < n ? agent_load(p + lane) : 0, min(n, 64u));
        if (n > 64) v = node_hash(v, wave_merkle<1, 6>(64 + lane < n ? agent_load(p + 64 + lane) : 0, n - 64));
        return v;
    };
    if (nt > 1) {
        if (lane == 0) agent_store(nodes + tile_id, node);
        if (!last_wavefront(w->group[G], nt)) return;
        node = wave_merkle<1, 3>(lane < nt ? agent_load(nodes + G * kSmallTiles + lane) : 0, nt);
    }
    if (ng > 1) {
        if (lane == 0) agent_store(group_nodes + G, node);
        if (!last_wavefront(&w->buf[b], ng)) return;
        node = reduce(group_nodes + info.group_begin, ng);
    }
    if (lane == 0) {
        if (tab.root[0]) ((g_u64 *)tab.root[0])[b] = node;
        if (tab.root[1]) ((g_u64 *)tab.root[1])[b] = node;
    }
    if (!tab.sroot[0] && !tab.sroot[1]) return;
    if (tab.nbuf > 1) {
        if (lane == 0) agent_store(buf_roots + b, node);
        if (!last_wavefront((uint32_t *)&w->job, tab.nbuf)) return;
        node = reduce(buf_roots, tab.nbuf);
    }
    if (lane == 0) {
        if (tab.sroot[0]) *(g_u64 *)tab.sroot[0] = node;
        if (tab.sroot[1]) *(g_u64 *)tab.sroot[1] = node;
    }
}

// Flags set by a diff or verify (n of them in this tile): the job's number of
// them to tab.tail_count (diff), or each buffer's label to tab.tail_labels
// (verify).  The tickets carry the counts; lane 0 alone.
template <int MODE>
__device__ __forceinline__ void tail_flags(const ArgTables &tab, const TileInfo &info, uint32_t tile_id, uint32_t n)
{
    TailWords *w = (TailWords *)tab.tail;
    const uint32_t G = tile_id / kSmallTiles;
    const uint64_t left = info.nchunks - (uint64_t)(G - info.group_begin) * kGroupChunks;
    const uint32_t nt = ((uint32_t)umin(left, kGroupChunks) + 7) / 8;
    if (nt > 1) {
        const uint32_t old = take_ticket(w->group[G], (1u << 16) + n);
        if ((old >> 16) + 1 != nt) return;
        agent_store(w->group[G], 0u);
        n += old & 0xFFFF;
    }
    if (MODE == kModeDiff) {
        const uint64_t old = take_ticket(&w->job, ((uint64_t)1 << 32) + n);
        if ((old >> 32) + 1 != gridDim.x / kSmallTiles) return;
        agent_store(&w->job, (uint64_t)0);
        *(volatile uint64_t *)tab.tail_count = (uint32_t)old + n;
        __threadfence_system();
    } else {
        const uint32_t ng = (uint32_t)((info.nchunks + kGroupChunks - 1) / kGroupChunks);
        if (ng > 1) {
            const uint32_t old = take_ticket(&w->buf[info.buf], (1u << 16) + (n ? 1u : 0u));
            if ((old >> 16) + 1 != ng) return;
            agent_store(&w->buf[info.buf], 0u);
            n += old & 0xFFFF;
        }
        ((g_u8 *)tab.tail_labels)[info.buf] = n ? 1 : 0;
    }
}

// Fingerprint tile kernels (k_hash, k_hash_staggered; the body is
// hash_tile).  One workgroup = one tile of CPW chunks of one
// buffer: a whole 64-chunk group, or for small jobs an eighth of one, so
// that a few groups still occupy many CUs (the tile's Merkle node is then an
// aligned 8-chunk subtree).  Step k moves the k-th SL-byte slice of every
// chunk of the tile:
// all T lanes load it with coalesced 16-byte loads (SL/16 lanes per chunk
// slice), kModePack stores it to the chunk's snapshot slot (zero-padding a
// partial last chunk) and kModeVerify to the buffer's pieces, and every lane
// writes it to an LDS tile; then lane quads of the first 4*CPW lanes hash
// the tile while the next slice's loads are in flight.  Lane q of a quad owns
// XXH64 accumulator q, which reads exactly bytes [8q, 8q+8) of each 32-byte
// stripe.  A wavefront issues a lane's rounds one after another, so one
// accumulator per lane halves the instructions a chunk's
// chain costs each wavefront and spreads the hashing over twice as many
// wavefronts as lane pairs with two accumulators each would.  For the same
// reason the words of a sub-tile, whose time is that chain's, reach LDS already
// multiplied by P2, the half of a round
// that does not depend on the accumulator: all T lanes share that work, and
// the chain keeps one multiplication of two.  (Whole groups are bound by
// memory, and the registers this takes cost them a workgroup per CU.)
// kModeDiff /
// kModeVerify ballot one flag per chunk into a per-group mask (the group is
// one bitmap word; a diff sub-tile writes its byte of the word).  WB: the
// pack stores go through the caches (write-back) instead of streaming past
// them; see kPackWriteBackMaxRounds.
template <class Tab, int MODE, int T, int SL, int CPW, bool STAGGER, bool WB>
__device__ __forceinline__ void hash_tile(const Tab &tab, uint64_t *__restrict__ nodes,
                                          uint64_t *__restrict__ flag_mask, uint64_t arena_base, const Stagger &stg)
{
    constexpr uint32_t kSteps = kChunk / SL;
    constexpr uint32_t kRow = SL + 32;                  // padded LDS row: the quads of 8 chunks hit distinct banks
    constexpr uint32_t LPS = SL / 16;                   // lanes per chunk slice
    constexpr int U = CPW * SL / 16 / T;                // granules per lane per step
    constexpr uint32_t kTiles = kGroupChunks / CPW;     // tiles per 64-chunk group
    constexpr uint32_t kHashers = 64 * ((4 * CPW + 63) / 64);  // lanes of the wavefronts that hold accumulators
    constexpr bool kScaled = CPW == 8;                  // words reach LDS multiplied by P2
    constexpr bool kFromSlots = MODE == kModeVerify;    // source is the snapshot, destination the pieces
    static_assert(U >= 1 && T % LPS == 0 && kGroupChunks % CPW == 0, "tile shape");
    static_assert(T >= 4 * CPW, "one lane per accumulator");
    constexpr bool kFlags = MODE == kModeDiff || MODE == kModeVerify;
    static_assert(kSteps > 1 || MODE != kModePack || WB, "one-step tiles store write-back");
    static_assert(CPW == kGroupChunks || CPW == 8, "a sub-tile is hashed by one wavefront and writes one mask byte");
    __shared__ __attribute__((aligned(16))) uint8_t tile[CPW * kRow];
    __shared__ ChunkLoc cloc[CPW];
    __shared__ TileInfo info;
    __shared__ uint64_t partial[4];
    __shared__ uint32_t dflag[CPW];
    // A chunk's last bytes past its whole stripes, zero padded; written and
    // read by the chunk's own lane quad.  (In registers, eight a lane for the
    // rare chunk that has any, they put the 1024-lane diff tile over its 64:
    // 12 bytes a lane of scratch memory.)
    __shared__ uint64_t tail[CPW][4];

    const uint32_t tile_id = xcd_tile();
    if constexpr (STAGGER) stagger_start(stg);
    const uint64_t G = tile_id / kTiles;
    const uint32_t t = threadIdx.x;
    tile_setup<MODE, CPW>(tab, G, tile_id % kTiles, arena_base, &info, cloc);
    const uint32_t nv = __builtin_amdgcn_readfirstlane(info.nv);
    if (nv == 0) {
        // A sub-tile owns byte (tile % 8) of its group's mask: an empty one
        // writes it as 0 so every byte of the mask is defined.
        if (kFlags && kTiles > 1 && t == 0 && flag_mask)
            ((g_u8 *)flag_mask)[G * kTiles + tile_id % kTiles] = 0;
        return;
    }
    const uint64_t c0 = info.c0;

    const uint32_t slot = (t % LPS) * 16;  // this lane's place in each slice
    const bool ragged = __builtin_amdgcn_readfirstlane(info.ragged);
    const uint32_t ci = t >> 2, q = t & 3;
    const bool hasher = t < 4 * CPW && ci < nv;
    const uint32_t len = hasher ? cloc[ci].len : 0;
    const uint32_t nst = len >> 5;
    const uint64_t i = c0 + ci;
    // What the chunk's fingerprint is compared with and, in an incremental
    // checkpoint, where the parent holds it (entered in the new manifest if
    // the chunk is clean; a dirty chunk's entry is its slot, written once the
    // slots are placed): fetched right after the tile's first loads, used at
    // the end.
    uint64_t parent_loc = 0, want = 0;
    bool compare = false;
    const auto fetch_parent = [&] {
        if (!kFlags || !hasher || q != 0) return;
        if (MODE == kModeDiff && i < info.parent_chunks) {
            compare = true;
            want = ((const g_u64 *)info.parent_hash)[i];
            if (info.manifest)
                parent_loc = info.parent_manifest ? ((const g_u64 *)info.parent_manifest)[i]
                                                    : info.parent_slot0 + i * kChunk;
        }
        if (MODE == kModeVerify) want = ((const g_u64 *)info.parent_hash)[i];
    };
    // Accumulator q with seed 0: P1 + P2, P2, 0, -P1.
    uint64_t va = q == 0 ? P1 + P2 : q == 1 ? P2 : q == 2 ? 0 : 0 - P1;

    // A granule's words to the LDS tile.
    const auto stage = [&](uint32_t c, uint32_t x, uint32_t clen, uint4 v) {
        uint64_t w0 = ((uint64_t)v.y << 32) | v.x, w1 = ((uint64_t)v.w << 32) | v.z;
        if (kScaled && x < (clen & ~31u)) {  // a whole stripe's words; the tail goes in as it is
            w0 *= P2;
            w1 *= P2;
        }
        *reinterpret_cast<ulonglong2 *>(tile + c * kRow + slot) = make_ulonglong2(w0, w1);
    };
    // Hashes the slice in the LDS tile.
    const auto hash_slice = [&](uint32_t step) {
        const uint32_t s0 = step * (SL / 32);
        const uint8_t *row = tile + (t < 4 * CPW ? ci : 0) * kRow;
        bool whole = false;
        if constexpr (kScaled) {
            whole = __all(!hasher || nst >= s0 + SL / 32);
            if (whole) va = chain<SL / 32>(va, row + 8 * q);
        }
        if (!whole && hasher) {
            const uint32_t ns = nst > s0 ? (uint32_t)umin(SL / 32, nst - s0) : 0;
#pragma unroll 8
            for (uint32_t s = 0; s < ns; ++s) {
                const uint64_t w = *reinterpret_cast<const uint64_t *>(row + 32 * s + 8 * q);
                va = kScaled ? xstep(va, w) : xround(va, w);
            }
            const uint32_t tp = nst * 32;  // tail start, 32-aligned, inside this slice if here
            if (tp < len && tp >= step * SL && tp < (step + 1) * SL) {
                tail[ci][q] = *reinterpret_cast<const uint64_t *>(row + tp - step * SL + 8 * q);
            }
        }
    };

    if (__builtin_amdgcn_readfirstlane(info.many)) {
        // A tile with a chunk of more than two pieces: a granule's place is read
        // from LDS, or located, each time (a loop of its own: the other one keeps
        // its granules' places in registers).  The next slice is fetched ahead
        // of the hashing where the registers of a second workgroup per CU
        // are not at stake.  One granule at a time, located anew each, took for
        // 2048 rings of 257 KiB, each with one such chunk, 193 us a
        // fingerprint, 261 a pack with fingerprint, 299 a restore (k_copy) and
        // 268 a verified one; so 108, 207, 186 and 197 (without such chunks
        // 98, 206, 182 and 194).
        constexpr bool kAhead = T != 1024 || MODE == kModePack || MODE == kModeVerify;
        uint4 r[U];
        const auto load_slice = [&](uint32_t x) {
            uint64_t at[U];
            uint32_t clen[U];
#pragma unroll
            for (int k = 0; k < U; ++k) {
                const uint32_t c = (k * T + t) / LPS;
                const ChunkLoc &l = cloc[c];
                // (slots are whole 4096-byte granules, zero padded)
                at[k] = kFromSlots ? l.slot + x : granule_at(info, l, c, x);
                clen[k] = kFromSlots ? (l.len + 15) & ~15u : l.len;
            }
            load_granules<U>(at, clen, x, ragged && !kFromSlots, r);
        };
        load_slice(slot);
        fetch_parent();
        for (uint32_t step = 0; step < kSteps; ++step) {
            const uint32_t x = step * SL + slot;
#pragma unroll
            for (int k = 0; k < U; ++k) {
                const uint32_t c = (k * T + t) / LPS;
                if (c < nv) {
                    const ChunkLoc &l = cloc[c];
                    if (MODE == kModePack) {
                        if (WB) store16(l.slot + x, r[k]);
                        else store16_nt(l.slot + x, r[k]);
                    }
                    if (kFromSlots && x < l.len) {
                        const uint64_t to = granule_at(info, l, c, x);
                        if (x + 16 <= l.len) store16_nt(to, r[k]);
                        else store_partial(to, r[k], l.len - x);
                    }
                    stage(c, x, l.len, r[k]);
                }
            }
            __syncthreads();
            if (kAhead && step + 1 < kSteps) load_slice(x + SL);
            if (t < kHashers) hash_slice(step);
            __syncthreads();
            if (!kAhead && step + 1 < kSteps) load_slice(x + SL);
        }
    } else if constexpr (kSteps == 1) {
        // Whole chunks in one step: nothing is prefetched, so a granule's
        // place is read from LDS where it is used (the memory clobber keeps
        // the compiler from holding all of them over the loads).
        uint4 r[U];
        uint64_t at[U];
        uint32_t clen[U];
#pragma unroll
        for (int k = 0; k < U; ++k) {
            const ChunkLoc &l = cloc[(k * T + t) / LPS];
            at[k] = (kFromSlots ? l.slot : slot < l.split ? l.a1 : l.a2) + slot;
            // (slots are whole 4096-byte granules, zero padded)
            clen[k] = kFromSlots ? (l.len + 15) & ~15u : l.len;
        }
        load_granules<U>(at, clen, slot, ragged && !kFromSlots, r);
        fetch_parent();
        asm volatile("" ::: "memory");
#pragma unroll
        for (int k = 0; k < U; ++k) {
            const uint32_t c = (k * T + t) / LPS;
            if (c < nv) {
                const ChunkLoc &l = cloc[c];
                if (MODE == kModePack) store16(l.slot + slot, r[k]);
                if (kFromSlots && slot < l.len) {
                    const uint64_t to = (slot < l.split ? l.a1 : l.a2) + slot;
                    if (slot + 16 <= l.len) store16_nt(to, r[k]);
                    else store_partial(to, r[k], l.len - slot);
                }
                stage(c, slot, l.len, r[k]);
            }
        }
        __syncthreads();
        if (t < kHashers) hash_slice(0);
        __syncthreads();
    } else {
        // This lane's granules: chunk (k*T + t) / LPS of each slice.
        uint64_t ga[U], gb[U];  // pieces side: where the chunk's bytes lie (ChunkLoc)
        uint64_t sa[U];         // slots side: the chunk's 4096-byte slot (0 if the group has no such chunk)
        uint32_t gs[U], gl[U];
#pragma unroll
        for (int k = 0; k < U; ++k) {
            const ChunkLoc l = cloc[(k * T + t) / LPS];
            ga[k] = l.a1;
            gb[k] = l.a2;
            gs[k] = l.split;
            gl[k] = l.len;
            sa[k] = l.slot;
        }
        const auto piece_addr = [&](int k, uint32_t x) -> uint64_t { return (x < gs[k] ? ga[k] : gb[k]) + x; };
        uint4 r[U];
        const auto load_slice = [&](uint32_t x) {
            uint64_t at[U];
#pragma unroll
            for (int k = 0; k < U; ++k) at[k] = kFromSlots ? sa[k] + x : piece_addr(k, x);
            load_granules<U>(at, gl, x, ragged && !kFromSlots, r);
            if (kFromSlots && ragged) {  // slots are whole 4096-byte granules, zero padded
#pragma unroll
                for (int k = 0; k < U; ++k)
                    if (x < gl[k] && x + 16 > gl[k]) r[k] = load16_nt(at[k]);
            }
        };
        load_slice(slot);
        fetch_parent();
        // Unrolled in the 1024-lane tiles: as a loop (the compiler's choice
        // once the function grew) a step's addresses and bounds are formed by
        // every lane anew, which a launch of one or two rounds shows.  Loop ->
        // unrolled, us: fingerprint of 128 / 200 MiB 32.1 / 49.8 -> 30.8 / 48.0,
        // incremental checkpoint of 128 / 512 MiB 38.6 / 107.4 -> 37.5 / 104.9 and of
        // a 512 MiB KV ring window 106.3 -> 102.7, verified restore of 88 MB
        // 46.8 -> 45.7.
#pragma unroll (T == 1024 ? kSteps : 1)
        for (uint32_t step = 0; step < kSteps; ++step) {
#pragma unroll
            for (int k = 0; k < U; ++k) {
                const uint32_t c = (k * T + t) / LPS;
                if (c < nv) {
                    const uint32_t x = step * SL + slot;
                    if (MODE == kModePack) {
                        if (WB) store16(sa[k] + x, r[k]);
                        else store16_nt(sa[k] + x, r[k]);
                    }
                    if (kFromSlots && x < gl[k]) {
                        if (x + 16 <= gl[k]) store16_nt(piece_addr(k, x), r[k]);
                        else store_partial(piece_addr(k, x), r[k], gl[k] - x);
                    }
                    stage(c, x, gl[k], r[k]);
                }
            }
            __syncthreads();
            if (step + 1 < kSteps) load_slice((step + 1) * SL + slot);
            if (t < kHashers) hash_slice(step);
            __syncthreads();
        }
    }

    // The wavefronts that hold no accumulator are done: they end here, not
    // behind the barrier below (which counts the living), so the CU can start
    // its next tile while the others finish the fingerprints and the node.
    // Packs with fingerprints of 90 / 200 MiB 45.5 / 82.5 -> 44.5 / 81.7 us, of 1 /
    // 2 GiB 343 / 674 -> 337 / 664.
    if (t >= kHashers) return;
    // Each lane's own part of the merge, then the quad's four together
    // (every lane of a quad ends with the same value).
    const uint64_t rot = rotl(va, q == 0 ? 1 : q == 1 ? 7 : q == 2 ? 12 : 18);
    uint64_t acc = rot + dpp64<0xB1>(rot);  // lanes 0+1, 2+3
    acc += dpp64<0x4E>(acc);
    const uint64_t m = xround(0, va);
    acc = (acc ^ dpp64<0x00>(m)) * P1 + P4;
    acc = (acc ^ dpp64<0x55>(m)) * P1 + P4;
    acc = (acc ^ dpp64<0xAA>(m)) * P1 + P4;
    acc = (acc ^ dpp64<0xFF>(m)) * P1 + P4;
    if (len < 32) acc = P5;
    acc += len;
    // Tail: 8-byte lanes, one 4-byte lane, single bytes (offsets
    // relative to the tail start).
    uint32_t o = 0;
    const uint32_t rem = len - nst * 32;
    for (; rem - o >= 8; o += 8) {
        acc ^= xround(0, tail[ci][o >> 3]);
        acc = rotl(acc, 27) * P1 + P4;
    }
    if (rem - o >= 4) {
        acc ^= (uint64_t)(uint32_t)tail[ci][o >> 3] * P1;
        acc = rotl(acc, 23) * P2 + P3;
        o += 4;
    }
    for (; o < rem; ++o) {
        const uint64_t byte = (tail[ci][o >> 3] >> (8 * (o & 7))) & 0xFF;
        acc ^= byte * P5;
        acc = rotl(acc, 11) * P1;
    }
    const uint64_t h = avalanche(acc);
    if (hasher && q == 0) {
        if (info.hash[0]) ((g_u64 *)info.hash[0])[i] = h;
        if (info.hash[1]) ((g_u64 *)info.hash[1])[i] = h;
        if (MODE == kModeDiff) {
            const bool d = !compare || want != h;
            dflag[ci] = d ? 1u : 0u;
            if (!d && info.manifest) ((g_u64 *)info.manifest)[i] = parent_loc;
        }
        if (MODE == kModeVerify) dflag[ci] = want != h ? 1u : 0u;
    }
    // The tile's Merkle node (an aligned subtree): 16 chunks per
    // wavefront, chunk c of it in lane 4c, then the wavefronts' roots.
    if (nodes) {
        const uint32_t wave = t >> 6, mine = nv > 16 * wave ? (uint32_t)umin(16, nv - 16 * wave) : 0;
        const uint64_t root = wave_merkle<4, CPW == 8 ? 3 : 4>(h, mine);
        if (CPW == 8) {
            bool finished = false;
            if constexpr (std::is_same<Tab, ArgTables>::value && !kFlags) {
                finished = tab.tail != 0;
                if (finished) tail_roots(tab, info, nodes, tile_id, root);
            }
            if (!finished && t == 0) nodes[tile_id] = root;
        } else if ((t & 63) == 0) {
            partial[wave] = root;
        }
    }
    if (CPW == 8 && !kFlags) return;
    __syncthreads();
    if (t < 64) {
        if (CPW != 8 && nodes) {
            const uint64_t root = wave_merkle<1, 2>(partial[t & 3], (nv + 15) / 16);
            if (t == 0) nodes[tile_id] = root;
        }
        if (kFlags) {
            // Bit c of group G's mask = chunk c of the group; a sub-tile
            // writes its 8 bits as byte (tile % 8) of the little-endian word.
            const uint64_t mask = __ballot(t < nv && dflag[t & (CPW - 1)] != 0);
            if (t == 0 && flag_mask) {
                if (kTiles == 1) flag_mask[G] = mask;
                else ((g_u8 *)flag_mask)[G * kTiles + tile_id % kTiles] = (uint8_t)mask;
            }
            if constexpr (CPW == 8 && std::is_same<Tab, ArgTables>::value)
                if (t == 0 && tab.tail) tail_flags<MODE>(tab, info, tile_id, (uint32_t)__popcll(mask));
        }
    }
}

// Wavefronts per SIMD a tile kernel's registers must leave room for.
constexpr int tile_waves(int MODE, int T, int CPW)
{
    if (CPW == 8) return 4;  // four 256-lane workgroups a CU, as many as LDS holds
    if (MODE == kModePack || MODE == kModeVerify) return 4;
    return T == 1024 ? 8 : 3;
}

template <class Tab, int MODE, int T, int SL, int CPW, bool WB>
__global__ __launch_bounds__(T, tile_waves(MODE, T, CPW)) void k_hash(const Tab tab, uint64_t *__restrict__ nodes,
                                                                      uint64_t *__restrict__ flag_mask,
                                                                      uint64_t arena_base)
{
    hash_tile<Tab, MODE, T, SL, CPW, false, WB>(tab, nodes, flag_mask, arena_base, Stagger{0, 0});
}

// k_hash with the first-round stagger (pack and verify jobs of a few rounds):
// a kernel of its own, so the others keep their code and arguments.  Its
// jobs are all within the write-back bound, so a pack stores write-back.
template <class Tab, int MODE, int T, int SL, int CPW>
__global__ __launch_bounds__(T) void k_hash_staggered(const Tab tab, uint64_t *__restrict__ nodes,
                                                      uint64_t *__restrict__ flag_mask, uint64_t arena_base,
                                                      Stagger stg)
{
    hash_tile<Tab, MODE, T, SL, CPW, true, MODE == kModePack>(tab, nodes, flag_mask, arena_base, stg);
}

// ---------------------------------------------------------------- Merkle lists

// Promote-odd Merkle root of src[0, m), computed by the whole workgroup
// (NT lanes; pre: the first level of a list of more than 4096 values is
// already in sa); the result is valid in thread 0.  Aligned 64-value blocks
// reduce independently (one wavefront each); up to two passes through global
// scratch sa/sb (each read only after it is fully written) bring the list to
// <= 4096 values, then the rest happens in LDS.  Ends with a barrier so the
// LDS buffers can be reused.
template <int NT>
__device__ uint64_t reduce_list(const uint64_t *src, uint64_t m, uint64_t *sa, uint64_t *sb, uint64_t *lds,
                                uint64_t *lds2, bool pre)
{
    constexpr uint32_t NW = NT / 64;  // wavefronts
    const uint32_t t = threadIdx.x, wave = t >> 6, lane = t & 63;
    uint64_t root = 0;
    if (m == 0) {
        root = empty_hash();
    } else {
        uint64_t *scratch[2] = {sa, sb};
        for (int k = 0; k < 2 && m > 4096; ++k) {
            // Four blocks per wavefront in flight: their loads issue before
            // the first reduction (a scheduling barrier keeps them there).
            // pre: the first level is already in sa (k_merkle_blocks).
            const uint64_t nb = (m + 63) / 64;
            for (uint64_t blk0 = wave; blk0 < nb && !(pre && k == 0); blk0 += 4 * NW) {
                uint64_t v[4];
                uint32_t cnt[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const uint64_t blk = blk0 + u * NW;
                    cnt[u] = blk < nb ? (uint32_t)umin(64, m - 64 * blk) : 0;
                    v[u] = lane < cnt[u] ? src[64 * blk + lane] : 0;
                }
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    if (!cnt[u]) continue;
                    const uint64_t r = wave_merkle<1, 6>(v[u], cnt[u]);
                    if (lane == 0) scratch[k][blk0 + u * NW] = r;
                }
            }
            __syncthreads();
            src = scratch[k];
            m = nb;
        }
        for (uint64_t j = t; j < m; j += NT) lds[j] = src[j];
        __syncthreads();
        const uint64_t *ls = lds;
        if (m > 64) {
            const uint64_t nb = (m + 63) / 64;
            for (uint64_t blk = wave; blk < nb; blk += NW) {
                const uint32_t cnt = (uint32_t)umin(64, m - 64 * blk);
                const uint64_t v = lane < cnt ? lds[64 * blk + lane] : 0;
                const uint64_t r = wave_merkle<1, 6>(v, cnt);
                if (lane == 0) lds2[blk] = r;
            }
            __syncthreads();
            ls = lds2;
            m = nb;
        }
        if (wave == 0) {
            const uint64_t v = lane < m ? ls[lane] : 0;
            root = wave_merkle<1, 6>(v, (uint32_t)m);
        }
    }
    __syncthreads();
    return root;
}

// One workgroup per list (device-memory list table); NT lanes (1024 when a
// list is long enough to need passes through memory, else 256).
template <int NT>
__global__ __launch_bounds__(NT) void k_merkle(const MerkleList *__restrict__ lists,
                                               const uint64_t *__restrict__ in,
                                               uint64_t *__restrict__ sa, uint64_t *__restrict__ sb,
                                               uint64_t *__restrict__ roots_out, bool pre)
{
    __shared__ uint64_t lds[4096];
    __shared__ uint64_t lds2[64];
    const MerkleList Lst = lists[blockIdx.x];
    const uint64_t root =
        reduce_list<NT>(in + Lst.begin, Lst.count, sa + Lst.begin, sb + Lst.begin, lds, lds2, pre);
    if (threadIdx.x == 0) {
        if (Lst.dst[0]) *(g_u64 *)Lst.dst[0] = root;
        if (Lst.dst[1]) *(g_u64 *)Lst.dst[1] = root;
        if (roots_out) roots_out[blockIdx.x] = root;
    }
}

// The Merkle lists of a job in the argument tables, as items: aligned blocks
// of 64 values of one buffer's list, numbered through the buffers.  Lane l of
// a wavefront holds the lists of buffers l and 64 + l: their counts, and the
// items up to and including theirs.  pre: the lists' first level is done, so
// each holds a value per block, at the list's own offset (k_merkle_items).
struct ArgItems {
    uint64_t begin[2], count[2];
    uint32_t incl[2], items[2];
    uint32_t total;
    __device__ __forceinline__ ArgItems(const ArgTables &t, uint32_t tiles, bool pre)
    {
        const uint32_t lane = threadIdx.x & 63;
        uint32_t base = 0;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const uint32_t j = h * 64 + lane;
            const ArgBuf &b = t.bufs[j < kArgBufs ? j : 0];
            const uint64_t n = j < t.nbuf ? chunks_of(b.nbytes) : 0;
            begin[h] = (uint64_t)b.group_begin * tiles;
            count[h] = merkle_values(n, tiles, pre);
            items[h] = merkle_items(count[h]);
            incl[h] = base + wave_incl_scan(items[h]);
            base = lane_word(incl[h], 63);
        }
        total = base;
    }
    // Item i < total: where its list begins (the first one whose items reach
    // past i), the values it holds and where they lie.
    __device__ __forceinline__ void item(uint32_t i, uint64_t &at, uint32_t &n, uint64_t &list) const
    {
        const uint64_t a = __ballot(incl[0] > i), b = __ballot(incl[1] > i);
        const uint32_t l = (uint32_t)__builtin_ctzll(a ? a : b);
        list = a ? lane_word(begin[0], l) : lane_word(begin[1], l);
        const uint64_t cnt = a ? lane_word(count[0], l) : lane_word(count[1], l);
        const uint32_t first = a ? lane_word(incl[0] - items[0], l) : lane_word(incl[1] - items[1], l);
        at = list + 64ull * (i - first);
        n = merkle_item_values(cnt, i - first);
    }
};

// Room for the items of any job: the most groups a job may have, their first
// level done, in lists that each end in a partial item.
constexpr int kMerkleItems = 4352;
// Every root of a job in the argument tables, by one workgroup of NT lanes:
// its wavefronts share the items of all lists (four in flight each), then the
// lists themselves, then wavefront 0 takes the session's.  Lists one after
// another, each behind barriers, took 17 us for a step's sixteen.  ITEMS:
// room for the items' roots.  Ends with a barrier.
template <int NT, int ITEMS>
__device__ void merkle_args(const ArgTables &tab, uint32_t tiles, const uint64_t *in, bool pre)
{
    constexpr uint32_t NW = NT / 64;
    __shared__ uint64_t part[ITEMS];
    __shared__ uint64_t roots[kArgBufs];
    const uint32_t t = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(t >> 6), lane = t & 63;
    const ArgItems it(tab, tiles, pre);
    for (uint32_t i0 = wave; i0 < it.total; i0 += 4 * NW) {
        uint64_t v[4];
        uint32_t n[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            n[u] = 0;
            v[u] = 0;
            if (i0 + u * NW < it.total) {
                uint64_t at, list;
                it.item(i0 + u * NW, at, n[u], list);
                if (lane < n[u]) v[u] = in[at + lane];
            }
        }
        __builtin_amdgcn_sched_barrier(0);
        const uint64_t r = wave_merkle4(v, n[0], n[1], n[2], n[3]);
        if (lane < 4 && i0 + lane * NW < it.total) part[i0 + lane * NW] = r;
    }
    __syncthreads();
    for (uint32_t b = wave; b < tab.nbuf; b += NW) {
        const uint32_t l = b & 63;
        uint32_t n = b < 64 ? lane_word(it.items[0], l) : lane_word(it.items[1], l);
        const uint64_t *p = part + (b < 64 ? lane_word(it.incl[0], l) : lane_word(it.incl[1], l)) - n;
        uint64_t v = empty_hash();
        if (ITEMS < kMerkleItems || n <= 64) {  // (the callers with less room have lists of at most 64 items)
            if (lane < n) v = p[lane];
        } else {  // a buffer of more than 64 GiB
            const uint32_t nb = merkle_items(n);
            for (uint32_t k = 0; k < nb; ++k) {
                const uint32_t c = merkle_item_values(n, k);
                const uint64_t r = lane_word(wave_merkle<1, 6>(lane < c ? p[64 * k + lane] : 0, c), 0);
                if (lane == k) v = r;
            }
            n = nb;
        }
        v = wave_merkle<1, 6>(v, n);
        if (lane == 0) {
            roots[b] = v;
            if (tab.root[0]) ((g_u64 *)tab.root[0])[b] = v;
            if (tab.root[1]) ((g_u64 *)tab.root[1])[b] = v;
        }
    }
    __syncthreads();
    if (wave == 0 && (tab.sroot[0] || tab.sroot[1])) {
        const uint32_t n = tab.nbuf;
        uint64_t v = n == 0 ? empty_hash() : wave_merkle<1, 6>(lane < n ? roots[lane] : 0, min(n, 64u));
        if (n > 64) v = node_hash(v, wave_merkle<1, 6>(64 + lane < n ? roots[64 + lane] : 0, n - 64));
        if (lane == 0) {
            if (tab.sroot[0]) *(g_u64 *)tab.sroot[0] = v;
            if (tab.sroot[1]) *(g_u64 *)tab.sroot[1] = v;
        }
    }
    __syncthreads();
}

__global__ __launch_bounds__(1024) void k_merkle_args(const ArgTables tab, uint32_t tiles,
                                                      const uint64_t *__restrict__ in, bool pre)
{
    merkle_args<1024, kMerkleItems>(tab, tiles, in, pre);
}

// Grid-wide first level of a job's lists: wavefront w reduces item w into
// out[begin + block], where the list's values then start.
__global__ __launch_bounds__(256) void k_merkle_items(const ArgTables tab, uint32_t tiles,
                                                      const uint64_t *__restrict__ in, uint64_t *__restrict__ out)
{
    const ArgItems it(tab, tiles, false);
    const uint32_t w = __builtin_amdgcn_readfirstlane(blockIdx.x * 4 + (threadIdx.x >> 6)), lane = threadIdx.x & 63;
    if (w >= it.total) return;
    uint64_t at, list;
    uint32_t n;
    it.item(w, at, n, list);
    const uint64_t r = wave_merkle<1, 6>(lane < n ? in[at + lane] : 0, n);
    if (lane == 0) out[list + (at - list) / 64] = r;
}

// Grid-wide first level of long Merkle lists (LongLists): wavefront w
// reduces aligned 64-value block w - block_begin[j] of list j into
// sa[begin[j] + block], where the list's own reduction would have put it.
__global__ __launch_bounds__(256) void k_merkle_blocks(const LongLists L, const uint64_t *__restrict__ in,
                                                       uint64_t *__restrict__ sa)
{
    const uint64_t w = (uint64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    const uint32_t lane = threadIdx.x & 63;
    if (w >= L.block_begin[L.n]) return;
    uint32_t j = 0;
    while (j + 1 < L.n && L.block_begin[j + 1] <= w) ++j;
    const uint64_t blk = w - L.block_begin[j];
    const uint32_t cnt = (uint32_t)umin(64, L.count[j] - 64 * blk);
    const uint64_t v = lane < cnt ? in[L.begin[j] + 64 * blk + lane] : 0;
    const uint64_t r = wave_merkle<1, 6>(v, cnt);
    if (lane == 0) sa[L.begin[j] + blk] = r;
}

// ---------------------------------------------------------------- copies

// Copy tile kernel: one workgroup moves one tile of CPW chunks (a 64-chunk
// group, or an eighth of one in small jobs), SL bytes of every chunk per
// step, with coalesced 16-byte loads and stores: the fused kernel's tile
// without the hash and the LDS staging, in a shape of its own (512 lanes and
// 1 KiB slices for whole groups, measured faster for copies than the fused
// kernel's 1024 lanes and 512-byte slices).
//   PACK:    the buffer's bytes -> the chunk slots of the snapshot; a partial
//            last chunk is zero-padded to the end of its slot.
//   !PACK:   the chunk slots (contiguous, or per chunk through a manifest of
//            arena offsets) -> the destination buffer; only logical
//            bytes are written.
template <class Tab, bool PACK, int T, int SL, int CPW>
__global__ __launch_bounds__(T) void k_copy(const Tab tab, uint64_t arena_base, bool wb)
{
    constexpr uint32_t kSteps = kChunk / SL, LPS = SL / 16;
    constexpr int U = CPW * SL / 16 / T;
    constexpr uint32_t kTiles = kGroupChunks / CPW;
    static_assert(U >= 1 && T % LPS == 0 && kGroupChunks % CPW == 0, "tile shape");
    __shared__ ChunkLoc cloc[CPW];
    __shared__ TileInfo info;
    const uint32_t tile_id = xcd_tile();
    const uint32_t t = threadIdx.x;
    tile_setup<PACK ? kModePack : kModeVerify, CPW>(tab, tile_id / kTiles, tile_id % kTiles, arena_base, &info, cloc);
    if (__builtin_amdgcn_readfirstlane(info.nv) == 0) return;  // a buffer's last group may end before this tile
    const uint32_t slot = (t % LPS) * 16;
    if (__builtin_amdgcn_readfirstlane(info.many)) {
        // A tile with a chunk of more than two pieces (see hash_tile).
        static_assert(T % (kChunk / 16) == 0, "a lane's granules lie at the same place of their chunks");
        const uint32_t x = t % (kChunk / 16) * 16, nv = info.nv;
        const bool ragged = __builtin_amdgcn_readfirstlane(info.ragged);
#pragma unroll 1
        for (uint32_t g = t; g < CPW * (kChunk / 16); g += U * T) {
            uint64_t at[U];
            uint32_t clen[U];
            uint4 v[U];
#pragma unroll
            for (int k = 0; k < U; ++k) {
                const uint32_t c = (g + k * T) / (kChunk / 16);
                const ChunkLoc &l = cloc[c];
                at[k] = PACK ? granule_at(info, l, c, x) : l.slot + x;
                clen[k] = PACK ? l.len : (l.len + 15) & ~15u;  // slots are whole 4096-byte granules
            }
            load_granules<U>(at, clen, x, PACK && ragged, v);
            asm volatile("" ::: "memory");
#pragma unroll
            for (int k = 0; k < U; ++k) {
                const uint32_t c = (g + k * T) / (kChunk / 16);
                const ChunkLoc &l = cloc[c];
                if (PACK) {
                    if (c >= nv) continue;
                    if (wb) store16(l.slot + x, v[k]);
                    else store16_nt(l.slot + x, v[k]);
                } else if (x < l.len) {
                    const uint64_t to = granule_at(info, l, c, x);
                    if (x + 16 <= l.len) store16_nt(to, v[k]);
                    else store_partial(to, v[k], l.len - x);
                }
            }
        }
        return;
    }
    uint64_t ra[U], rb[U], sa[U];
    uint32_t rs[U], gl[U];
#pragma unroll
    for (int k = 0; k < U; ++k) {
        const ChunkLoc l = cloc[(k * T + t) / LPS];
        ra[k] = l.a1;
        rb[k] = l.a2;
        rs[k] = l.split;
        gl[k] = l.len;
        sa[k] = l.slot;
    }
    auto piece_addr = [&](int k, uint32_t x) -> uint64_t { return (x < rs[k] ? ra[k] : rb[k]) + x; };
    // The lanes move the tile in lockstep steps (a barrier per step); the
    // next step's loads are issued before this step's stores.  Chunk c moves
    // its slices in an order rotated by c and the tile index, so that a
    // step's accesses cover every offset within a chunk instead of one (all
    // tiles touching the same offsets at once loads the HBM channels
    // unevenly): restores of flat buffers are 3-8% faster with the rotation,
    // the 1024-session batch 1.5% slower.
    uint4 v[U], n[U];
    auto off = [&](int k, uint32_t step) -> uint32_t {
        const uint32_t c = (k * T + t) / LPS;
        return ((step + c + tile_id) % kSteps) * SL + slot;
    };
    const bool ragged = __builtin_amdgcn_readfirstlane(info.ragged);
    // Whole granules first, as load_granules (each chunk at its own offset).
    const auto load = [&](uint4 (&v)[U], uint32_t step) {
#pragma unroll
        for (int k = 0; k < U; ++k) {
            const uint32_t x = off(k, step);
            v[k] = make_uint4(0, 0, 0, 0);
            if (PACK ? x + 16 <= gl[k] : x < gl[k])  // slots are whole 4096-byte granules
                v[k] = load16_nt(PACK ? piece_addr(k, x) : sa[k] + x);
        }
        if (PACK && ragged) {
#pragma unroll
            for (int k = 0; k < U; ++k) {
                const uint32_t x = off(k, step);
                if (x < gl[k] && x + 16 > gl[k]) v[k] = load_partial(piece_addr(k, x), gl[k] - x);
            }
        }
    };
    load(v, 0);
    for (uint32_t step = 0; step < kSteps; ++step) {
        wait_loads();
        if (step + 1 < kSteps) load(n, step + 1);
#pragma unroll
        for (int k = 0; k < U; ++k) {
            const uint32_t x = off(k, step);
            if (PACK) {  // wb: write-back stores (jobs within kPackWriteBackMaxRounds)
                if (sa[k]) {
                    if (wb) store16(sa[k] + x, v[k]);
                    else store16_nt(sa[k] + x, v[k]);
                }
            } else if (x < gl[k]) {
                if (x + 16 <= gl[k]) store16_nt(piece_addr(k, x), v[k]);
                else store_partial(piece_addr(k, x), v[k], gl[k] - x);
            }
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < U; ++k) v[k] = n[k];
    }
}

// ---------------------------------------------------------------- incremental

// A scan's entry j: the number of set bits of the 64-bit dirty mask of
// group j of an incremental checkpoint.
struct MaskBits {
    const uint64_t *p;
    __device__ uint64_t operator()(uint64_t j) const { return (uint64_t)__popcll(p[j]); }
};

// Exclusive scan of n counts (one workgroup; Hillis-Steele over 1024
// per-thread partial sums).  Writes offsets[] and *total; returns nothing
// else.  `offsets` may be LDS or global memory.
template <class Count>
__device__ void scan_counts(const Count counts, uint64_t n, uint64_t *offsets, uint64_t *total,
                            uint64_t (*sums)[1024])
{
    const uint32_t t = threadIdx.x;
    const uint64_t per = (n + 1023) / 1024;
    const uint64_t s0 = umin(n, t * per), s1 = umin(n, s0 + per);
    uint64_t s = 0;
    for (uint64_t j = s0; j < s1; ++j) s += counts(j);
    int cur = 0;
    sums[0][t] = s;
    __syncthreads();
    for (uint32_t d = 1; d < 1024; d <<= 1) {
        const uint64_t v = sums[cur][t] + (t >= d ? sums[cur][t - d] : 0);
        sums[cur ^ 1][t] = v;
        cur ^= 1;
        __syncthreads();
    }
    uint64_t run = sums[cur][t] - s;  // exclusive prefix of this thread's segment
    for (uint64_t j = s0; j < s1; ++j) {
        offsets[j] = run;
        run += counts(j);
    }
    if (t == 1023) *total = sums[cur][t];
    __syncthreads();
}

// Thread 1023 of a scan of dirty masks, once the stored-chunk count is
// known: takes this call's payload top from the bump word (bump_now, loaded
// when the kernel started; or sb.reset), writes it lowered by the count's
// slots to the next call's bump word, then publishes the count and the top
// to the host words.  Returns the top (0 when sb.bump is null: the host
// sets the top itself once it has read the count).
__device__ uint64_t place_slots(const SlotBump &sb, uint64_t count, uint64_t bump_now)
{
    uint64_t top = 0;
    if (sb.bump) {
        top = sb.reset ? sb.reset : bump_now;
        *sb.bump_out = top - count * kChunk;
        *sb.top_out = top;
    }
    if (sb.host) {
        ((volatile uint64_t *)sb.host)[0] = count;
        ((volatile uint64_t *)sb.host)[1] = top;
        __threadfence_system();
    }
    return top;
}

// Exclusive scan of counts (offsets and total); for the dirty masks of an
// incremental checkpoint also the placement of its slots (place_slots).
template <class Count>
__global__ __launch_bounds__(1024) void k_scan(const Count counts, uint64_t n, uint64_t *__restrict__ offsets,
                                               uint64_t *__restrict__ total, const SlotBump sb)
{
    __shared__ uint64_t sums[2][1024];
    const uint64_t bump_now = threadIdx.x == 1023 && sb.bump && !sb.reset ? *sb.bump : 0;
    scan_counts(counts, n, offsets, total, sums);
    if (threadIdx.x == 1023) place_slots(sb, *total, bump_now);
}

// Exclusive scan of the dirty masks' set bits of a small incremental job
// (at most kScanCompactMaxGroups groups): thread t holds the masks of groups
// 4t .. 4t+3 (0 past the job), loaded when the kernel started; DPP
// wavefront scans, then one over the 16 wavefront totals (counts stay below
// 2^32).  Writes offsets[] (LDS or global) and returns the total in every
// thread.  Ends with a barrier.
__device__ __forceinline__ uint64_t scan_masks_small(const uint64_t (&mk)[4], uint64_t ngroups, uint64_t *offsets, uint32_t *wsum)
{
    const uint32_t t = threadIdx.x, wave = t >> 6, lane = t & 63;
    uint32_t c[4], sum = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        c[k] = (uint32_t)__popcll(mk[k]);
        sum += c[k];
    }
    const uint32_t incl = wave_incl_scan(sum);
    if (lane == 63) wsum[wave] = incl;
    __syncthreads();
    if (wave == 0) {
        const uint32_t w = lane < 16 ? wsum[lane] : 0;
        const uint32_t wi = wave_incl_scan(w);
        if (lane < 16) wsum[16 + lane] = wi - w;
        if (lane == 15) wsum[32] = wi;
    }
    __syncthreads();
    uint64_t run = incl - sum + wsum[16 + wave];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        if (4 * t + k < ngroups) offsets[4 * t + k] = run;
        run += c[k];
    }
    const uint64_t total = wsum[32];
    __syncthreads();
    return total;
}

// Moves chunk i of a buffer (its logical bytes, zero-padded to 4096) to
// device address dst: the 64 lanes of a wavefront, 64 bytes each, four
// 16-byte loads in flight per lane.
__device__ __forceinline__ void copy_chunk(const Geom &g, uint64_t i, uint64_t dst, uint32_t lane)
{
    const uint64_t cb = i * kChunk;
    const uint64_t len = umin(kChunk, g.nbytes - cb);
    uint4 v[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const uint32_t x = (k * 64 + lane) * 16;
        v[k] = make_uint4(0, 0, 0, 0);
        if (x < len) {
            const uint64_t a = locate(g, cb + x).addr;
            v[k] = x + 16 <= len ? load16(a) : load_partial(a, (uint32_t)(len - x));
        }
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) store16(dst + (k * 64 + lane) * 16, v[k]);
}

// Small incremental jobs (tables in the kernel arguments, at most
// kScanCompactMaxGroups groups), after the fingerprint + diff tiles, in one
// launch of 1024-lane workgroups that need nothing from one another.
// Workgroup 0 reduces the Merkle lists (buffer and session roots), scans
// the dirty masks' set bits and publishes the stored-chunk count and the
// payload top (place_slots: *total, the next call's bump word, the host
// words).  Every other workgroup scans the masks itself (at most 4096
// words, the same for all, so mostly from L2) into LDS and takes the top
// from *bump.bump, which only an earlier launch wrote; its wavefront w
// then stores slots w, w + stride, ...: slot s belongs to the last group
// whose exclusive offset is at most s (a group with no dirty chunk shares
// its offset with the next group, so the last such group holds s), and
// within it to the dirty chunk with s - offset dirty chunks below it.
// Slots therefore follow (buffer, chunk) order, as k_place_dirty assigns
// them.  Lane 0 enters the slot in the manifest (clean chunks' entries
// were written by the diff tiles) and the wavefront copies the chunk.
__global__ __launch_bounds__(1024) void k_merkle_scan_place(const ArgTables tab, uint32_t tiles,
                                                            const uint64_t *__restrict__ nodes, uint64_t ngroups,
                                                            const uint64_t *__restrict__ dirty_mask,
                                                            const SlotBump bump, uint64_t *__restrict__ total,
                                                            uint64_t arena_base)
{
    __shared__ uint64_t offs[kScanCompactMaxGroups];
    __shared__ uint64_t msk[kScanCompactMaxGroups];
    __shared__ uint32_t wsum[33];
    static_assert(kScanCompactMaxGroups <= 4 * 1024, "four dirty masks per thread");
    const uint32_t t = threadIdx.x;
    uint64_t mk[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) mk[k] = 4 * t + k < ngroups ? dirty_mask[4 * t + k] : 0;
    const uint64_t top = !bump.bump ? 0 : bump.reset ? bump.reset : *bump.bump;
    if (blockIdx.x == 0) {
        // The masks' round trip to memory overlaps the Merkle reduction.
        merkle_args<1024, kScanCompactMaxGroups / 64 + kArgBufs>(tab, tiles, nodes, false);
        const uint64_t count = scan_masks_small(mk, ngroups, offs, wsum);
        if (t == 0) *total = count;
        if (t == 1023) place_slots(bump, count, top);
        return;
    }
#pragma unroll
    for (int k = 0; k < 4; ++k)
        if (4 * t + k < ngroups) msk[4 * t + k] = mk[k];
    const ArgLanes lanes(tab);
    const uint64_t count = scan_masks_small(mk, ngroups, offs, wsum);  // ends with a barrier: msk is visible
    const uint32_t lane = t & 63;
    const uint64_t stride = (uint64_t)(gridDim.x - 1) * 16;
    for (uint64_t s = (uint64_t)(blockIdx.x - 1) * 16 + __builtin_amdgcn_readfirstlane(t >> 6); s < count; s += stride) {
        uint32_t lo = 0, hi = (uint32_t)ngroups;  // offs[lo] <= s (offs[0] = 0)
        while (hi - lo > 1) {
            const uint32_t mid = (lo + hi) >> 1;
            if (offs[mid] <= s) lo = mid; else hi = mid;
        }
        lo = __builtin_amdgcn_readfirstlane(lo);
        const uint64_t m = msk[lo];
        const uint32_t k = (uint32_t)(s - offs[lo]);
        const uint32_t below = (uint32_t)__popcll(lane ? m & ((1ULL << lane) - 1) : 0);
        const uint32_t c = (uint32_t)__ffsll((unsigned long long)__ballot(((m >> lane) & 1) && below == k)) - 1;
        const uint32_t b = lanes.find(lo);
        const ArgBuf buf = lanes.buf(b);
        const uint64_t i = (uint64_t)(lo - buf.group_begin) * kGroupChunks + c;
        const uint64_t slot_off = top - (s + 1) * kChunk;  // arena offset
        if (lane == 0) ((g_u64 *)tab.manifest)[buf.chunk_begin + i] = slot_off;
        copy_chunk(lanes.geom(b, buf), i, arena_base + slot_off, lane);
    }
}

// The last group whose exclusive offset is at most s, for a whole wavefront
// (every lane gets it): 64 probes a step, so one to four steps.  Offsets do not
// decrease and begin at 0; a group without a dirty chunk shares its offset with
// the next group, so the group found holds slot s.
__device__ __forceinline__ uint32_t group_of_slot(const uint64_t *offsets, uint32_t ngroups, uint32_t s)
{
    uint32_t lo = 0, n = ngroups;
    while (n > 1) {
        const uint32_t step = (n + 63) / 64, d = (threadIdx.x & 63) * step;
        const uint64_t at_most = __ballot(d < n && offsets[lo + (d < n ? d : 0)] <= s);
        const uint32_t skip = (63 - (uint32_t)__builtin_clzll(at_most)) * step;
        lo += skip;
        n = min(step, n - skip);
    }
    return __builtin_amdgcn_readfirstlane(lo);
}

// Slot assignment and dirty copy in one launch (jobs with device tables,
// or whose slots the host placed, after the scan of the dirty masks).  The
// *total slots are dealt to the wavefronts in equal shares of consecutive
// slots, at most kPlaceShare at a time; a wavefront finds its share's first
// group by search and then walks the set bits from there (a clean group in
// between makes it search again).  Slots follow (buffer, chunk) order below the
// payload top in *top_word, as k_merkle_scan_place; lane 0 enters the slot in
// the manifest and all 64 lanes copy the chunk into it, 64 bytes per lane,
// zero-padding a partial chunk.  (The diff tiles entered the clean chunks.)
// Bound: the latency of a chunk's copy, about 2 us, times the chunks one
// wavefront takes, so what matters is an even deal; for large counts HBM.  A
// workgroup per group put appended state, whose dirty chunks fill a few groups,
// on a few workgroups: 391 chunks in seven groups of 200 to 400 took 32 us,
// now 8.7; a wavefront per chunk position, dirty or not, took 81 us for
// 131,072 positions of which 576 were dirty.  Whole checkpoints of 2 GiB, every
// chunk dirty, by share: 1 slot 1280 us (a search a chunk), 4 1157, 8 1144, an
// equal part of the whole 1188 (every wavefront at the same offset of its own
// 256 KiB), a workgroup per group 1199.
constexpr uint64_t kPlaceBlocks = 2048;
constexpr uint32_t kPlaceShare = 8;
template <class Tab>
__global__ __launch_bounds__(256) void k_place_dirty(const Tab tab, uint32_t ngroups, const uint64_t *__restrict__ dirty_mask,
                                                     const uint64_t *__restrict__ offsets,
                                                     const uint64_t *__restrict__ total,
                                                     const uint64_t *__restrict__ top_word, uint64_t arena_base)
{
    const uint32_t lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t waves = gridDim.x * 4, count = (uint32_t)*total;  // at most 2^30 chunks
    const uint32_t share = min((count + waves - 1) / waves, kPlaceShare);
    const uint64_t top = *top_word;  // arena offset
    for (uint64_t first = (uint64_t)(blockIdx.x * 4 + wave) * share; first < count; first += (uint64_t)waves * share) {
        const uint32_t end = (uint32_t)umin(first + share, count);
        uint32_t s = (uint32_t)first, G = group_of_slot(offsets, ngroups, s);
        uint64_t mask = dirty_mask[G];
        for (uint32_t below = s - (uint32_t)offsets[G]; below; --below) mask &= mask - 1;
        TileBuf b = tile_buf<kModeDiff, kGroupChunks>(tab, G);
        for (; s < end; ++s) {
            if (!mask) {
                mask = dirty_mask[++G];  // (slot s lies in a later group)
                if (!mask) {
                    G = group_of_slot(offsets, ngroups, s);
                    mask = dirty_mask[G];
                }
                b = tile_buf<kModeDiff, kGroupChunks>(tab, G);
            }
            const uint64_t i = (G - b.group_begin) * kGroupChunks + (uint64_t)__builtin_ctzll(mask);
            mask &= mask - 1;
            const uint64_t slot_off = top - ((uint64_t)s + 1) * kChunk;
            if (lane == 0) ((g_u64 *)b.manifest)[i] = slot_off;
            copy_chunk(b.g, i, arena_base + slot_off, lane);
        }
    }
}

// Copies n slots stored downwards from `top` into increasing order at dst
// (slot s -> dst + s*4096): the readable form of an incremental payload.
__global__ __launch_bounds__(256) void k_reverse_slots(uint64_t top, uint64_t dst, uint64_t n)
{
    const uint64_t s = blockIdx.x;
    if (s >= n) return;
    const uint32_t x = threadIdx.x * 16;
    store16(dst + s * kChunk + x, load16(top - (s + 1) * kChunk + x));
}

// ---------------------------------------------------------------- classify

// The chunks and groups of a buffer: group G's, and buffer b's.
struct ChunkRange {
    uint64_t nchunks, chunk_begin, group_begin;
};
__device__ __forceinline__ ChunkRange range_of(const JobBuf &b) { return ChunkRange{b.nchunks(), b.chunk_begin, b.group_begin}; }
__device__ __forceinline__ ChunkRange range_of(const ArgBuf &b)
{
    return ChunkRange{chunks_of(b.nbytes), b.chunk_begin, b.group_begin};
}
struct DevRanges {
    const DevTables &t;
    __device__ __forceinline__ explicit DevRanges(const DevTables &tab) : t(tab) {}
    __device__ __forceinline__ ChunkRange group(uint64_t G) const { return range_of(t.bufs[t.map[G]]); }
};
// (One buffer: its entry alone.  A wavefront classifies one word, so reading
// the whole table, 3 KB, is most of what it does: 8192 groups of one buffer
// 38.5 us with the table read, 37.0 without.)
struct ArgRange {
    const ArgTables &t;
    __device__ __forceinline__ explicit ArgRange(const ArgTables &tab) : t(tab) {}
    __device__ __forceinline__ ChunkRange group(uint64_t G) const
    {
        if (t.nbuf == 1) return range_of(t.bufs[0]);
        const ArgLanes lanes(t);
        return range_of(lanes.buf(lanes.find(G)));
    }
};
// The same for several words of a wavefront: the table is read once.
struct ArgRanges {
    ArgLanes lanes;
    __device__ __forceinline__ explicit ArgRanges(const ArgTables &tab) : lanes(tab) {}
    __device__ __forceinline__ ChunkRange group(uint64_t G) const { return range_of(lanes.buf(lanes.find(G))); }
};
__device__ __forceinline__ DevRanges ranges_of(const DevTables &t) { return DevRanges(t); }
__device__ __forceinline__ ArgRange ranges_of(const ArgTables &t) { return ArgRange(t); }

// Bitmap words g[0..U) (each one 64-chunk group of one buffer; g >= ngroups:
// none), computed by one wavefront: chunk i differs iff its K replay
// fingerprints are not all equal; the wave's ballot is the word.  The first
// kReplays fingerprints of every word are loaded before any is compared.
constexpr int kReplays = 4;
template <int U, class R>
__device__ __forceinline__ void classify_words(const R &ranges, const uint64_t (&g)[U], uint64_t ngroups, uint32_t lane,
                                               const uint64_t *hashes, uint32_t K, uint64_t total, uint64_t (&word)[U])
{
    const uint64_t *p[U];
    uint64_t h[U][kReplays];
    bool in[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        in[u] = false;
        p[u] = hashes;
        if (g[u] < ngroups) {
            const ChunkRange r = ranges.group(g[u]);
            const uint64_t i = (g[u] - r.group_begin) * kGroupChunks + lane;
            in[u] = i < r.nchunks;
            if (in[u]) p[u] = hashes + r.chunk_begin + i;
        }
#pragma unroll
        for (int k = 0; k < kReplays; ++k) h[u][k] = p[u][in[u] && k < (int)K ? k * total : 0];
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
        bool differs = false;
#pragma unroll
        for (int k = 1; k < kReplays; ++k) differs |= h[u][k] != h[u][0];
        for (uint32_t k0 = kReplays; k0 < K; k0 += kReplays) {
            uint64_t e[kReplays];
#pragma unroll
            for (int k = 0; k < kReplays; ++k) e[k] = p[u][in[u] ? min(k0 + k, K - 1) * total : 0];
#pragma unroll
            for (int k = 0; k < kReplays; ++k) differs |= e[k] != h[u][0];
        }
        word[u] = __ballot(in[u] && differs);
    }
}

// One wavefront per bitmap word.
template <class Tab>
__global__ __launch_bounds__(256) void k_classify(const Tab tab, uint64_t ngroups, const uint64_t *__restrict__ hashes,
                                                  uint32_t K, uint64_t total, uint64_t *__restrict__ bitmap)
{
    const uint64_t g[1] = {(uint64_t)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6)};
    if (g[0] >= ngroups) return;
    uint64_t word[1];
    classify_words<1>(ranges_of(tab), g, ngroups, threadIdx.x & 63, hashes, K, total, word);
    if ((threadIdx.x & 63) == 0) bitmap[g[0]] = word[0];
}

// Per buffer: 1 iff any of its bitmap words is non-zero (one wavefront per
// buffer, lanes striding over the words, eight loads in flight per lane; past the
// end they read the first word again).  One load at a time took 9.0 us for a
// buffer of 2048 groups, where a small job's table in the arguments had already
// cost the classification before it half a microsecond; now 2.6.
template <class Tab>
__global__ __launch_bounds__(64) void k_labels(const Tab tab, const uint64_t *__restrict__ bitmap,
                                               uint8_t *__restrict__ labels)
{
    const uint32_t b = blockIdx.x;
    const ChunkRange r = range_of(tab.bufs[b]);
    const uint64_t nw = (r.nchunks + kGroupChunks - 1) / kGroupChunks;
    const uint64_t *words = bitmap + r.group_begin;
    uint64_t any = 0;
    for (uint64_t w0 = threadIdx.x; w0 < nw; w0 += 512) {
        uint64_t v[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) v[k] = words[w0 + 64 * k < nw ? w0 + 64 * k : 0];
#pragma unroll
        for (int k = 0; k < 8; ++k) any |= v[k];
    }
    const bool set = __ballot(any != 0) != 0;
    if (threadIdx.x == 0) labels[b] = set ? 1 : 0;
}

// Small jobs (tables in the kernel arguments, at most kClassifyFusedGroups
// groups): the bitmap and the labels in one workgroup and one launch.
// Wavefront w computes words w, w + 16, ..., four at a time (also kept in
// LDS); after a barrier, one wavefront per buffer ORs its words into the
// buffer's label.
__global__ __launch_bounds__(1024) void k_classify_small(const ArgTables tab, uint64_t ngroups,
                                                         const uint64_t *__restrict__ hashes, uint32_t K,
                                                         uint64_t total, uint64_t *__restrict__ bitmap,
                                                         uint8_t *__restrict__ labels)
{
    __shared__ uint64_t words[kClassifyFusedGroups];
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const ArgRanges ranges(tab);
    for (uint64_t G = wave; G < ngroups; G += 64) {
        const uint64_t g[4] = {G, G + 16, G + 32, G + 48};
        uint64_t word[4];
        classify_words<4>(ranges, g, ngroups, lane, hashes, K, total, word);
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (lane == 0 && g[u] < ngroups) {
                bitmap[g[u]] = word[u];
                words[g[u]] = word[u];
            }
    }
    __syncthreads();
    for (uint32_t b = wave; b < tab.nbuf; b += 16) {
        const ChunkRange r = range_of(tab.bufs[b]);
        const uint64_t nw = (r.nchunks + kGroupChunks - 1) / kGroupChunks;
        uint64_t any = 0;
        for (uint64_t w = lane; w < nw; w += 64) any |= words[r.group_begin + w];
        const bool set = __ballot(any != 0) != 0;
        if (lane == 0) labels[b] = set ? 1 : 0;
    }
}

// Workgroup sizes (lanes) and slice bytes of the tile kernels, from
// measurement on MI355X.
// A pack tile's 80 registers let a CU hold one (16 wavefronts of six a SIMD)
// and take the next as soon as twelve of the last one's wavefronts have ended.
// (48 KB of LDS reserved beside the tile's own, meant to keep a second one
// out, only kept the next one from starting: packs with fingerprints of 90 /
// 200 MiB 45.9 / 83.3 us with it, 45.5 / 82.5 without, 1 / 2 GiB 347 / 678 -> 343 /
// 674.)
constexpr int kPackLanes = 1024, kPackSlice = 512;
// The staggered verified restore (jobs of 2-9 rounds) moves 1 KiB slices:
// 2-4% faster there than 512 B (the KV ring window 187 -> 182 us, flat
// 128-576 MiB within -4% .. +2%), while the staggered pack is 1-3% slower
// with them and keeps 512 B.
constexpr int kVerifyStaggerSlice = 1024;
// The fused pack of a job of at most this many rounds (one workgroup per CU)
// stores the snapshot through the caches (plain stores), a larger job past
// them (nontemporal stores).  Measured on MI355X in one process, alternating,
// with the loads nontemporal in both: pack + fingerprint of flat 64-127 MiB
// 15-21% faster, 128-576 MiB 3-10%, KV ring windows of 64-576 MiB 4-20%, and
// a checkpoint followed by a restore of it 3-17% faster per step (the
// restore also finds part of the snapshot still in the caches); the 512 MiB
// KV ring step (checkpoint, fork, two restores) 564 -> 551 us.  Above the
// bound write-back stops paying: the 1024-session batch 10.84 -> 11.40 ms
// and flat 1-4 GiB 3-4% slower in the same process.  Restores keep
// nontemporal stores whatever the size (plain ones: the KV ring restore 177
// -> 196 us, its verified restore 181 -> 196 us).
constexpr uint32_t kPackWriteBackMaxRounds = kStaggerMaxRounds;
constexpr int kHashLanes = 256, kHashSlice = 512;
constexpr int kCopyLanes = 512, kCopySlice = 1024;
// Fingerprint and diff tiles of jobs whose tables travel in the kernel
// arguments take 1024 lanes where that saves a round of tiles.  A CU holds two
// 1024-lane tiles (64 registers) or three 256-lane ones, whose round takes half
// as long again (26 us for 512 groups, 39 for 760, without the roots).  So wide tiles
// pay up to two tiles per CU (one round either way) and from three to four (two
// rounds either way); between, and from four on, they need a round more or
// gain nothing.  Fingerprint / incremental checkpoint, us, 1024 against 256
// lanes, one flat buffer, groups (256 CUs): 256 19.8 / 26.2 against 20.9 / 26.9; 512
// 30.9 / 37.8, 31.6 / 38.4; 513 38.0 / 45.8, 35.4 / 42.0; 760 45.3 / 52.4, 44.1 / 50.8;
// 840 49.2 / 56.5, 53.6 / 60.3; 1024 55.4 / 62.7, 57.7 / 63.8; 1100 64.3 / 73.2, 58.4 /
// 65.4; 1536 76.3 / 84.3, 75.2 / 81.7; 2048 96.3 / 105.7, 95.4 / 102.4.  20 buffers and
// ring windows draw the line at the same places, and so do 2 to 96 buffers of
// equal or mixed sizes: what a job of many buffers was thought to lose to its
// partial groups is the round begun at 513 groups.
// With device tables a tile's first access is a dependent load of its group-map
// entry, which three 256-lane tiles per CU hide and two 1024-lane tiles do not
// (a wrapping KV ring window: diff 115 -> 131 us, fingerprint 89 -> 106 us), so
// those keep 256 lanes.
inline bool wide_pays(uint64_t ngroups, uint32_t cus)
{
    return ngroups <= 2ull * cus || (ngroups > 3ull * cus && ngroups <= 4ull * cus);
}
constexpr int kSmallLanes = 256;  // sub-tiles of small jobs: 8 chunks per workgroup
// A sub-tile moves whole chunks in one step (8 granules per lane): a small
// job's time is a tile's latency, one load round trip per step.
constexpr int kSmallSlice = 4096;

// ---------------------------------------------------------------- bank shrink

// Total order on float32 relevance scores as unsigned keys: negative values
// reversed below the positive ones (-0.0 just below +0.0), every NaN above
// +inf.
__device__ __forceinline__ uint32_t score_key(uint32_t bits)
{
    if ((bits & 0x7F800000u) == 0x7F800000u && (bits & 0x007FFFFFu)) return 0xFFFFFFFFu;
    return (bits & 0x80000000u) ? ~bits : (bits | 0x80000000u);
}

// hist[b] += 1 for every lane of the wavefront with m set.  Lanes that share
// the first such lane's bucket are added with one atomic: ties, the common
// conflict, cost one LDS atomic per wavefront, not 64 serialised ones.
__device__ __forceinline__ void hist_add(uint32_t *hist, uint32_t b, bool m)
{
    const uint64_t act = __ballot(m);
    if (!act) return;
    const int leader = __builtin_ctzll(act);
    const uint32_t lb = (uint32_t)__builtin_amdgcn_readlane((int)b, leader);
    const bool same = m && b == lb;
    const uint64_t sm = __ballot(same);
    if ((int)(threadIdx.x & 63) == leader) atomicAdd(&hist[lb], (uint32_t)__popcll(sm));
    else if (m && !same) atomicAdd(&hist[b], 1u);
}

// Set bits of a wavefront mask in the lanes below this one.
__device__ __forceinline__ uint32_t lanes_below(uint64_t m)
{
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

// How a selection reads its n scores.  The array starts head = (address mod
// 16) / 4 scores past a 16-byte boundary; in the aligned view that starts
// there (group g = scores 4g - head .. 4g - head + 3), the whole groups
// [gf0, gf1) are read 16 bytes at a time, and the at most three scores before
// them, [0, e_lo), and after them, [e_hi, n), one at a time.
struct SelView {
    uint64_t base;  // address of score -head (16-byte aligned)
    uint64_t gf0, gf1, e_lo, e_hi;
    uint32_t head;
};
__device__ __forceinline__ SelView sel_view(uint64_t scores, uint32_t n)
{
    SelView v;
    v.head = (uint32_t)(scores & 15) / 4;
    v.base = scores - 4 * v.head;
    v.gf0 = v.head ? 1 : 0;
    const uint64_t g1 = ((uint64_t)n + v.head) / 4;
    v.gf1 = g1 > v.gf0 ? g1 : v.gf0;
    v.e_lo = umin(n, 4 * v.gf0 - v.head);
    const uint64_t hi = umin(n, 4 * v.gf1 - v.head);
    v.e_hi = hi > v.e_lo ? hi : v.e_lo;
    return v;
}
// Keys of U groups: group g0 + stride * u for u < U, or group end - 1 where
// that lies at or past `end` (ok[u] false; a valid address, its keys unused).  All U loads are issued before
// any key is formed (a scheduling barrier keeps the compiler from moving each
// load down to its first use, which would wait on them one at a time).
template <int U>
__device__ __forceinline__ void load_keys(const SelView &v, uint64_t g0, uint64_t stride, uint64_t end,
                                          uint32_t (&k)[U][4], bool (&ok)[U])
{
    v4u32 x[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const uint64_t g = g0 + stride * u;
        ok[u] = g < end;
        x[u] = *(const g_v4u32 *)(v.base + 16 * (ok[u] ? g : end - 1));
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
        for (int j = 0; j < 4; ++j) k[u][j] = score_key(x[u][j]);
}
// The single scores a selection reads one at a time (before and after the
// whole groups), one per lane of wavefront 0: lane l < 8 holds score l of
// [0, e_lo) ++ [e_hi, n).  `raw` is loaded at once; its key is formed later,
// so that the load overlaps others.
struct SelSingle {
    uint64_t i;
    bool in, head, tail;
    uint32_t raw;
};
__device__ __forceinline__ SelSingle sel_single(const SelView &v, uint64_t scores, uint32_t n, uint32_t lane,
                                                bool wave0)
{
    SelSingle s;
    s.i = lane < v.e_lo ? lane : v.e_hi + (lane - v.e_lo);
    s.in = wave0 && lane < 8 && s.i < n && (lane < v.e_lo || s.i >= v.e_hi);
    s.head = s.in && lane < v.e_lo;
    s.tail = s.in && lane >= v.e_lo;
    s.raw = 0;
    if (s.in) s.raw = ((const g_u32 *)scores)[s.i];
    return s;
}

// Counts of keys below and equal to K* among the single scores (head pair,
// tail pair); every lane of wavefront 0 gets them.
__device__ __forceinline__ void count_singles(const SelSingle &s, uint32_t key, uint32_t prefix, uint32_t (&c)[4])
{
    c[0] = (uint32_t)__popcll(__ballot(s.head && key < prefix));
    c[1] = (uint32_t)__popcll(__ballot(s.head && key == prefix));
    c[2] = (uint32_t)__popcll(__ballot(s.tail && key < prefix));
    c[3] = (uint32_t)__popcll(__ballot(s.tail && key == prefix));
}

// Writes the kept single scores, wavefront 0: lane order is index order
// within the head and the tail; (ph, rh) and (pt, rt) are the kept entries
// and K* keys before each.
__device__ __forceinline__ void place_singles(const SelSingle &s, uint32_t key, uint32_t prefix, uint32_t need,
                                              uint32_t ph, uint32_t rh, uint32_t pt, uint32_t rt,
                                              uint32_t *__restrict__ kept)
{
    const uint64_t eqh = __ballot(s.head && key == prefix), eqt = __ballot(s.tail && key == prefix);
    const uint32_t r = s.head ? rh + lanes_below(eqh) : rt + lanes_below(eqt);
    const bool take = s.in && (key < prefix || (key == prefix && r < need));
    const uint64_t th = __ballot(s.head && take), tt = __ballot(s.tail && take);
    if (take) kept[s.head ? ph + lanes_below(th) : pt + lanes_below(tt)] = (uint32_t)s.i;
}

// Writes the kept indices of one whole group per lane of a wavefront, in
// index order (lane by lane, score by score); every lane takes part
// (ballots).  The K* keys and kept entries before score j of a lane: those
// of the lanes below, then its own before j.  pos and rank (kept entries and
// K* keys before this wavefront's groups) advance, the same in every lane.
__device__ __forceinline__ void place_group(const uint32_t (&k)[4], bool ok, uint64_t g, uint32_t head,
                                            uint32_t prefix, uint32_t need, uint32_t &pos, uint32_t &rank,
                                            uint32_t *__restrict__ kept)
{
    uint64_t em[4], tm[4];
    uint32_t r = rank, take = 0, o = pos;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        em[j] = __ballot(ok && k[j] == prefix);
        r += lanes_below(em[j]);
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        if (!ok) continue;
        if (k[j] < prefix) take |= 1u << j;
        else if (k[j] == prefix && r++ < need) take |= 1u << j;
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        tm[j] = __ballot((take >> j) & 1);
        o += lanes_below(tm[j]);
    }
    const uint64_t e0 = 4 * g - head;
#pragma unroll
    for (int j = 0; j < 4; ++j)
        if ((take >> j) & 1) kept[o++] = (uint32_t)(e0 + j);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        rank += (uint32_t)__popcll(em[j]);
        pos += (uint32_t)__popcll(tm[j]);
    }
}

// Exclusive prefix of x over the NT threads (at most 1024) of a workgroup (ws: a
// word per wavefront): each wavefront scans the totals itself, behind one barrier.
template <int NT>
__device__ __forceinline__ uint32_t block_excl_scan(uint32_t x, uint32_t *ws)
{
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const uint32_t incl = wave_incl_scan(x);
    if (lane == 63) ws[wave] = incl;
    __syncthreads();
    const uint32_t w = wave_incl_scan(ws[lane & (NT / 64 - 1)]);  // (lanes past the wavefronts: unused)
    return incl - x + (wave ? lane_word(w, wave - 1) : 0);
}

// Selection of a bank of at most kSelectOneWorkgroupEntries scores in one
// workgroup of NT lanes (256 up to 1024 scores, else 1024): the `keep` best-ranked entries (a smaller key, or
// an equal key at a lower index, ranks first) in increasing index order.
//   0. A range of a multiple of 64 whole groups per wavefront;
//      each lane holds its R groups of its wavefront's range (the smallest R
//      of 1, 2, 4 and 8 that does), read once, all loads in flight.
//      The single scores before and after the whole groups
//      are ranges of their own, first and last, held by wavefront 0.
//   1. Radix select, most significant bits first: passes over the next 11, 11
//      and 10 bits histogram the candidates (LDS atomics, two copies of the
//      histogram beyond 4096 scores so that fewer wavefronts meet in one) and narrow to the
//      bucket that holds the keep-th smallest key (a prefix sum over the
//      buckets finds it), which ends as K*, with `need` = how many entries
//      with key K* are kept (those with the lowest indices).  Eight-bit
//      digits put most keys of a pass into a few buckets, whose LDS atomics
//      serialise.  A bucket that is kept whole ends the search: K* is then the
//      bucket's largest possible key, and every key equal to it is kept.
//   2. Each range counts its keys below K* and equal to K*; the counts of the
//      ranges before a range give the rank
//      of its first K* key, hence how many entries it keeps, and where its
//      kept indices go.
//   3. Each wavefront compacts its kept indices with ballots.
// Larger banks take the multi-workgroup selection (k_sel_*), which follows
// the same steps with a launch per pass.
// Measured (us a call, distinct scores / nearly all tied, so that every pass runs):
// 4.2 / 4.9 at 512, 4.2 / 5.2 at 1024, 5.3 / 7.2 at 3000, 8.0 / 11.8 at 8000, 22 / 36 at
// 30000.  Reading the scores anew in each of four 8-bit passes, one load in
// flight, took 14 / 18 and 41 / 57 at the last two.  1024 lanes at 512 scores: 4.9
// / 5.8, most of it barriers of sixteen wavefronts of which two hold scores, and
// 4.9 / 5.2 with four passes of 8 bits.  At 65536 (16 groups a lane) one workgroup
// takes 42, the five launches 40.
constexpr uint32_t kSelectOneWorkgroupEntries = 32768;
constexpr uint32_t kSelDigits = 2048;
template <int R, int NT>
__global__ __launch_bounds__(NT) void k_shrink_select(uint64_t scores, uint32_t n, uint32_t keep,
                                                        uint32_t *__restrict__ kept)
{
    // Per range: keys below K* (cnt[r]) and equal to K* (cnt[kRanges + r]);
    // range 0 = the single scores before the whole groups, 1 + w = wavefront
    // w's groups, the last = the single scores after.
    constexpr int kSelCopies = R > 1 ? 2 : 1;
    constexpr uint32_t kWaves = NT / 64, kRanges = kWaves + 2, kPer = kSelDigits / NT;
    __shared__ __attribute__((aligned(16))) uint32_t hist[kSelCopies][kSelDigits];
    __shared__ uint32_t cnt[2 * kRanges];
    __shared__ uint32_t ws[kWaves];
    __shared__ uint32_t pick[3];
    const uint32_t t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const SelView v = sel_view(scores, n);
    const uint64_t nfull = v.gf1 - v.gf0, per = (nfull + NT - 1) / NT * 64;  // at most 64 R
    const uint64_t w0 = v.gf0 + umin(wave * per, nfull), w1 = v.gf0 + umin(wave * per + per, nfull);
    const SelSingle es = sel_single(v, scores, n, lane, wave == 0);
    uint32_t rk[R][4];
    bool rok[R];
#pragma unroll
    for (int u = 0; u < R; ++u) {
        rok[u] = false;
#pragma unroll
        for (int j = 0; j < 4; ++j) rk[u][j] = 0;
    }
    if (w0 < w1) load_keys<R>(v, w0 + lane, 64, w1, rk, rok);
    const uint32_t ek = score_key(es.raw);
    uint32_t *const mine = hist[wave % kSelCopies];

    uint32_t prefix = 0, pmask = 0, need = keep;  // need: 1-based rank of K* among the candidates
    // Thread t's buckets are kPer t .. kPer t + kPer - 1; it clears them for the
    // next pass as it reads them.
#pragma unroll
    for (int c = 0; c < kSelCopies; ++c)
#pragma unroll
        for (uint32_t i = 0; i < kPer; ++i) hist[c][kPer * t + i] = 0;
    __syncthreads();
#pragma unroll 1
    for (int p = 0; p < 3; ++p) {
        const uint32_t shift = p == 0 ? 21 : p == 1 ? 10 : 0, digits = p == 2 ? kSelDigits / 2 : kSelDigits;
#pragma unroll
        for (int u = 0; u < R; ++u)
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (rok[u] && (rk[u][j] & pmask) == prefix) atomicAdd(&mine[(rk[u][j] >> shift) & (digits - 1)], 1u);
        if (es.in && (ek & pmask) == prefix) atomicAdd(&mine[(ek >> shift) & (digits - 1)], 1u);
        __syncthreads();
        uint32_t h[kPer], sum = 0;
#pragma unroll
        for (uint32_t i = 0; i < kPer; ++i) h[i] = 0;
#pragma unroll
        for (int c = 0; c < kSelCopies; ++c)
#pragma unroll
            for (uint32_t i = 0; i < kPer; ++i) {
                h[i] += hist[c][kPer * t + i];
                hist[c][kPer * t + i] = 0;
            }
#pragma unroll
        for (uint32_t i = 0; i < kPer; ++i) sum += h[i];
        uint32_t before = block_excl_scan<NT>(sum, ws);
        if (before < need && before + sum >= need) {
#pragma unroll
            for (uint32_t i = 0; i < kPer; ++i) {
                if (before < need && before + h[i] >= need) {
                    pick[0] = kPer * t + i;
                    pick[1] = need - before;
                    pick[2] = h[i];
                }
                before += h[i];
            }
        }
        __syncthreads();
        prefix |= pick[0] << shift;
        pmask |= (digits - 1) << shift;
        need = pick[1];
        if (need == pick[2]) {
            prefix |= ~pmask;
            need = n;
            break;
        }
    }

    // 2. Counts per range (wavefront totals, the same in every lane).
    uint32_t lt = 0, eq = 0;
#pragma unroll
    for (int u = 0; u < R; ++u)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            lt += (uint32_t)__popcll(__ballot(rok[u] && rk[u][j] < prefix));
            eq += (uint32_t)__popcll(__ballot(rok[u] && rk[u][j] == prefix));
        }
    if (lane == 0) {
        cnt[1 + wave] = lt;
        cnt[kRanges + 1 + wave] = eq;
    }
    if (wave == 0) {
        uint32_t c[4];
        count_singles(es, ek, prefix, c);
        if (lane == 0) {
            cnt[0] = c[0];
            cnt[kRanges] = c[1];
            cnt[kRanges - 1] = c[2];
            cnt[2 * kRanges - 1] = c[3];
        }
    }
    __syncthreads();

    // 3. Placement.  Kept entries (pos) and K* keys (rank) in the ranges
    // before range r:
    const auto range_start = [&](uint32_t r, uint32_t &pos, uint32_t &rank) {
        pos = rank = 0;
        for (uint32_t x = 0; x < r; ++x) {
            const uint32_t e = cnt[kRanges + x];
            pos += cnt[x] + (need > rank ? min(need - rank, e) : 0u);
            rank += e;
        }
    };
    if (wave == 0) {
        uint32_t ph, rh, pt, rt;
        range_start(0, ph, rh);
        range_start(kRanges - 1, pt, rt);
        place_singles(es, ek, prefix, need, ph, rh, pt, rt, kept);
    }
    uint32_t pos, rank;
    range_start(1 + wave, pos, rank);
#pragma unroll
    for (int u = 0; u < R; ++u) place_group(rk[u], rok[u], w0 + 64 * u + lane, v.head, prefix, need, pos, rank, kept);
}

// ---- multi-workgroup selection (banks of more than kSelectOneWorkgroupEntries
// scores), five launches: three histogram passes over the next 8, 12 and 12
// bits, k_sel_count and k_sel_place.  In each of the first four, the last
// workgroup to finish does what needs every workgroup's part: it finds the
// pass's bucket (the prefix of K* grows), or turns the ranges' counts into
// the places of their kept indices.  Bound: launches and the round trips to
// memory within each (the scores' own reads are under 1 us of 40 us at 48,000
// scores).  A launch per step (init, four 8-bit passes with a pick each,
// count, scan, place: twelve) took 64 us there, 350 us at 2^24 (now 141 us:
// five streams over the scores, at most 512 workgroups) and 1.7 ms at 2^28.
//
// The whole groups are cut into one range of a multiple of 64 groups per
// wavefront of the grid, read with 8 groups per lane in flight; range 0 and
// range R - 1 are the single scores, held by wavefront 0 of workgroup 0.
// The first pass counts into a histogram the caller keeps at zero (it and
// the tickets lie in the arena's first unit): its last workgroup clears it
// again, and clears the other passes' histogram, which lies in scratch.
constexpr uint32_t kSelBuckets = 4096;
struct SelState {
    uint32_t prefix, need, pad[2];
    uint32_t hist[kSelBuckets];  // passes 1 and 2
};
struct SelUnit {
    uint32_t ticket[kSelectTickets];
    uint32_t hist[kSelectFirstBuckets];
};
static_assert(sizeof(SelUnit) == kUnitSelectBytes, "selection words of the first unit");
constexpr int kSelU = 8;
__device__ __forceinline__ void sel_wave_range(const SelView &v, uint64_t gw, uint64_t nwaves, uint64_t &w0,
                                               uint64_t &w1)
{
    const uint64_t nfull = v.gf1 - v.gf0;
    const uint64_t per = (nfull + 64 * nwaves - 1) / (64 * nwaves) * 64;
    w0 = v.gf0 + umin(gw * per, nfull);
    w1 = v.gf0 + umin(gw * per + per, nfull);
}

// Pass P narrows K* by its bits [kShift, kShift + log2(kBuckets)).
template <int P>
__global__ __launch_bounds__(1024) void k_sel_hist(uint64_t scores, uint32_t n, uint32_t keep,
                                                   SelState *__restrict__ st, SelUnit *__restrict__ unit)
{
    constexpr uint32_t kBuckets = P == 0 ? kSelectFirstBuckets : kSelBuckets;
    constexpr uint32_t kShift = P == 0 ? 24 : P == 1 ? 12 : 0;
    constexpr uint32_t kAbove = P == 0 ? 0 : P == 1 ? 0xFF000000u : 0xFFFFF000u;  // bits already known
    __shared__ uint32_t hist[kBuckets];
    __shared__ uint32_t ws[16];
    __shared__ uint32_t flag;
    const uint32_t t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const SelView v = sel_view(scores, n);
    const uint32_t prefix = P == 0 ? 0 : st->prefix, need = P == 0 ? keep : st->need;
    for (uint32_t b = t; b < kBuckets; b += 1024) hist[b] = 0;
    __syncthreads();
    uint64_t w0, w1;
    sel_wave_range(v, (uint64_t)blockIdx.x * 16 + wave, (uint64_t)gridDim.x * 16, w0, w1);
    for (uint64_t g0 = w0; g0 < w1; g0 += 64ull * kSelU) {
        uint32_t k[kSelU][4];
        bool ok[kSelU];
        load_keys<kSelU>(v, g0 + lane, 64, w1, k, ok);
#pragma unroll
        for (int u = 0; u < kSelU; ++u)
#pragma unroll
            for (int j = 0; j < 4; ++j)
                hist_add(hist, (k[u][j] >> kShift) & (kBuckets - 1), ok[u] && (k[u][j] & kAbove) == prefix);
    }
    if (blockIdx.x == 0 && wave == 0) {
        const SelSingle es = sel_single(v, scores, n, lane, true);
        const uint32_t ek = score_key(es.raw);
        hist_add(hist, (ek >> kShift) & (kBuckets - 1), es.in && (ek & kAbove) == prefix);
    }
    __syncthreads();
    uint32_t *global = P == 0 ? unit->hist : st->hist;
    for (uint32_t b = t; b < kBuckets; b += 1024)
        if (hist[b]) atomicAdd(&global[b], hist[b]);
    if (!last_workgroup(&unit->ticket[P], gridDim.x, &flag)) return;
    // The bucket in which the running count first reaches `need`.
    constexpr uint32_t kPer = (kBuckets + 1023) / 1024;
    uint32_t h[kPer], sum = 0;
#pragma unroll
    for (uint32_t i = 0; i < kPer; ++i) {
        h[i] = t * kPer + i < kBuckets ? agent_load(&global[t * kPer + i]) : 0;
        sum += h[i];
    }
    uint32_t cum = block_excl_scan<1024>(sum, ws);
    if (cum < need && cum + sum >= need) {
        uint32_t i = 0;
#pragma unroll
        for (uint32_t k = 0; k + 1 < kPer; ++k)
            if (i == k && cum + h[k] < need) {
                cum += h[k];
                i = k + 1;
            }
        st->prefix = prefix | (t * kPer + i) << kShift;
        st->need = need - cum;
    }
    // Each thread clears what it read, for the next pass or call.
    if (P != 2)
        for (uint32_t i = 0; i < kPer; ++i)
            if (t * kPer + i < kBuckets) global[t * kPer + i] = 0;
    if (P == 0)
        for (uint32_t b = t; b < kSelBuckets; b += 1024) st->hist[b] = 0;
}

// Range r's keys below K* (lt[r]) and equal to K* (eq[r]); then, in the last
// workgroup, where each range starts: the kept entries before it (pos) are
// the keys below K* before it plus the first `need` K* keys, so pos =
// LT + min(need, EQ) and rank = EQ for the exclusive prefix sums LT and EQ of
// the counts.
__global__ __launch_bounds__(1024) void k_sel_count(uint64_t scores, uint32_t n, const SelState *__restrict__ st,
                                                    SelUnit *__restrict__ unit, uint32_t *__restrict__ lt_out,
                                                    uint32_t *__restrict__ eq_out, uint32_t *__restrict__ pos_out,
                                                    uint32_t *__restrict__ rank_out)
{
    __shared__ uint32_t ws[16];
    __shared__ uint32_t flag;
    const uint32_t t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const SelView v = sel_view(scores, n);
    const uint32_t prefix = st->prefix, need = st->need;
    const uint64_t gw = (uint64_t)blockIdx.x * 16 + wave, nwaves = (uint64_t)gridDim.x * 16;
    uint64_t w0, w1;
    sel_wave_range(v, gw, nwaves, w0, w1);
    uint32_t lt = 0, eq = 0;
    for (uint64_t g0 = w0; g0 < w1; g0 += 64ull * kSelU) {
        uint32_t k[kSelU][4];
        bool ok[kSelU];
        load_keys<kSelU>(v, g0 + lane, 64, w1, k, ok);
#pragma unroll
        for (int u = 0; u < kSelU; ++u)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                lt += (uint32_t)__popcll(__ballot(ok[u] && k[u][j] < prefix));
                eq += (uint32_t)__popcll(__ballot(ok[u] && k[u][j] == prefix));
            }
    }
    if (lane == 0) {
        agent_store(&lt_out[1 + gw], lt);
        agent_store(&eq_out[1 + gw], eq);
    }
    if (blockIdx.x == 0 && wave == 0) {
        const SelSingle es = sel_single(v, scores, n, lane, true);
        uint32_t c[4];
        count_singles(es, score_key(es.raw), prefix, c);
        if (lane == 0) {
            agent_store(&lt_out[0], c[0]);
            agent_store(&eq_out[0], c[1]);
            agent_store(&lt_out[nwaves + 1], c[2]);
            agent_store(&eq_out[nwaves + 1], c[3]);
        }
    }
    if (!last_workgroup(&unit->ticket[3], gridDim.x, &flag)) return;
    const uint32_t R = (uint32_t)nwaves + 2, per = (R + 1023) / 1024, s0 = min(t * per, R), s1 = min(s0 + per, R);
    uint32_t a = 0, b = 0;
    for (uint32_t r = s0; r < s1; ++r) {
        a += agent_load(&lt_out[r]);
        b += agent_load(&eq_out[r]);
    }
    uint32_t LT = block_excl_scan<1024>(a, ws);
    __syncthreads();
    uint32_t EQ = block_excl_scan<1024>(b, ws);
    for (uint32_t r = s0; r < s1; ++r) {
        pos_out[r] = LT + min(need, EQ);
        rank_out[r] = EQ;
        LT += agent_load(&lt_out[r]);
        EQ += agent_load(&eq_out[r]);
    }
}

__global__ __launch_bounds__(1024) void k_sel_place(uint64_t scores, uint32_t n, const SelState *__restrict__ st,
                                                    const uint32_t *__restrict__ pos_in,
                                                    const uint32_t *__restrict__ rank_in, uint32_t *__restrict__ kept)
{
    const uint32_t t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const SelView v = sel_view(scores, n);
    const uint32_t prefix = st->prefix, need = st->need;
    const uint64_t gw = (uint64_t)blockIdx.x * 16 + wave, nwaves = (uint64_t)gridDim.x * 16;
    if (blockIdx.x == 0 && wave == 0) {
        const SelSingle es = sel_single(v, scores, n, lane, true);
        place_singles(es, score_key(es.raw), prefix, need, pos_in[0], rank_in[0], pos_in[nwaves + 1],
                      rank_in[nwaves + 1], kept);
    }
    uint64_t w0, w1;
    sel_wave_range(v, gw, nwaves, w0, w1);
    uint32_t pos = pos_in[1 + gw], rank = rank_in[1 + gw];
    const uint32_t pos_end = pos_in[2 + gw];  // the next range's start
    for (uint64_t g0 = w0; g0 < w1 && pos < pos_end; g0 += 64ull * kSelU) {
        uint32_t k[kSelU][4];
        bool ok[kSelU];
        load_keys<kSelU>(v, g0 + lane, 64, w1, k, ok);
#pragma unroll
        for (int u = 0; u < kSelU; ++u) place_group(k[u], ok[u], g0 + 64ull * u + lane, v.head, prefix, need, pos, rank, kept);
    }
}

// Moves of a bank shrink, every part in one launch.  Kept indices increase,
// so kept[j] >= j, and in place the entries overwritten are the destinations
// j < keep.  A source kept[j] < keep (other than j itself) is such a
// destination, written by another item of the same pass: STAGE copies those
// sources to the part's staging area (slot j) first.  The place pass then
// writes destination j from the staging area, or straight from a source
// kept[j] >= keep, which no destination overwrites, and in place skips
// kept[j] == j (already there).  Out-of-place parts gather straight from the
// source and do nothing in the stage pass.
//
// Bound: HBM, 2 x kept bytes.  Each lane moves kMoveUnroll granules, all
// their indices loaded before the first granule and all granules before the
// first store, and short entries are laid end to end: one 256-lane workgroup
// per entry and one granule per lane left three lanes of four idle on a
// 1 KiB row, with one load in flight on the fourth: 24,000 rows of 16 such
// arrays (788 MB moved) 457 us, now 130 us.
template <int G>
struct Granule {
    uint64_t v;
};
template <>
struct Granule<16> {
    uint4 v;
};
template <int G>
__device__ __forceinline__ Granule<G> load_granule_nt(uint64_t a)
{
    Granule<G> r;
    if constexpr (G == 16) r.v = load16_nt(a);
    else if constexpr (G == 8) r.v = __builtin_nontemporal_load((const g_u64 *)a);
    else if constexpr (G == 4) r.v = *(const g_u32 *)a;
    else if constexpr (G == 2) r.v = *(const g_u16 *)a;
    else r.v = *(const g_u8 *)a;
    return r;
}
template <int G>
__device__ __forceinline__ void store_granule_nt(uint64_t a, const Granule<G> &r)
{
    if constexpr (G == 16) store16_nt(a, r.v);
    else if constexpr (G == 8) __builtin_nontemporal_store(r.v, (g_u64 *)a);
    else if constexpr (G == 4) *(g_u32 *)a = (uint32_t)r.v;
    else if constexpr (G == 2) *(g_u16 *)a = (uint16_t)r.v;
    else *(g_u8 *)a = (uint8_t)r.v;
}

// One work item: kMoveUnroll granules per lane.  first: the item's number
// within its part.
template <bool STAGE, int G>
__device__ __forceinline__ void move_item(const ShrinkPart &q, uint64_t first, const uint32_t *__restrict__ kept,
                                          uint64_t keep)
{
    const uint64_t gpe = q.eb / G, spe = move_slices(gpe);
    uint64_t j[kMoveUnroll], x[kMoveUnroll];
    bool ok[kMoveUnroll];
    if (spe) {
        const uint64_t e = first / spe, g0 = (first % spe) * kMoveItem;
#pragma unroll
        for (uint32_t u = 0; u < kMoveUnroll; ++u) {
            j[u] = e;
            x[u] = g0 + u * kMoveLanes + threadIdx.x;
            ok[u] = x[u] < gpe;
        }
    } else {
        // The item's first granule belongs to entry e0, at granule r0 of it;
        // r0 + an offset within the item stays far below 2^32.
        const uint64_t g0 = first * kMoveItem, e0 = g0 / gpe;
        const uint32_t r0 = (uint32_t)(g0 - e0 * gpe), per = (uint32_t)gpe;
#pragma unroll
        for (uint32_t u = 0; u < kMoveUnroll; ++u) {
            const uint32_t r = r0 + u * kMoveLanes + threadIdx.x, d = r / per;
            j[u] = e0 + d;
            x[u] = r - d * per;
            ok[u] = j[u] < keep;
        }
    }
    uint64_t e[kMoveUnroll];
#pragma unroll
    for (uint32_t u = 0; u < kMoveUnroll; ++u) e[u] = kept[ok[u] ? j[u] : 0];
    const bool in_place = q.stage != 0;
    uint64_t a[kMoveUnroll], d[kMoveUnroll];
#pragma unroll
    for (uint32_t u = 0; u < kMoveUnroll; ++u) {
        const bool staged = in_place && e[u] < keep;
        if (STAGE) ok[u] = ok[u] && staged && e[u] != j[u];
        else ok[u] = ok[u] && !(in_place && e[u] == j[u]);
        a[u] = (!STAGE && staged ? q.stage + j[u] * q.eb : q.src + e[u] * q.eb) + x[u] * G;
        d[u] = (STAGE ? q.stage : q.dst) + j[u] * q.eb + x[u] * G;
    }
    Granule<G> v[kMoveUnroll];
#pragma unroll
    for (uint32_t u = 0; u < kMoveUnroll; ++u)
        if (ok[u]) v[u] = load_granule_nt<G>(a[u]);
#pragma unroll
    for (uint32_t u = 0; u < kMoveUnroll; ++u)
        if (ok[u]) store_granule_nt<G>(d[u], v[u]);
}

template <bool STAGE>
__global__ __launch_bounds__(kMoveLanes) void k_move_entries(const ShrinkParts P, const uint32_t *__restrict__ kept,
                                                             uint64_t keep)
{
    // The part's index: the last one that begins at or before the item, by
    // one vector load of every part's begin (parts without items share the
    // begin of the next part and lose, parts past n never match).
    const uint64_t begin = P.item_begin[threadIdx.x & (kShrinkParts - 1)];
    for (uint64_t w = blockIdx.x; w < P.items; w += gridDim.x) {
        const uint32_t p = (uint32_t)__popcll(__ballot(begin <= w)) - 1;
        const ShrinkPart &q = P.p[p];
        const uint64_t first = w - P.item_begin[p];
        switch (q.gl) {
        case 4: move_item<STAGE, 16>(q, first, kept, keep); break;
        case 3: move_item<STAGE, 8>(q, first, kept, keep); break;
        case 2: move_item<STAGE, 4>(q, first, kept, keep); break;
        case 1: move_item<STAGE, 2>(q, first, kept, keep); break;
        default: move_item<STAGE, 1>(q, first, kept, keep); break;
        }
    }
}

// Clears n words (the tickets in the arena's first unit, before a context's
// first launch that takes any).
__global__ __launch_bounds__(256) void k_clear(uint64_t addr, uint32_t n)
{
    for (uint32_t i = threadIdx.x; i < n; i += 256) ((g_u32 *)addr)[i] = 0;
}

// Flips the lowest bit of one byte (the control of the discovery procedure
// gives a component a wrong value this way).
__global__ void k_flip_bit(uint64_t addr)
{
    if (threadIdx.x == 0) *(g_u8 *)addr ^= 1;
}

}  // namespace

// ---------------------------------------------------------------- launchers

hipError_t launch_stage(uint64_t host, uint64_t dev, uint64_t bytes, const JobBuf *host_bufs, uint32_t nbuf,
                        uint32_t *map, hipStream_t s)
{
    const uint64_t n16 = bytes / 16;
    const uint32_t copy_blocks = (uint32_t)((n16 + kStageUnits - 1) / kStageUnits);
    const uint32_t per = kStageLanes / 64, map_blocks = (nbuf + per - 1) / per;
    if (copy_blocks + map_blocks == 0) return hipSuccess;
    run_kernel(k_stage, dim3(copy_blocks + map_blocks), dim3(kStageLanes), s, host, dev, n16, copy_blocks, host_bufs,
               nbuf, map);
    return hipGetLastError();
}

template <class Tab>
hipError_t launch_tile(const Tab &tab, uint64_t ngroups, int mode, uint64_t *nodes, uint64_t *flag_mask,
                       uint64_t arena_base, hipStream_t s, uint32_t tiles_per_group, TileDevice dev)
{
    if (ngroups == 0) return hipSuccess;
    const bool split = tiles_per_group != 1;
    Stagger stg{0, 0};
    if (!split && (mode == kModePack || mode == kModeVerify) && dev.cus && dev.wall_khz &&
        ngroups >= (uint64_t)kStaggerMinRounds * dev.cus && ngroups <= (uint64_t)kStaggerMaxRounds * dev.cus)
        stg = Stagger{dev.cus, (uint32_t)((uint64_t)kStaggerPhaseNs * dev.wall_khz / 1000000)};
    const dim3 grid((uint32_t)(ngroups * tiles_per_group));
    if (tiles_per_group == kSmallTiles) {
        constexpr int kCPW = kGroupChunks / kSmallTiles;
        static_assert(kCPW == 8, "a sub-tile writes one mask byte");
        if (mode == kModeHash)
            run_kernel((k_hash<Tab, kModeHash, kSmallLanes, kSmallSlice, kCPW, false>), grid, dim3(kSmallLanes), s,
                       tab, nodes, flag_mask, arena_base);
        else if (mode == kModePack)  // sub-tile jobs are far within the write-back bound
            run_kernel((k_hash<Tab, kModePack, kSmallLanes, kSmallSlice, kCPW, true>), grid, dim3(kSmallLanes), s, tab,
                       nodes, flag_mask, arena_base);
        else if (mode == kModeDiff)
            run_kernel((k_hash<Tab, kModeDiff, kSmallLanes, kSmallSlice, kCPW, false>), grid, dim3(kSmallLanes), s,
                       tab, nodes, flag_mask, arena_base);
        else
            run_kernel((k_hash<Tab, kModeVerify, kSmallLanes, kSmallSlice, kCPW, false>), grid, dim3(kSmallLanes), s,
                       tab, nodes, flag_mask, arena_base);
        return hipGetLastError();
    }
    if (split) return hipErrorInvalidValue;
    constexpr bool kArgTab = std::is_same<Tab, ArgTables>::value;
    switch (mode) {
    case kModeHash:
        if (kArgTab && wide_pays(ngroups, dev.cus))
            run_kernel((k_hash<Tab, kModeHash, kPackLanes, kHashSlice, kGroupChunks, false>), grid, dim3(kPackLanes), s,
                       tab, nodes, flag_mask, arena_base);
        else
            run_kernel((k_hash<Tab, kModeHash, kHashLanes, kHashSlice, kGroupChunks, false>), grid, dim3(kHashLanes), s,
                       tab, nodes, flag_mask, arena_base);
        break;
    case kModePack:
        if (stg.ticks)
            run_kernel((k_hash_staggered<Tab, kModePack, kPackLanes, kPackSlice, kGroupChunks>), grid, dim3(kPackLanes), s,
                       tab, nodes, flag_mask, arena_base, stg);
        else if (ngroups <= (uint64_t)kPackWriteBackMaxRounds * std::max<uint32_t>(dev.cus, 1))
            run_kernel((k_hash<Tab, kModePack, kPackLanes, kPackSlice, kGroupChunks, true>), grid, dim3(kPackLanes), s, tab,
                       nodes, flag_mask, arena_base);
        else
            run_kernel((k_hash<Tab, kModePack, kPackLanes, kPackSlice, kGroupChunks, false>), grid, dim3(kPackLanes), s, tab,
                       nodes, flag_mask, arena_base);
        break;
    case kModeDiff:
        if (kArgTab && wide_pays(ngroups, dev.cus))
            run_kernel((k_hash<Tab, kModeDiff, kPackLanes, kHashSlice, kGroupChunks, false>), grid, dim3(kPackLanes), s,
                       tab, nodes, flag_mask, arena_base);
        else
            run_kernel((k_hash<Tab, kModeDiff, kHashLanes, kHashSlice, kGroupChunks, false>), grid, dim3(kHashLanes), s,
                       tab, nodes, flag_mask, arena_base);
        break;
    case kModeVerify:
        if (stg.ticks)
            run_kernel((k_hash_staggered<Tab, kModeVerify, kPackLanes, kVerifyStaggerSlice, kGroupChunks>), grid,
                       dim3(kPackLanes), s, tab, nodes, flag_mask, arena_base, stg);
        else
            run_kernel((k_hash<Tab, kModeVerify, kPackLanes, kPackSlice, kGroupChunks, false>), grid,
                       dim3(kPackLanes), s, tab, nodes, flag_mask, arena_base);
        break;
    default:
        return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

// Copies need no per-group output, so a small job is cut into sub-tiles here.
template <class Tab>
hipError_t launch_copy(const Tab &tab, uint64_t ngroups, bool pack, uint64_t arena_base, hipStream_t s, uint32_t cus)
{
    if (ngroups == 0) return hipSuccess;
    const uint32_t tiles = tile_split(ngroups);
    const dim3 grid((uint32_t)(ngroups * tiles));
    const bool wb = pack && ngroups <= (uint64_t)kPackWriteBackMaxRounds * cus;
    if (tiles == kSmallTiles) {
        constexpr int kCPW = kGroupChunks / kSmallTiles;
        if (pack)
            run_kernel((k_copy<Tab, true, kSmallLanes, kSmallSlice, kCPW>), grid, dim3(kSmallLanes), s, tab,
                       arena_base, wb);
        else
            run_kernel((k_copy<Tab, false, kSmallLanes, kSmallSlice, kCPW>), grid, dim3(kSmallLanes), s, tab,
                       arena_base, false);
    } else if (pack) {
        run_kernel((k_copy<Tab, true, kCopyLanes, kCopySlice, kGroupChunks>), grid, dim3(kCopyLanes), s, tab,
                   arena_base, wb);
    } else {
        run_kernel((k_copy<Tab, false, kCopyLanes, kCopySlice, kGroupChunks>), grid, dim3(kCopyLanes), s, tab,
                   arena_base, false);
    }
    return hipGetLastError();
}

template <class Tab>
hipError_t launch_place_dirty(const Tab &tab, uint64_t ngroups, const uint64_t *dirty_mask, const uint64_t *offsets,
                              const uint64_t *total, const uint64_t *top_word, uint64_t arena_base, hipStream_t s)
{
    if (ngroups == 0) return hipSuccess;
    // One wavefront a chunk if every chunk is dirty, up to kPlaceBlocks
    // workgroups (what the chip holds at once).
    const uint32_t blocks = (uint32_t)std::min<uint64_t>(ngroups * (kGroupChunks / 4), kPlaceBlocks);
    run_kernel((k_place_dirty<Tab>), dim3(blocks), dim3(256), s, tab, (uint32_t)ngroups, dirty_mask, offsets, total,
               top_word, arena_base);
    return hipGetLastError();
}

template <class Tab>
hipError_t launch_classify(const Tab &tab, uint64_t ngroups, const uint64_t *hashes, uint32_t K, uint64_t total,
                           uint64_t *bitmap, hipStream_t s)
{
    if (ngroups == 0) return hipSuccess;
    run_kernel((k_classify<Tab>), dim3((uint32_t)((ngroups + 3) / 4)), dim3(256), s, tab, ngroups, hashes, K, total, bitmap);
    return hipGetLastError();
}

template <class Tab>
hipError_t launch_labels(const Tab &tab, const uint64_t *bitmap, uint8_t *labels, hipStream_t s)
{
    if (tab.nbuf == 0) return hipSuccess;
    run_kernel((k_labels<Tab>), dim3(tab.nbuf), dim3(64), s, tab, bitmap, labels);
    return hipGetLastError();
}

hipError_t launch_classify_small(const ArgTables &tab, uint64_t ngroups, const uint64_t *hashes, uint32_t K,
                                 uint64_t total, uint64_t *bitmap, uint8_t *labels, hipStream_t s)
{
    if (ngroups > kClassifyFusedGroups) return hipErrorInvalidValue;
    if (tab.nbuf == 0) return hipSuccess;
    run_kernel(k_classify_small, dim3(1), dim3(1024), s, tab, ngroups, hashes, K, total, bitmap, labels);
    return hipGetLastError();
}

hipError_t launch_merkle(const MerkleList *lists, uint32_t nlists, const uint64_t *in,
                         uint64_t *scratch_a, uint64_t *scratch_b, uint64_t *roots_out,
                         uint64_t max_count, bool pre, hipStream_t s)
{
    if (nlists == 0) return hipSuccess;
    if (max_count > kMerkleLdsValues)
        run_kernel(k_merkle<1024>, dim3(nlists), dim3(1024), s, lists, in, scratch_a, scratch_b, roots_out, pre);
    else
        run_kernel(k_merkle<256>, dim3(nlists), dim3(256), s, lists, in, scratch_a, scratch_b, roots_out, pre);
    return hipGetLastError();
}

hipError_t launch_merkle_blocks(const LongLists &lists, const uint64_t *in, uint64_t *scratch_a, hipStream_t s)
{
    if (lists.n == 0 || lists.n > kLongLists) return lists.n ? hipErrorInvalidValue : hipSuccess;
    const uint64_t waves = lists.block_begin[lists.n];
    if (waves == 0) return hipSuccess;
    run_kernel(k_merkle_blocks, dim3((uint32_t)((waves + 3) / 4)), dim3(256), s, lists, in, scratch_a);
    return hipGetLastError();
}

hipError_t launch_merkle_args(const ArgTables &tab, uint32_t tiles, uint64_t nodes, const uint64_t *in,
                              uint64_t *scratch, bool first, hipStream_t s)
{
    const bool pre = nodes > kMerkleArgValues;
    if (first) {
        if (!pre) return hipSuccess;
        const uint64_t items = nodes / 64 + tab.nbuf;  // at least the lists' items
        run_kernel(k_merkle_items, dim3((uint32_t)((items + 3) / 4)), dim3(256), s, tab, tiles, in, scratch);
    } else {
        run_kernel(k_merkle_args, dim3(1), dim3(1024), s, tab, tiles, pre ? (const uint64_t *)scratch : in, pre);
    }
    return hipGetLastError();
}

hipError_t launch_scan(const uint64_t *dirty_mask, uint64_t n, uint64_t *offsets, uint64_t *total,
                       const SlotBump &bump, hipStream_t s)
{
    run_kernel(k_scan<MaskBits>, dim3(1), dim3(1024), s, MaskBits{dirty_mask}, n, offsets, total, bump);
    return hipGetLastError();
}

hipError_t launch_merkle_scan_place(const ArgTables &tab, uint32_t tiles, const uint64_t *nodes, uint64_t ngroups,
                                    const uint64_t *dirty_mask, const SlotBump &bump, uint64_t *total,
                                    uint64_t arena_base, hipStream_t s)
{
    if (ngroups > kScanCompactMaxGroups) return hipErrorInvalidValue;
    if (ngroups && (!bump.bump || !bump.bump_out || bump.bump == bump.bump_out)) return hipErrorInvalidValue;
    // Workgroup 0, then enough 16-wavefront workgroups for one stored chunk
    // per wavefront if every chunk is stored (at most kPlaceBlocks / 4).
    const uint64_t npos = ngroups * kGroupChunks;
    const uint32_t blocks = 1 + (uint32_t)std::min<uint64_t>((npos + 15) / 16, kPlaceBlocks / 4);
    run_kernel(k_merkle_scan_place, dim3(blocks), dim3(1024), s, tab, tiles, nodes, ngroups, dirty_mask, bump, total,
               arena_base);
    return hipGetLastError();
}

// Scratch of a multi-workgroup selection: SelState, then lt, eq, pos and
// rank arrays of R = 16 x workgroups + 2 ranges.
constexpr uint32_t kSelBlocks = 512;
static uint32_t select_blocks(uint32_t n)
{
    return std::max<uint32_t>(1, std::min<uint32_t>(n / 4096 + (n % 4096 != 0), kSelBlocks));
}
static uint64_t sel_array_bytes(uint32_t R) { return ((uint64_t)R * 4 + 255) / 256 * 256; }
static uint64_t sel_state_bytes() { return (sizeof(SelState) + 255) / 256 * 256; }

uint32_t select_steps(uint32_t n) { return n > kSelectOneWorkgroupEntries ? 5 : 1; }

uint64_t select_scratch_bytes(uint32_t n)
{
    if (n <= kSelectOneWorkgroupEntries) return 0;
    return sel_state_bytes() + 4 * sel_array_bytes(select_blocks(n) * 16 + 2);
}

hipError_t launch_shrink_select(const float *scores, uint32_t n, uint32_t keep, uint32_t *kept, uint64_t scratch,
                                uint64_t unit, uint32_t step, hipStream_t s)
{
    if (n == 0 || keep == 0) return hipSuccess;
    if (keep > n || step >= select_steps(n)) return hipErrorInvalidValue;
    if ((uint64_t)scores & 3) return hipErrorInvalidValue;
    const uint64_t sc = (uint64_t)scores;
    if (n <= kSelectOneWorkgroupEntries) {
        // R groups of four scores a lane.
        if (n <= 1024) run_kernel(k_shrink_select<1, 256>, dim3(1), dim3(256), s, sc, n, keep, kept);
        else if (n <= 4096) run_kernel(k_shrink_select<1, 1024>, dim3(1), dim3(1024), s, sc, n, keep, kept);
        else if (n <= 8192) run_kernel(k_shrink_select<2, 1024>, dim3(1), dim3(1024), s, sc, n, keep, kept);
        else if (n <= 16384) run_kernel(k_shrink_select<4, 1024>, dim3(1), dim3(1024), s, sc, n, keep, kept);
        else run_kernel(k_shrink_select<8, 1024>, dim3(1), dim3(1024), s, sc, n, keep, kept);
        return hipGetLastError();
    }
    if (!scratch || (scratch & 255) || !unit) return hipErrorInvalidValue;
    const uint32_t B = select_blocks(n), R = B * 16 + 2;
    SelState *st = (SelState *)scratch;
    SelUnit *su = (SelUnit *)unit;
    uint32_t *lt = (uint32_t *)(scratch + sel_state_bytes());
    uint32_t *eq = (uint32_t *)((uint64_t)lt + sel_array_bytes(R));
    uint32_t *pos = (uint32_t *)((uint64_t)eq + sel_array_bytes(R));
    uint32_t *rank = (uint32_t *)((uint64_t)pos + sel_array_bytes(R));
    switch (step) {
    case 0: run_kernel(k_sel_hist<0>, dim3(B), dim3(1024), s, sc, n, keep, st, su); break;
    case 1: run_kernel(k_sel_hist<1>, dim3(B), dim3(1024), s, sc, n, keep, st, su); break;
    case 2: run_kernel(k_sel_hist<2>, dim3(B), dim3(1024), s, sc, n, keep, st, su); break;
    case 3: run_kernel(k_sel_count, dim3(B), dim3(1024), s, sc, n, (const SelState *)st, su, lt, eq, pos, rank); break;
    default:
        run_kernel(k_sel_place, dim3(B), dim3(1024), s, sc, n, (const SelState *)st, (const uint32_t *)pos,
                   (const uint32_t *)rank, kept);
    }
    return hipGetLastError();
}

hipError_t launch_move_entries(const ShrinkParts &parts, const uint32_t *kept, uint64_t keep, bool stage,
                               hipStream_t s)
{
    if (parts.n > kShrinkParts) return hipErrorInvalidValue;
    if (parts.items == 0) return hipSuccess;
    const uint32_t grid = (uint32_t)std::min<uint64_t>(parts.items, 1u << 20);
    if (stage) run_kernel(k_move_entries<true>, dim3(grid), dim3(kMoveLanes), s, parts, kept, keep);
    else run_kernel(k_move_entries<false>, dim3(grid), dim3(kMoveLanes), s, parts, kept, keep);
    return hipGetLastError();
}

hipError_t launch_clear(uint64_t addr, uint32_t bytes, hipStream_t s)
{
    run_kernel(k_clear, dim3(1), dim3(256), s, addr, bytes / 4);
    return hipGetLastError();
}

hipError_t launch_flip_bit(uint64_t addr, hipStream_t s)
{
    run_kernel(k_flip_bit, dim3(1), dim3(64), s, addr);
    return hipGetLastError();
}

hipError_t launch_reverse_slots(uint64_t top, uint64_t dst, uint64_t n, hipStream_t s)
{
    if (n == 0) return hipSuccess;
    run_kernel(k_reverse_slots, dim3((uint32_t)n), dim3(256), s, top, dst, n);
    return hipGetLastError();
}

#define PCS_INSTANTIATE(Tab)                                                                                        \
    template hipError_t launch_tile<Tab>(const Tab &, uint64_t, int, uint64_t *, uint64_t *, uint64_t, hipStream_t, \
                                         uint32_t, TileDevice);                                                   \
    template hipError_t launch_copy<Tab>(const Tab &, uint64_t, bool, uint64_t, hipStream_t, uint32_t);           \
    template hipError_t launch_place_dirty<Tab>(const Tab &, uint64_t, const uint64_t *, const uint64_t *,        \
                                                const uint64_t *, const uint64_t *, uint64_t, hipStream_t);       \
    template hipError_t launch_classify<Tab>(const Tab &, uint64_t, const uint64_t *, uint32_t, uint64_t,         \
                                             uint64_t *, hipStream_t);                                            \
    template hipError_t launch_labels<Tab>(const Tab &, const uint64_t *, uint8_t *, hipStream_t);
PCS_INSTANTIATE(DevTables)
PCS_INSTANTIATE(ArgTables)
#undef PCS_INSTANTIATE

void set_kernel_events(hipEvent_t start, hipEvent_t stop)
{
    t_start = start;
    t_stop = stop;
    t_used = false;
}

bool take_kernel_events_used()
{
    const bool used = t_used;
    t_start = t_stop = nullptr;
    t_used = false;
    return used;
}

}  // namespace pcs
