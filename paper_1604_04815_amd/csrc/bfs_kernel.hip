// bfs_kernel.hip -- breadth-first search as a persistent grid of workgroups
// that talk to each other only through epoch-tagged flag words: the paper's
// inter-block hand-off (Section 4.3) used for the graph search it names as
// the next application of that hand-off (Section 6), in place of the atomic
// queue-tail counter that level-synchronous GPU searches usually use.
//
// One launch runs the whole search, level by level (top-down expansion):
//   * The frontier of a level is a queue of the vertices found at the level
//     before that have at least one edge, with the exclusive prefix of their
//     degrees beside it, so the level's edges have flat ranks 0 .. D - 1.
//     The ranks are cut into chunks of kBfsChunkEdges; chunk c is taken by
//     workgroup c mod B, in increasing c (the cyclic distribution of the
//     scan).  Every chunk has the same number of edges, however skewed the
//     degrees: a hub's edges spread over many chunks.
//   * Per chunk, the workgroup loads the frontier vertices its ranks fall in
//     (a table written while the frontier was built gives the first one) and
//     maps each rank to its vertex by counting heads in LDS (map_ranks).
//   * What is found goes one of three ways, by the level's edges D:
//     - D >= kBfsWideEdges and D >= V / 4 (wide_level): endpoints are marked
//       with plain byte stores and the next frontier is gathered by a sweep
//       over the marks, the workgroups' counts handed forward through flag
//       words.  Bound by random reads of the marks: on an R-MAT graph of 2^22
//       vertices and 2^27 column entries the largest level (109 M edges) takes
//       450 us, 240 G edges/s, against 65 G edges/s for the chunks below (a
//       probe reads random words of a 4 MiB array at 250 G/s and makes 27 G
//       atomics/s at any scope).  Neither bits set by atomics (1040 us: every
//       atomic takes the line from eight L2s) nor one map of marks per XCD
//       (456 us, and eight times the sweep) did better.
//     - D <= kBfsChunkEdges (solo_levels): workgroup 0 runs the level alone,
//       and the small ones after it, with the frontier in LDS: 2.3 us a level
//       on a path of single vertices, against 6.9 us with chunks and a grid
//       barrier per level.
//     - otherwise, chunk by chunk: every endpoint not yet found is claimed by
//       an atomic or on its mark; the chunk's winners are staged in LDS (one
//       discovery per edge at most, so they always fit), it publishes
//       (vertices, edges) packed in one 64-bit value in its flag words at
//       once, obtains its offsets from its own previous chunk's running total
//       and the values of the chunks in between (the window fold of the
//       scan), and writes its vertices, their edge offsets and the next
//       level's chunk table there.  No shared tail counter.  Up to 2^20 edges
//       this is as fast as a sweep and its extra barrier (R-MAT 2^18, 0.9 M
//       edges: 16-24 us).
//   * A level (or run of solo levels) ends with a grid barrier built from the
//     same flag words: each workgroup publishes its sums under the level's
//     tag, workgroup 0 adds them up and publishes the totals, which every
//     workgroup waits for.  The next frontier's writes are released before
//     the arrival and acquired after the release word, at agent scope.  One
//     workgroup of 1024 threads per CU: a barrier, a window and a sweep then
//     have 256 members (four of 256 threads: R-MAT 2^18 379 us a search,
//     2^20 653, against 191 and 357).
//   * Every flag word carries the tag of its level, so nothing is cleared
//     between levels or launches; the host hands each launch a fresh range
//     of tags.  Every wait is bounded and honours the abort word, so a grid
//     that is not co-resident ends with a timeout instead of hanging.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "bfs_kernel.hpp"
#include "scan_kernel.hpp"  // flag words, bounded waits, window fold, co-residency test

namespace lscan {

namespace {

constexpr int kWaves = kBfsThreads / 64;
constexpr int K = kBfsChunkEdges;
constexpr int kPer = K / kBfsThreads;  // edges per thread per chunk
constexpr int kWidePer = 4;             // edges per thread at a time in wide levels
constexpr int kWideChunks = kWidePer / kPer;  // chunks a workgroup takes at a time there
constexpr int KW = K * kWideChunks;
constexpr int kFilter = 16384;          // vertices a workgroup remembers as found
constexpr int64_t kCountMask = (int64_t(1) << kBfsCountBits) - 1;
constexpr int kBarrierWords = 4;
constexpr int kGatherPer = (kBfsMaxGrid + kBfsThreads - 1) / kBfsThreads;  // arrivals gathered per thread of workgroup 0
constexpr int kGatherBatch = kGatherPer < 4 ? kGatherPer : 4;  // arrivals in flight per thread
constexpr int kFoldBatch = 1;  // chunk values in flight per thread in the window sum

// Vertex and edge counts of a workgroup's vertices packed in 64 bits: at most
// eight vertices per thread, at most 2^42 edges.
constexpr int kTileBits = 14;
constexpr int64_t kTileMask = (int64_t(1) << kTileBits) - 1;
static_assert(8 * kBfsThreads <= kTileMask, "the vertices fit their field");

struct BfsShared {
    int64_t shift[KW];       // of the chunk's vertices: edge index = rank in the chunk + shift
    int32_t u[KW];           // the chunk's vertices
    uint64_t heads[2][KW / 64];  // one bit per rank: a vertex's first (the buffer not in use is clear)
    int32_t filter[kFilter];    // filter[v mod kFilter] = v: v is found (-1: none)
    int32_t stage[2][K];     // discovered vertices that have edges: the chunk being
                             // claimed and the one waiting to be placed
    int64_t wave_tot[kWaves];
    uint64_t found_e[2];     // edges of the vertices in stage[] (cleared for the next chunk
                             // while other waves still read this chunk's)
    uint32_t found[2];       // vertices in stage[]
    uint32_t found2[2];      // vertices found by a solo level, alternating
    uint32_t found_all;      // vertices this workgroup discovered in the current level
    uint32_t bad;            // malformed entries this workgroup met
    int32_t ok;
    int64_t p_n, p_e;        // the chunk's offsets in the next frontier
    int64_t res[kBarrierWords];
    int64_t gather[kWaves][4];
};

__device__ __forceinline__ uint32_t lanes_before(uint64_t mask)
{
    return __builtin_amdgcn_mbcnt_hi(uint32_t(mask >> 32), __builtin_amdgcn_mbcnt_lo(uint32_t(mask), 0u));
}

// A value that is the same in every lane, kept in scalar registers (the
// compiler cannot see that one read from LDS or a table is).
template <class T>
__device__ __forceinline__ T uniform(const T& v)
{
    return read_lane(v, 0);
}

__device__ __forceinline__ void give_up(const BfsArgs& a, uint32_t tag)
{
    __hip_atomic_store(a.abort_word, tag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(a.timeout_flag, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Whether some level may be a wide one: only those read the settled bits, and
// setting them costs an atomic per vertex, on one word for 32 neighbours (a star of
// 30 000 leaves 67.6 us a search with them, 44.8 without; 262 144 vertices in a binary
// tree 327 / 241).
__device__ __forceinline__ bool any_wide(const BfsArgs& a) { return a.ne >= kBfsWideEdges && a.ne >= a.nv / 4; }

// Degree of v with *beg its first edge, or -1 if its row range is not
// inside [0, E].
__device__ __forceinline__ int64_t row_range(const BfsArgs& a, int64_t v, int64_t* beg)
{
    const int64_t b0 = a.row[v], b1 = a.row[v + 1];
    *beg = b0;
    return (b0 >= 0 && b1 >= b0 && b1 <= a.ne) ? b1 - b0 : -1;
}

// Exclusive +-scan of one int64 per thread over the workgroup; *total gets
// the sum.  Ends with the workgroup synchronised.
__device__ __forceinline__ int64_t block_exclusive_sum(int64_t v, BfsShared& s, int64_t* total)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t inc = wave_inclusive_scan<AddI64>(v);
    if (lane == 63) s.wave_tot[wave] = inc;
    __syncthreads();
    int64_t before = 0, all = 0;
#pragma unroll
    for (int k = 0; k < kWaves; ++k) {
        const int64_t t = s.wave_tot[k];
        before += (k < wave) ? t : 0;
        all += t;
    }
    *total = uniform(all);
    __syncthreads();
    return before + inc - v;
}

// Sum of the packed values of chunks [lo, lo + cnt) (cnt < kBfsMaxGrid),
// read by the whole workgroup: every load in flight before the first wait,
// so the window costs one round trip.  Integer sums, so the order of the
// additions does not matter.  `ok` (every thread's) turns false if a wait
// gave up.  Ends with the workgroup synchronised.
__device__ __forceinline__ int64_t block_window_sum(const BfsArgs& a, BfsShared& s, int64_t lo, int64_t cnt,
                                                    uint32_t tag, bool& ok)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int64_t sum = 0;
    for (int i0 = 0; i0 < kGatherPer; i0 += kFoldBatch) {
        if (threadIdx.x + int64_t(i0) * kBfsThreads >= cnt) break;
        uint64_t w[kFoldBatch][2];
#pragma unroll
        for (int i = 0; i < kFoldBatch; ++i) {
            const int64_t j = threadIdx.x + int64_t(i0 + i) * kBfsThreads;
#pragma unroll
            for (int k = 0; k < 2; ++k)
                w[i][k] = (j < cnt) ? slot_load(a.slots + 2 * (lo + j) + k) : (uint64_t(tag) << 32);
        }
#pragma unroll
        for (int i = 0; i < kFoldBatch; ++i) {
            const int64_t j = threadIdx.x + int64_t(i0 + i) * kBfsThreads;
            if (j < cnt) {
#pragma unroll
                for (int k = 0; k < 2; ++k)
                    w[i][k] = await_word(a.slots + 2 * (lo + j) + k, w[i][k], tag, a.spin_limit, a.abort_word, ok);
                sum += int64_t(uint64_t(uint32_t(w[i][0])) | (uint64_t(uint32_t(w[i][1])) << 32));
            }
        }
    }
    const bool wave_ok = __ballot(!ok) == 0;
    sum = read_lane(wave_inclusive_scan<AddI64>(sum), 63);
    if (lane == 0) {
        s.gather[wave][0] = sum;
        s.gather[wave][3] = wave_ok ? 1 : 0;
    }
    __syncthreads();
    int64_t all = 0;
    bool all_ok = true;
#pragma unroll
    for (int k = 0; k < kWaves; ++k) {
        all += s.gather[k][0];
        all_ok = all_ok && s.gather[k][3] != 0;
    }
    ok = uniform(int(all_ok)) != 0;
    __syncthreads();
    return uniform(all);
}

// Grid barrier over flag words.  Every workgroup publishes the four 32-bit
// values v[] (thread 0's) under `tag`; workgroup 0 adds them up over the
// grid (word 1 and 2 are the low and high halves of one 64-bit value) and
// publishes the sums, which every workgroup reads into s.res.  Writes made
// before the call are visible to every workgroup after it.  Returns false
// if a wait gave up.
__device__ __forceinline__ bool grid_barrier(const BfsArgs& a, BfsShared& s, uint32_t tag, const uint32_t (&v)[kBarrierWords])
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    static_assert(kGatherPer * kBfsThreads >= kBfsMaxGrid, "workgroup 0 gathers the whole grid");
    // The workgroup barrier orders every wave's frontier writes before
    // thread 0's agent-scope release below, which makes them visible to the
    // whole device (a release is cumulative over what happens before it).
    __syncthreads();
    if (threadIdx.x == 0) {
        __hip_atomic_store(a.partial + blockIdx.x, int64_t(s.bad), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
#pragma unroll
        for (int k = 0; k < kBarrierWords; ++k)
            slot_store(a.arrive + kBarrierWords * blockIdx.x + k, (uint64_t(tag) << 32) | v[k]);
    }
    if (blockIdx.x == 0) {
        // every thread of workgroup 0 gathers up to kGatherPer workgroups'
        // arrivals, kGatherBatch of them in flight before the first wait
        bool ok = true;
        int64_t n = 0, e = 0, found = 0;
        for (int i0 = 0; i0 < kGatherPer; i0 += kGatherBatch) {
            if (threadIdx.x + int64_t(i0) * kBfsThreads >= int64_t(gridDim.x)) break;
            uint64_t w[kGatherBatch][kBarrierWords];
#pragma unroll
            for (int i = 0; i < kGatherBatch; ++i) {
                const int64_t j = threadIdx.x + int64_t(i0 + i) * kBfsThreads;
#pragma unroll
                for (int k = 0; k < kBarrierWords; ++k)
                    w[i][k] = (j < int64_t(gridDim.x)) ? slot_load(a.arrive + kBarrierWords * j + k)
                                                       : (uint64_t(tag) << 32);
            }
#pragma unroll
            for (int i = 0; i < kGatherBatch; ++i) {
                const int64_t j = threadIdx.x + int64_t(i0 + i) * kBfsThreads;
                if (j < int64_t(gridDim.x)) {
#pragma unroll
                    for (int k = 0; k < kBarrierWords; ++k)
                        w[i][k] = await_word(a.arrive + kBarrierWords * j + k, w[i][k], tag, a.spin_limit,
                                             a.abort_word, ok);
                }
                n += uint32_t(w[i][0]);
                e += int64_t(uint64_t(uint32_t(w[i][1])) | (uint64_t(uint32_t(w[i][2])) << 32));
                found += uint32_t(w[i][3]);
            }
        }
        // workgroup sums: waves through LDS
        const bool wave_ok = __ballot(!ok) == 0;
        n = read_lane(wave_inclusive_scan<AddI64>(n), 63);
        e = read_lane(wave_inclusive_scan<AddI64>(e), 63);
        found = read_lane(wave_inclusive_scan<AddI64>(found), 63);
        if (lane == 0) {
            s.gather[wave][0] = n;
            s.gather[wave][1] = e;
            s.gather[wave][2] = found;
            s.gather[wave][3] = wave_ok ? 1 : 0;
        }
        __syncthreads();
        if (threadIdx.x == 0) {
            bool all_ok = true;
            n = e = found = 0;
#pragma unroll
            for (int k = 0; k < kWaves; ++k) {
                n += s.gather[k][0];
                e += s.gather[k][1];
                found += s.gather[k][2];
                all_ok = all_ok && s.gather[k][3] != 0;
            }
            if (all_ok) {
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "agent");
                const uint32_t out[kBarrierWords] = {uint32_t(n), uint32_t(uint64_t(e)), uint32_t(uint64_t(e) >> 32),
                                                     uint32_t(found)};
#pragma unroll
                for (int k = 0; k < kBarrierWords; ++k) slot_store(a.go + k, (uint64_t(tag) << 32) | out[k]);
            } else {
                give_up(a, tag);
            }
        }
    }
    if (threadIdx.x == 0) {
        bool ok = true;
        uint64_t w[kBarrierWords];
#pragma unroll
        for (int k = 0; k < kBarrierWords; ++k) {
            w[k] = slot_load(a.go + k);
            w[k] = await_word(a.go + k, w[k], tag, a.spin_limit, a.abort_word, ok);
        }
        if (!ok) give_up(a, tag);
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        s.ok = ok ? 1 : 0;
        s.res[0] = uint32_t(w[0]);
        s.res[1] = int64_t(uint64_t(uint32_t(w[1])) | (uint64_t(uint32_t(w[2])) << 32));
        s.res[2] = 0;
        s.res[3] = uint32_t(w[3]);
    }
    __syncthreads();
    return uniform(s.ok) != 0;
}

// The frontier of one level: f vertices with their edge offsets and first
// edges, D edges in nc chunks, and the vertex of each chunk's first edge.
struct Frontier {
    const int32_t* vertex;
    const int64_t* edge_off;
    const int64_t* edge_shift;
    const int32_t* chunk_first;
    int64_t f, D, nc;
};
struct ChunkRange {
    int64_t k0;  // the chunk's first frontier vertex
    int n;       // frontier vertices its ranks fall in
};
struct FrontierEntry {
    int64_t off, shift;
    int32_t u;
};

// The table entries of the G chunks from c on, as loaded: waited for where
// frontier_range reads them.
struct ChunkHead {
    int32_t first, last;
};
template <int G>
__device__ __forceinline__ ChunkHead chunk_head(const Frontier& fr, int64_t c)
{
    return ChunkHead{fr.chunk_first[c], (c + G < fr.nc) ? fr.chunk_first[c + G] : int32_t(fr.f - 1)};
}
template <int G>
__device__ __forceinline__ ChunkRange frontier_range(const Frontier& fr, const ChunkHead& h)
{
    int64_t k0 = uniform(h.first);
    int64_t kend = uniform(h.last);
    k0 = (k0 < 0) ? 0 : (k0 >= fr.f ? fr.f - 1 : k0);  // memory guards: the table is consistent
    kend = (kend < k0) ? k0 : (kend >= fr.f ? fr.f - 1 : kend);
    if (kend - k0 > G * K) kend = k0 + G * K;
    return ChunkRange{k0, int(kend - k0 + 1)};
}

// Edges of the G chunks from c on (the last ones may be short).
template <int G>
__device__ __forceinline__ int chunk_edges(const Frontier& fr, int64_t c)
{
    return int((fr.D - c * K < G * K) ? fr.D - c * K : G * K);
}

// This thread's first entry of the range (few chunks have more vertices than threads).
__device__ __forceinline__ FrontierEntry frontier_entry(const Frontier& fr, const ChunkRange& r)
{
    const int64_t j = r.k0 + ((int(threadIdx.x) < r.n) ? int(threadIdx.x) : r.n - 1);
    return FrontierEntry{fr.edge_off[j], fr.edge_shift[j], fr.vertex[j]};
}

// Entry j of a chunk into LDS: a vertex whose first rank in the chunk is
// `rank` and first edge there rank + shift.
__device__ __forceinline__ void put_entry(BfsShared& s, int hb, int j, int rank, int64_t shift, int32_t u)
{
    s.shift[j] = shift;
    s.u[j] = u;
    atomicOr(reinterpret_cast<unsigned long long*>(&s.heads[hb][rank >> 6]), 1ull << (rank & 63));
}

// The frontier vertices of the G chunks from c on into LDS (first: this
// thread's first entry).  The workgroup synchronises before it reads them.
template <int G>
__device__ __forceinline__ void frontier_to_lds(const Frontier& fr, BfsShared& s, int hb, int64_t c,
                                                const ChunkRange& r, const FrontierEntry& first)
{
    auto put = [&](int j, const FrontierEntry& e) {
        const int64_t at = e.off - c * K;
        if (at < G * K) put_entry(s, hb, j, (at < 0) ? 0 : int(at), e.shift + c * K, e.u);
    };
    int j = threadIdx.x;
    if (j < r.n) put(j, first);
    for (j += kBfsThreads; j < r.n; j += kBfsThreads)
        put(j, FrontierEntry{fr.edge_off[r.k0 + j], fr.edge_shift[r.k0 + j], fr.vertex[r.k0 + j]});
}

// Each thread's ranks of a chunk of cnt edges, whose vertices are in LDS, to
// their edges: edge index and vertex (u = -1: past the last edge, or an edge
// outside the graph).  The vertex of a rank is the number of heads at or
// before it: a wave's row of ranks is one 64-bit word of heads, so that is a
// count of the heads in the words before and a bit count below the lane (a
// binary search of the chunk's vertices took a third of the kernel's VALU
// instructions).  Clears the other buffer of heads.
template <int PER>
__device__ __forceinline__ void map_ranks(const BfsArgs& a, BfsShared& s, int hb, int cnt, int64_t (&e)[PER],
                                          int32_t (&u)[PER])
{
    constexpr int kWords = PER * kWaves;        // of heads, one per wave-row
    constexpr int kHold = (kWords + 63) / 64;   // words held per lane: word 64q + lane
    const int lane = threadIdx.x & 63, wave = uniform(int(threadIdx.x) >> 6);
    uint64_t word[kHold];
    int32_t before[kHold], sum = 0;
#pragma unroll
    for (int q = 0; q < kHold; ++q) {
        word[q] = (64 * q + lane < kWords) ? s.heads[hb][64 * q + lane] : 0u;
        const int32_t heads = __builtin_popcountll(word[q]);
        const int32_t inc = wave_inclusive_scan<AddI32>(heads);
        before[q] = sum + inc - heads;
        sum += read_lane(inc, 63);
    }
    for (int j = threadIdx.x; j < KW / 64; j += kBfsThreads) s.heads[hb ^ 1][j] = 0;
#pragma unroll
    for (int p = 0; p < PER; ++p) {
        const int r = p * kBfsThreads + int(threadIdx.x);
        constexpr int kRows = 64 / kWaves;  // wave-rows whose words one register holds
        static_assert(64 % kWaves == 0, "whole rows per register");
        const int at = (p % kRows) * kWaves + wave;
        const uint64_t w = read_lane(word[p / kRows], at);
        const uint32_t k0 = uint32_t(read_lane(before[p / kRows], at)) + uint32_t(w & 1u) - 1u;
        const uint32_t kr = k0 + lanes_before(w >> 1);
        const uint32_t k = (kr < uint32_t(KW)) ? kr : uint32_t(KW - 1);  // memory guard: rank 0 has a head
        e[p] = 0;
        u[p] = -1;
        if (r < cnt) {
            e[p] = r + s.shift[k];
            if (uint64_t(e[p]) < uint64_t(a.ne))
                u[p] = s.u[k];
            else
                atomicAdd(&s.bad, 1u);
        }
    }
}

// Chunk-table entries of a frontier vertex at `pos` whose edges have ranks
// [eoff, eoff + d) (on: this lane has one): every chunk that starts in that
// range.  Called by whole waves: the long runs of a hub are written by all
// lanes.
__device__ __forceinline__ void fill_chunk_table(int32_t* table, int64_t cap, bool on, int64_t pos, int64_t eoff,
                                                 int64_t d)
{
    constexpr int kOwn = 4;  // entries a lane writes by itself
    const int lane = threadIdx.x & 63;
    const int64_t b0 = (eoff + K - 1) / K;
    int64_t b1 = on ? (eoff + d + K - 1) / K : b0;
    if (b1 > cap) b1 = cap;
    for (int i = 0; i < kOwn; ++i)
        if (b0 + i < b1) table[b0 + i] = int32_t(pos);
    uint64_t m = __ballot(b1 - b0 > kOwn);
    while (m) {
        const int l = __builtin_ctzll(m);
        m &= m - 1;
        const int64_t lo = read_lane(b0, l) + kOwn, hi = read_lane(b1, l);
        const int32_t at = read_lane(int32_t(pos), l);
        for (int64_t b = lo + lane; b < hi; b += 64) table[b] = at;
    }
}

// One wide level: every edge's endpoint is marked with a plain byte store and
// the next frontier is gathered by a sweep over the marks, so that no edge
// pays for an atomic.
//   expand  every edge whose endpoint is neither in the workgroup's filter of
//           vertices known to be found (LDS; an R-MAT graph's hubs: 1015 ->
//           975 us a search) nor settled (a bitmap that no level writes while
//           it reads it: 1400 -> 1340 us) reads the byte of its endpoint and,
//           if that is 0, stores 1 and the parent; several edges may find one
//           vertex and store the same byte and one of its valid parents;
//   sweep   (after a grid barrier) every workgroup takes an equal run of
//           vertices, counts those marked but not settled and their edges,
//           publishes the two sums, adds up what the workgroups before it
//           published, and writes its vertices' levels and frontier entries
//           behind them; the vertices become settled.
// *out_n, *out_e and *found get this workgroup's frontier vertices, their
// edges and its vertices found; tag advances by one for the inner barrier.
// Returns false if a wait gave up.
__device__ __forceinline__ bool wide_level(const BfsArgs& a, BfsShared& s, const Frontier& fr, uint32_t& tag, int& hb,
                                           int32_t lev, int64_t* out_n, int64_t* out_e, uint32_t* found)
{
    const int64_t nc = fr.nc;
    const int q = lev & 1;
    auto load_entry = [&](const ChunkRange& r) { return frontier_entry(fr, r); };
    auto store_chunk = [&](int64_t c, const ChunkRange& r, const FrontierEntry& e0) {
        frontier_to_lds<kWideChunks>(fr, s, hb, c, r, e0);
    };
    // the endpoints of each thread's ranks of chunk c and the vertices they leave (-1: no edge)
    auto load_ends = [&](int64_t c, int32_t (&v)[kWidePer], int32_t (&u)[kWidePer]) {
        int64_t e[kWidePer];
        map_ranks(a, s, hb, chunk_edges<kWideChunks>(fr, c), e, u);
        hb ^= 1;
#pragma unroll
        for (int p = 0; p < kWidePer; ++p) v[p] = (u[p] >= 0) ? __builtin_nontemporal_load(a.col + e[p]) : -1;
    };
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t B = gridDim.x, wg = blockIdx.x;
    const int64_t V = a.nv;

    const int64_t first = wg * kWideChunks, step = B * kWideChunks;
    if (first < nc) {
        // Software pipeline: while chunk c's marks are on their way, the
        // frontier entries of this workgroup's next chunk are fetched, its ranks
        // mapped and its column loads issued; the table entries that name the
        // chunk after that are fetched one step earlier still.
        ChunkRange next = frontier_range<kWideChunks>(fr, chunk_head<kWideChunks>(fr, first));
        FrontierEntry fe = load_entry(next);
        ChunkHead after{};
        if (first + step < nc) after = chunk_head<kWideChunks>(fr, first + step);
        store_chunk(first, next, fe);
        __syncthreads();
        int32_t v[kWidePer], u[kWidePer];
        load_ends(first, v, u);
        // the edges of the chunk before whose endpoints were not settled, and their marks
        int32_t pv[kWidePer], pu[kWidePer];
        uint8_t mark[kWidePer];
#pragma unroll
        for (int p = 0; p < kWidePer; ++p) pv[p] = -1;
        auto store_marks = [&]() {
#pragma unroll
            for (int p = 0; p < kWidePer; ++p) {
                if (pv[p] < 0) continue;
                s.filter[pv[p] & (kFilter - 1)] = pv[p];
                if (mark[p] == 0) {
                    a.found[pv[p]] = 1;
                    if (a.parent) a.parent[pv[p]] = pu[p];
                }
            }
        };
        for (int64_t c = first;; c += step) {
            const bool more = c + step < nc;
            if (more) {
                next = frontier_range<kWideChunks>(fr, after);
                fe = load_entry(next);
                if (c + 2 * step < nc) after = chunk_head<kWideChunks>(fr, c + 2 * step);
            }
            uint8_t bits[kWidePer];
#pragma unroll
            for (int p = 0; p < kWidePer; ++p) {
                if (uint32_t(v[p]) >= uint32_t(V)) {
                    if (u[p] >= 0) atomicAdd(&s.bad, 1u);
                    v[p] = -1;
                }
                if (v[p] >= 0 && s.filter[v[p] & (kFilter - 1)] == v[p]) v[p] = -1;
                bits[p] = (v[p] < 0) ? uint8_t(0xff) : a.settled[v[p] >> 3];
            }
            store_marks();
            int32_t v2[kWidePer], u2[kWidePer];
            if (more) {
                __syncthreads();  // chunk c's entries were read
                store_chunk(c + step, next, fe);
                __syncthreads();
                load_ends(c + step, v2, u2);
            }
#pragma unroll
            for (int p = 0; p < kWidePer; ++p) {
                const bool open = !((bits[p] >> (v[p] & 7)) & 1u);
                pv[p] = v[p];
                pu[p] = u[p];
                mark[p] = open ? a.found[v[p]] : uint8_t(1);  // a stale 0 only costs the stores again
            }
            if (!more) break;
#pragma unroll
            for (int p = 0; p < kWidePer; ++p) {
                v[p] = v2[p];
                u[p] = u2[p];
            }
        }
        store_marks();
    }
    const uint32_t v0[kBarrierWords] = {0u, 0u, 0u, 0u};
    if (!grid_barrier(a, s, tag, v0)) return false;
    ++tag;

    // the sweep, in groups of eight vertices (one byte of settled bits): this workgroup's run [g0, g1)
    const int64_t groups = (V + 7) / 8;
    const int64_t run = (groups + B - 1) / B;
    const int64_t g0 = (wg * run < groups) ? wg * run : groups;
    const int64_t g1 = (g0 + run < groups) ? g0 + run : groups;
    // the new vertices of group i (i < g1) as a bit mask; *was: the settled ones
    auto load_new = [&](int64_t i, uint32_t* was) -> uint32_t {
        *was = 0xffu;
        if (i >= g1) return 0u;
        const uint64_t m = reinterpret_cast<const uint64_t*>(a.found)[i];  // eight bytes, each 0 or 1
        *was = a.settled[i];
        return uint32_t((m * 0x0102040810204080ull) >> 56) & ~*was;
    };
    auto load_rows = [&](int64_t i, uint32_t fresh, int64_t (&row)[9]) {
#pragma unroll
        for (int j = 0; j < 9; ++j) row[j] = fresh ? a.row[(8 * i + j < V) ? 8 * i + j : V] : 0;
    };
    auto degree = [&](const int64_t (&row)[9], int j) -> int64_t {  // -1: not inside [0, E]
        return (row[j] >= 0 && row[j + 1] >= row[j] && row[j + 1] <= a.ne) ? row[j + 1] - row[j] : -1;
    };
    int64_t n = 0, e = 0;
    uint32_t all = 0;
    for (int64_t t0 = g0; t0 < g1; t0 += kBfsThreads) {
        int64_t row[9];
        uint32_t was;
        const uint32_t fresh = load_new(t0 + tid, &was);
        load_rows(t0 + tid, fresh, row);
        all += uint32_t(__builtin_popcount(fresh));
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            if ((fresh >> j) & 1u) {
                const int64_t d = degree(row, j);
                if (d < 0) atomicAdd(&s.bad, 1u);
                n += (d > 0) ? 1 : 0;
                e += (d > 0) ? d : 0;
            }
        }
    }
    // workgroup sums, published at once
    n = read_lane(wave_inclusive_scan<AddI64>(n), 63);
    e = read_lane(wave_inclusive_scan<AddI64>(e), 63);
    const int64_t f = read_lane(wave_inclusive_scan<AddI64>(int64_t(all)), 63);
    if (lane == 0) {
        s.gather[wave][0] = n;
        s.gather[wave][1] = e;
        s.gather[wave][2] = f;
    }
    __syncthreads();
    n = e = 0;
    all = 0;
#pragma unroll
    for (int k = 0; k < kWaves; ++k) {
        n += s.gather[k][0];
        e += s.gather[k][1];
        all += uint32_t(s.gather[k][2]);
    }
    if (tid == 0) {
        const uint32_t out[3] = {uint32_t(n), uint32_t(uint64_t(e)), uint32_t(uint64_t(e) >> 32)};
#pragma unroll
        for (int k = 0; k < 3; ++k) slot_store(a.swept + 4 * wg + k, (uint64_t(tag) << 32) | out[k]);
    }
    __syncthreads();  // s.gather is read before it is written again
    *out_n = uniform(n);
    *out_e = uniform(e);
    *found = uniform(all);

    // what the workgroups before this one found: four of them in flight per thread
    int64_t p_n = 0, p_e = 0;
    bool ok = true;
    constexpr int kBatch = kGatherBatch;
    for (int64_t j0 = 0; j0 < wg; j0 += kBatch * kBfsThreads) {
        uint64_t w[kBatch][3];
#pragma unroll
        for (int i = 0; i < kBatch; ++i) {
            const int64_t j = j0 + i * kBfsThreads + tid;
#pragma unroll
            for (int k = 0; k < 3; ++k) w[i][k] = (j < wg) ? slot_load(a.swept + 4 * j + k) : (uint64_t(tag) << 32);
        }
#pragma unroll
        for (int i = 0; i < kBatch; ++i) {
            const int64_t j = j0 + i * kBfsThreads + tid;
            if (j < wg) {
#pragma unroll
                for (int k = 0; k < 3; ++k)
                    w[i][k] = await_word(a.swept + 4 * j + k, w[i][k], tag, a.spin_limit, a.abort_word, ok);
            }
            p_n += uint32_t(w[i][0]);
            p_e += int64_t(uint64_t(uint32_t(w[i][1])) | (uint64_t(uint32_t(w[i][2])) << 32));
        }
    }
    const bool wave_ok = __ballot(!ok) == 0;
    p_n = read_lane(wave_inclusive_scan<AddI64>(p_n), 63);
    p_e = read_lane(wave_inclusive_scan<AddI64>(p_e), 63);
    if (lane == 0) {
        s.gather[wave][0] = p_n;
        s.gather[wave][1] = p_e;
        s.gather[wave][3] = wave_ok ? 1 : 0;
    }
    __syncthreads();
    p_n = p_e = 0;
    ok = true;
#pragma unroll
    for (int k = 0; k < kWaves; ++k) {
        p_n += s.gather[k][0];
        p_e += s.gather[k][1];
        ok = ok && s.gather[k][3] != 0;
    }
    p_n = uniform(p_n);
    p_e = uniform(p_e);
    __syncthreads();
    if (uniform(int(ok)) == 0) {
        if (tid == 0) give_up(a, tag);
        return false;
    }

    // the run's new vertices: levels, frontier entries, the next level's chunk table
    int32_t* nxt = a.queue[q ^ 1];
    int64_t* nxt_eo = a.edge_off[q ^ 1];
    int64_t* nxt_sh = a.edge_shift[q ^ 1];
    int32_t* nxt_cf = a.chunk_first[q ^ 1];
    for (int64_t t0 = g0; t0 < g1; t0 += kBfsThreads) {
        const int64_t i = t0 + tid;
        int64_t row[9];
        uint32_t was;
        const uint32_t fresh = load_new(i, &was);
        load_rows(i, fresh, row);
        int64_t mine = 0;  // edges << kTileBits | vertices
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            if ((fresh >> j) & 1u) {
                const int64_t d = degree(row, j);
                mine += (d > 0) ? ((d << kTileBits) | 1) : 0;
            }
        }
        int64_t tot = 0;
        const int64_t before = block_exclusive_sum(mine, s, &tot);
        int64_t pos = p_n + (before & kTileMask), eoff = p_e + (before >> kTileBits);
        p_n += tot & kTileMask;
        p_e += tot >> kTileBits;
        if (__ballot(fresh != 0) == 0) continue;
        if (fresh) a.settled[i] = uint8_t(was | fresh);
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const bool on = ((fresh >> j) & 1u) != 0;
            const int64_t v = 8 * i + j;
            if (on) a.level[v] = lev + 1;
            const int64_t d = on ? degree(row, j) : 0;
            const bool queued = d > 0 && pos < V;
            if (queued) {
                nxt[pos] = int32_t(v);
                nxt_eo[pos] = eoff;
                nxt_sh[pos] = row[j] - eoff;
            }
            fill_chunk_table(nxt_cf, a.chunk_cap, queued, pos, eoff, d);
            if (d > 0) {
                ++pos;
                eoff += d;
            }
        }
    }
    return true;
}

// Levels of at most K edges, run by one workgroup from the frontier in
// global memory: the next frontier stays in LDS, and a level is the chain
// column, claim, row range (four round trips with the frontier kept in
// memory and a grid barrier after each level).  Stops at a frontier of more
// edges, at an empty one, or after kSoloLevels (the other workgroups wait in
// the barrier meanwhile, and every wait is bounded).
constexpr int kSoloLevels = 32;
struct SoloResult {
    int64_t n, e;        // the next frontier (written to global memory)
    int64_t reached, scanned;
    int32_t levels;      // levels that found a vertex
    int32_t steps;       // levels run
};
__device__ __forceinline__ SoloResult solo_levels(const BfsArgs& a, BfsShared& s, int& hb, int32_t lev, int64_t f,
                                                  int64_t D)
{
    const int tid = threadIdx.x, lane = tid & 63;
    const int64_t V = a.nv;
    SoloResult out{};
    for (int j = tid; j < f; j += kBfsThreads) {
        const int64_t at = a.edge_off[lev & 1][j];
        if (j < K && at >= 0 && at < K) put_entry(s, hb, j, int(at), a.edge_shift[lev & 1][j], a.queue[lev & 1][j]);
    }
    if (tid == 0) s.found2[0] = 0;
    __syncthreads();
    for (;;) {
        out.scanned += D;
        int64_t e[kPer];
        int32_t u[kPer], v[kPer];
        map_ranks(a, s, hb, int(D), e, u);
        hb ^= 1;
#pragma unroll
        for (int p = 0; p < kPer; ++p) v[p] = (u[p] >= 0) ? a.col[e[p]] : -1;
        bool win[kPer];
#pragma unroll
        for (int p = 0; p < kPer; ++p) {
            win[p] = false;
            if (uint32_t(v[p]) < uint32_t(V)) {
                const uint32_t mask = 1u << (8 * (v[p] & 3));
                win[p] = !(atomicOr(reinterpret_cast<uint32_t*>(a.found) + (v[p] >> 2), mask) & mask);
            } else if (u[p] >= 0) {
                atomicAdd(&s.bad, 1u);
            }
        }
        int64_t d[kPer], beg[kPer];
#pragma unroll
        for (int p = 0; p < kPer; ++p) {
            d[p] = beg[p] = 0;
            if (win[p]) d[p] = row_range(a, v[p], &beg[p]);
        }
        int64_t mine = 0;  // edges << kTileBits | vertices
        uint32_t all = 0;
#pragma unroll
        for (int p = 0; p < kPer; ++p) {
            if (win[p]) {
                if (any_wide(a)) atomicOr(reinterpret_cast<uint32_t*>(a.settled) + (v[p] >> 5), 1u << (v[p] & 31));
                a.level[v[p]] = lev + out.steps + 1;
                if (a.parent) a.parent[v[p]] = u[p];
                if (d[p] < 0) atomicAdd(&s.bad, 1u);
                mine += (d[p] > 0) ? ((d[p] << kTileBits) | 1) : 0;
            }
            all += uint32_t(__popcll(__ballot(win[p])));
        }
        const int slot = out.steps & 1;
        if (lane == 0 && all) atomicAdd(&s.found2[slot], all);
        int64_t tot = 0;
        const int64_t before = block_exclusive_sum(mine, s, &tot);
        const uint32_t found = uniform(s.found2[slot]);
        if (tid == 0) s.found2[slot ^ 1] = 0;
        int64_t pos = before & kTileMask, eoff = before >> kTileBits;
        out.n = tot & kTileMask;
        out.e = tot >> kTileBits;
        ++out.steps;
        out.levels += (found > 0) ? 1 : 0;
        out.reached += found;
        const bool stay = out.n > 0 && out.e <= K && out.steps < kSoloLevels;
        const int q = (lev + out.steps) & 1;
#pragma unroll
        for (int p = 0; p < kPer; ++p) {
            const bool queued = d[p] > 0;
            if (stay) {
                if (queued) put_entry(s, hb, int(pos), int(eoff), beg[p] - eoff, v[p]);
            } else {
                if (queued) {
                    a.queue[q][pos] = v[p];
                    a.edge_off[q][pos] = eoff;
                    a.edge_shift[q][pos] = beg[p] - eoff;
                }
                fill_chunk_table(a.chunk_first[q], a.chunk_cap, queued, pos, eoff, d[p]);
            }
            if (queued) {
                ++pos;
                eoff += d[p];
            }
        }
        if (!stay) return out;
        D = out.e;
        __syncthreads();
    }
}

__global__ void __launch_bounds__(kBfsThreads) bfs_kernel(BfsArgs a)
{
    if (a.residency_check) {
        check_residency(a.ctrl, a.spin_limit);
        return;
    }
    __shared__ BfsShared s;

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t B = gridDim.x, wg = blockIdx.x;
    const int64_t V = a.nv;

    // Initial state: nothing visited but the source; the first frontier is
    // the source if it has edges.  Every
    // workgroup also counts the places where the row offsets decrease: rows
    // that overlap would break the bound of the chunk tables, so such a
    // graph is not searched.
    int64_t src_beg = 0;
    const int64_t src_deg = uniform(row_range(a, a.src, &src_beg));
    src_beg = uniform(src_beg);
    uint32_t decreasing = 0;
    constexpr int kInit = 4;  // vertices per thread in flight
    for (int64_t v0 = wg * kBfsThreads + tid; v0 < V; v0 += kInit * B * kBfsThreads) {
        int64_t r0[kInit], r1[kInit];
#pragma unroll
        for (int k = 0; k < kInit; ++k) {
            const int64_t v = v0 + k * B * kBfsThreads;
            r0[k] = (v < V) ? a.row[v] : 0;
            r1[k] = (v < V) ? a.row[v + 1] : 0;
        }
#pragma unroll
        for (int k = 0; k < kInit; ++k) {
            const int64_t v = v0 + k * B * kBfsThreads;
            if (v >= V) break;
            const bool is_src = (v == a.src);
            a.level[v] = is_src ? 0 : -1;
            if (a.parent) a.parent[v] = is_src ? a.src : -1;
            decreasing += (r0[k] > r1[k]) ? 1u : 0u;
        }
    }
    const int64_t groups = (V + 7) / 8;
    for (int64_t i = wg * kBfsThreads + tid; i < groups; i += B * kBfsThreads) {
        // vertices past the last one count as found
        uint32_t b = (8 * i + 8 > V) ? 0xffu << uint32_t(V - 8 * i) & 0xffu : 0u;
        if ((a.src >> 3) == i) b |= 1u << (a.src & 7);
        uint64_t m = 0;
#pragma unroll
        for (int j = 0; j < 8; ++j) m |= uint64_t((b >> j) & 1u) << (8 * j);
        reinterpret_cast<uint64_t*>(a.found)[i] = m;
        a.settled[i] = uint8_t(b);
    }
    const int64_t d0 = (src_deg > 0) ? src_deg : 0;
    if (wg == 0 && tid == 0 && d0 > 0) {
        a.queue[0][0] = a.src;
        a.edge_off[0][0] = 0;
        a.edge_shift[0][0] = src_beg;
    }
    for (int64_t b = wg * kBfsThreads + tid; b * K < d0 && b < a.chunk_cap; b += B * kBfsThreads)
        a.chunk_first[0][b] = 0;
    for (int j = tid; j < KW / 64; j += kBfsThreads) s.heads[0][j] = s.heads[1][j] = 0;
    for (int j = tid; j < kFilter; j += kBfsThreads) s.filter[j] = -1;
    int hb = 0;  // the buffer of heads to be filled next (clear)
    if (tid == 0) {
        s.bad = (wg == 0 && src_deg < 0) ? 1u : 0u;
        s.found_all = 0;
        s.found[0] = 0;
    }
    __syncthreads();
    if (decreasing) atomicAdd(&s.found[0], decreasing);
    __syncthreads();

    uint32_t tag = a.base_tag + 1u;
    uint32_t v0[kBarrierWords] = {0u, 0u, 0u, s.found[0]};
    bool ok = grid_barrier(a, s, tag, v0);
    const int64_t bad_rows = s.res[3];
    if (ok && bad_rows > 0) {
        // not searched: nothing reached, the decreasing steps reported
        if (wg == 0 && tid == 0) {
            a.level[a.src] = -1;
            if (a.parent) a.parent[a.src] = -1;
            if (a.stats) {
                a.stats[0] = 0;
                a.stats[1] = 0;
                a.stats[2] = 0;
                a.stats[3] = bad_rows;
            }
        }
        return;
    }

    int64_t f = (d0 > 0) ? 1 : 0, D = d0;
    int64_t levels = 1, reached = 1, scanned = 0;
    int32_t lev = 0;
    while (ok && f > 0) {
        ++tag;
        const int q = lev & 1;
        const int32_t* cur = a.queue[q];
        const int64_t* cur_eo = a.edge_off[q];
        const int64_t* cur_sh = a.edge_shift[q];
        const int32_t* cur_cf = a.chunk_first[q];
        int32_t* nxt = a.queue[q ^ 1];
        int64_t* nxt_eo = a.edge_off[q ^ 1];
        int64_t* nxt_sh = a.edge_shift[q ^ 1];
        int32_t* nxt_cf = a.chunk_first[q ^ 1];
        const int64_t nc = (D + K - 1) / K;
        if (nc > a.chunk_cap) break;  // cannot happen with non-decreasing rows (memory guard)
        if (D <= K) {
            // few edges: workgroup 0 runs this level, and those after it that are
            // as small, without a grid barrier between them
            SoloResult r{};
            if (wg == 0) r = solo_levels(a, s, hb, lev, f, D);
            levels += r.levels;
            reached += r.reached;
            scanned += r.scanned;
            const uint32_t vb[kBarrierWords] = {uint32_t(r.n), uint32_t(uint64_t(r.e)), uint32_t(uint64_t(r.e) >> 32),
                                                uint32_t(r.steps)};
            ok = grid_barrier(a, s, tag, vb);
            f = uniform(s.res[0]);
            D = uniform(s.res[1]);
            lev += uniform(int32_t(s.res[3]));
            continue;
        }
        scanned += D;
        const Frontier fr{cur, cur_eo, cur_sh, cur_cf, f, D, nc};
        if (D >= kBfsWideEdges && D >= V / 4) {
            int64_t out_n = 0, out_e = 0;
            uint32_t found = 0;
            ok = wide_level(a, s, fr, tag, hb, lev, &out_n, &out_e, &found);
            if (!ok) break;
            const uint32_t vb[kBarrierWords] = {uint32_t(out_n), uint32_t(uint64_t(out_e)),
                                                uint32_t(uint64_t(out_e) >> 32), found};
            ok = grid_barrier(a, s, tag, vb);
            if (!ok) break;
            f = uniform(s.res[0]);
            D = uniform(s.res[1]);
            if (f > V) f = V;  // cannot happen: each vertex is found once (memory guard)
            if (const int64_t more = uniform(s.res[3])) {
                ++levels;
                reached += more;
            }
            ++lev;
            continue;
        }
        int64_t run_n = 0, run_e = 0;    // offsets through this workgroup's previous chunk
        int64_t mine_n = 0, mine_e = 0;  // what this workgroup placed in this level
        if (tid == 0) s.found_all = 0;
        // Software pipeline: the iteration that claims chunk c places this
        // workgroup's previous chunk c - B, whose window of counts was
        // published about a round earlier, so placing rarely waits.
        int64_t prev_c = -1, prev_n = 0, prev_e = 0;
        int sb = 0;  // stage buffer of the chunk being claimed
        for (int64_t c = wg;; c += B) {
            const bool have = c < nc;
            int64_t A_n = 0, A_e = 0;  // the claimed chunk's staged vertices and their edges
            if (have) {
                // (a) the chunk's frontier vertices
                const ChunkRange cr = frontier_range<1>(fr, chunk_head<1>(fr, c));
                frontier_to_lds<1>(fr, s, hb, c, cr, frontier_entry(fr, cr));
                if (tid == 0) {
                    s.found[sb] = 0;
                    s.found_e[sb] = 0;
                }
                __syncthreads();

                // (b) map each rank to its edge and vertex, then claim every
                //     endpoint not yet visited; stage the winners that have edges
                int64_t e[kPer];
                int32_t u[kPer];
                bool act[kPer];
                map_ranks(a, s, hb, chunk_edges<1>(fr, c), e, u);
                hb ^= 1;
#pragma unroll
                for (int p = 0; p < kPer; ++p) act[p] = u[p] >= 0;
                int32_t v[kPer];
#pragma unroll
                for (int p = 0; p < kPer; ++p) v[p] = act[p] ? a.col[e[p]] : -1;
                uint8_t seen[kPer];
#pragma unroll
                for (int p = 0; p < kPer; ++p) {
                    if (act[p] && uint32_t(v[p]) >= uint32_t(V)) {
                        atomicAdd(&s.bad, 1u);
                        act[p] = false;
                    }
                    seen[p] = act[p] ? a.found[v[p]] : uint8_t(1);  // a stale 0 only costs an atomic
                }
                bool win[kPer];
#pragma unroll
                for (int p = 0; p < kPer; ++p) {
                    win[p] = false;
                    if (!seen[p]) {
                        const uint32_t mask = 1u << (8 * (v[p] & 3));
                        win[p] = !(atomicOr(reinterpret_cast<uint32_t*>(a.found) + (v[p] >> 2), mask) & mask);
                    }
                    if (any_wide(a) && win[p])
                        atomicOr(reinterpret_cast<uint32_t*>(a.settled) + (v[p] >> 5), 1u << (v[p] & 31));
                }
                int64_t dv[kPer];
#pragma unroll
                for (int p = 0; p < kPer; ++p) {
                    dv[p] = 0;
                    if (win[p]) {
                        a.level[v[p]] = lev + 1;
                        if (a.parent) a.parent[v[p]] = u[p];
                        int64_t beg;
                        dv[p] = row_range(a, v[p], &beg);
                        if (dv[p] < 0) {
                            atomicAdd(&s.bad, 1u);
                            dv[p] = 0;
                        }
                    }
                }
#pragma unroll
                for (int p = 0; p < kPer; ++p) {
                    const bool keep = win[p] && dv[p] > 0;
                    const uint64_t m_all = __ballot(win[p]);
                    const uint64_t m = __ballot(keep);
                    uint32_t base = 0;
                    if (lane == 0) {
                        if (m_all) atomicAdd(&s.found_all, uint32_t(__popcll(m_all)));
                        if (m) base = atomicAdd(&s.found[sb], uint32_t(__popcll(m)));
                    }
                    base = __builtin_amdgcn_readlane(base, 0);
                    if (keep) {
                        const uint32_t pos = base + lanes_before(m);  // < K: one discovery per edge at most
                        s.stage[sb][pos] = v[p];
                        atomicAdd(reinterpret_cast<unsigned long long*>(&s.found_e[sb]), (unsigned long long)dv[p]);
                    }
                }
                __syncthreads();
                A_n = uniform(s.found[sb]);
                A_e = uniform(int64_t(s.found_e[sb]));

                // (c) publish (edges, vertices) packed, at once
                if (wave == 0) publish_slot(a.slots + 2 * c, (A_e << kBfsCountBits) | A_n, tag, lane);
                mine_n += A_n;
                mine_e += A_e;
                if (prev_c < 0) {
                    prev_c = c;
                    prev_n = A_n;
                    prev_e = A_e;
                    sb ^= 1;
                    continue;
                }
            }
            if (prev_c < 0) break;  // no chunks in this level

            // (d) place the previous chunk: offsets = own running total + the
            //     values of the chunks in between; then its vertices, their
            //     edge offsets and first edges, and the next level's chunk
            //     table entries that fall in their edge ranges
            {
                const int32_t* st = s.stage[sb ^ 1];  // where the previous chunk was staged
                int32_t vl[kPer];
                int64_t bl[kPer], dl[kPer];
                int64_t dsum = 0;
#pragma unroll
                for (int t = 0; t < kPer; ++t) {  // loads in flight during the window wait
                    const int j = tid * kPer + t;
                    vl[t] = -1;
                    bl[t] = 0;
                    dl[t] = 0;
                    if (j < prev_n) {
                        vl[t] = st[j];
                        bl[t] = a.row[vl[t]];
                        dl[t] = a.row[vl[t] + 1] - bl[t];
                    }
                }
                const int64_t lo = (prev_c - B + 1 > 0) ? prev_c - B + 1 : 0;
                bool good = true;
                const int64_t between = block_window_sum(a, s, lo, prev_c - lo, tag, good);
                if (!good) {
                    if (tid == 0) give_up(a, tag);
                    ok = false;
                    break;
                }
                const int64_t p_n = run_n + (between & kCountMask);
                const int64_t p_e = run_e + (between >> kBfsCountBits);
                run_n = p_n + prev_n;
                run_e = p_e + prev_e;
#pragma unroll
                for (int t = 0; t < kPer; ++t) dsum += dl[t];
                int64_t tot = 0;
                int64_t eoff = p_e + block_exclusive_sum(dsum, s, &tot);
#pragma unroll
                for (int t = 0; t < kPer; ++t) {
                    const int j = tid * kPer + t;
                    const int64_t pos = p_n + j;
                    const bool queued = j < prev_n && pos < V;
                    if (queued) {
                        nxt[pos] = vl[t];
                        nxt_eo[pos] = eoff;
                        nxt_sh[pos] = bl[t] - eoff;
                    }
                    fill_chunk_table(nxt_cf, a.chunk_cap, queued, pos, eoff, dl[t]);
                    eoff += dl[t];
                }
            }
            if (!have) break;
            prev_c = c;
            prev_n = A_n;
            prev_e = A_e;
            sb ^= 1;
        }
        if (!ok) break;
        // (e) the level barrier: the next frontier's size and edges
        const uint32_t vb[kBarrierWords] = {uint32_t(mine_n), uint32_t(uint64_t(mine_e)),
                                            uint32_t(uint64_t(mine_e) >> 32), s.found_all};
        ok = grid_barrier(a, s, tag, vb);
        if (!ok) break;
        f = uniform(s.res[0]);
        D = uniform(s.res[1]);
        if (f > V) f = V;  // cannot happen: each vertex is claimed once (memory guard)
        if (const int64_t more = uniform(s.res[3])) {
            ++levels;
            reached += more;
        }
        ++lev;
    }

    if (ok && wg == 0 && a.stats) {
        int64_t mine = 0, bad = 0;
        for (int64_t j = tid; j < B; j += kBfsThreads)
            mine += __hip_atomic_load(a.partial + j, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        block_exclusive_sum(mine, s, &bad);
        if (tid != 0) return;
        a.stats[0] = levels;
        a.stats[1] = reached;
        a.stats[2] = scanned;
        a.stats[3] = bad;
    }
}

}  // namespace

hipError_t launch_bfs(const BfsArgs& a, int grid, hipStream_t stream)
{
    (void)hipGetLastError();
    hipLaunchKernelGGL(bfs_kernel, dim3(unsigned(grid)), dim3(kBfsThreads), 0, stream, a);
    return hipGetLastError();
}

const void* bfs_kernel_func() { return reinterpret_cast<const void*>(&bfs_kernel); }

}  // namespace lscan
