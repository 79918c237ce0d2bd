// radix_kernel.hip -- digit counts for the digit offsets of one radix-sort
// pass (a consumer of the scan; the paper names sorting among the uses of
// the scan, Section 1).
//
// The keys are cut into blocks of block_items; count[d][b] is the number of
// keys of block b whose digit (key >> shift) & (2^bits - 1) is d.  Written in
// digit-major order, the exclusive +-scan of that matrix is the digit
// offsets: where block b's first key of digit d lands in a stable partition
// of the keys by digit.  The runtime runs this kernel and then the plain
// single-pass scan (exclusive, int64) over the matrix in place.
//
// One workgroup takes G consecutive blocks: per block, each wave counts into
// its own LDS histogram (LDS atomics), the wave histograms are summed into
// the workgroup's G x 2^bits table, and at the end the table leaves in
// digit-major order, G consecutive counts per digit.
//
// The reads of the keys bound it (the LDS atomics take about 11 of 38 us at
// 50 million keys).  So the next round's vectors, of this block or the next
// one, are loaded before this round is counted; two sets of histograms leave
// one barrier per block; and vectors are read at any alignment of the keys
// and of the blocks.  Measured with the scan of the counts, int32 keys, 8
// bits, before and after: 50 million keys in blocks of 4096 54.7 / 53.3 us,
// the same off a 16-byte line 84.7 / 51.5, 300 million 304 / 296 (4.1 TB/s
// of keys).  Four vectors in flight at 256 threads take 252 against 245 us
// where the reads already run at the copy rate (400 million keys in blocks of
// 100 000).  The LDS of a workgroup, 8 KiB of histograms and up to 32 KiB of
// table, lets exactly four share a CU: 2^27 keys in blocks of 4096 are 1024
// workgroups, all resident at once (122 us; 31 blocks in a padded table
// instead of 32 160 us, for the 33 workgroups left over).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "radix_kernel.hpp"

namespace lscan {

namespace {

constexpr int kHistThreads = 256;
constexpr int kHistThreadsWide = 1024;
constexpr int kMaxDigits = 256;

// Blocks of at most this many keys per thread are read key by key, the others as
// vectors: a vector leaves most of the threads of a small block without work
// (with the scan, 4 bits, 50 million int32 keys: blocks of 64 437 us against
// 812 as vectors, 500 60 / 105, 1000 44 / 59; int64 keys: 500 94 / 111, 700 79 /
// 97, but 1000 78 / 72).
template <class K>
constexpr int kOwnKeys = sizeof(K) == 4 ? 4 : 3;

// Launches of at most two workgroups per CU (of 256) with large blocks take 1024
// threads and four vectors in flight per thread: 256 threads leave the CUs
// short of loads (int32 keys, 48 blocks of 2^20: 82 against 195 us; 382:
// 253 / 356; 501 blocks of 100 000: 38 / 44; int64 keys, 367 blocks of 16 384:
// 14.5 / 18.3).  With more workgroups the chip is full either way and the 1024
// threads of a block wait on its barrier (763 blocks of 65 536: 41 against 37 us).
constexpr int64_t kHistWideGroups = 512;
constexpr int64_t kHistWideBytes = int64_t(128) << 10;  // of keys per block

typedef uint32_t u32x4v __attribute__((ext_vector_type(4)));
typedef u32x4v VecU __attribute__((aligned(4)));  // keys need no more than their own alignment

template <class K>
__device__ __forceinline__ uint32_t digit_of(K key, int shift, uint32_t mask)
{
    return uint32_t(uint64_t(key) >> shift) & mask;
}

template <class K, int THREADS>
__global__ void __launch_bounds__(THREADS) digit_count_kernel(RadixArgs a)
{
    constexpr int kHistWaves = THREADS / 64;
    __shared__ uint32_t s_wave_hist[2][kHistWaves][kMaxDigits];  // of this block and the next
    extern __shared__ uint32_t s_table[];                        // [G][digits]

    const int tid = threadIdx.x;
    const int wave = tid >> 6;
    const int digits = 1 << a.bits;
    const uint32_t mask = uint32_t(digits - 1);
    // row g of the table is rotated by g, or by as many rows as 64 words hold: its rows
    // are written and its columns read by consecutive lanes, and a padded row would
    // take the 256-thread workgroups' LDS past a quarter of the CU's
    const int rot = a.bits < 6 ? 6 - a.bits : 0;
    auto entry = [&](int g, int d) -> uint32_t& {
        return s_table[g * digits + int(uint32_t(d + (g >> rot)) & mask)];
    };
    const int64_t b0 = int64_t(blockIdx.x) * a.group;
    const int gcount = int((a.num_blocks - b0 < a.group) ? (a.num_blocks - b0) : a.group);
    const K* keys = static_cast<const K*>(a.keys);
    constexpr int E = 16 / int(sizeof(K));
    constexpr int64_t kStride = int64_t(THREADS) * E;
    constexpr int kVecs = THREADS == kHistThreads ? 2 : 4;  // vectors of one round per thread

    for (int d = tid; d < 2 * kHistWaves * kMaxDigits; d += THREADS) (&s_wave_hist[0][0][0])[d] = 0;
    __syncthreads();

    // One round: kVecs vectors per thread from key `base` on.  Addresses past
    // the array's last whole vector are drawn back to it, their keys are not
    // counted; an array without a whole vector is not read as vectors.
    const int64_t last_vec = a.n - E;
    VecU w[kVecs];
    auto load_round = [&](int64_t base, int64_t end) {
        const K* from = keys + base + tid * E;
        if (base + kVecs * kStride <= end) {
#pragma unroll
            for (int u = 0; u < kVecs; ++u)
                w[u] = __builtin_nontemporal_load(reinterpret_cast<const VecU*>(from + u * kStride));
            return;
        }
#pragma unroll
        for (int u = 0; u < kVecs; ++u) {
            if (base + u * kStride >= end) break;
            const int64_t q = base + u * kStride + tid * E;
            w[u] = __builtin_nontemporal_load(reinterpret_cast<const VecU*>(keys + (q < last_vec ? q : last_vec)));
        }
    };
    auto block_end = [&](int64_t first) { return first + a.block_items < a.n ? first + a.block_items : a.n; };

    // Block g's counts: the waves' histograms summed into the table and cleared.
    // The other set of histograms is clear at the barrier: its last counts were
    // summed before it by every thread.
    auto sum_block = [&](int g) {
        __syncthreads();
        for (int d = tid; d < digits; d += THREADS) {
            uint32_t c = 0;
#pragma unroll
            for (int v = 0; v < kHistWaves; ++v) {
                c += s_wave_hist[g & 1][v][d];
                s_wave_hist[g & 1][v][d] = 0;
            }
            entry(g, d) = c;
        }
    };

    int64_t lo = b0 * a.block_items;
    if (THREADS == kHistThreads && a.block_items <= kOwnKeys<K> * THREADS) {
        // the next block's keys are in flight while this one's are counted
        K key[kOwnKeys<K>], now[kOwnKeys<K>];
        auto load_keys = [&](int64_t first) {
#pragma unroll
            for (int u = 0; u < kOwnKeys<K>; ++u) {
                if (u * THREADS >= a.block_items) break;
                const int64_t q = first + u * THREADS + tid;
                if (q < block_end(first)) key[u] = keys[q];
            }
        };
        load_keys(lo);
        for (int g = 0; g < gcount; ++g, lo += a.block_items) {
            const int64_t hi = block_end(lo);
#pragma unroll
            for (int u = 0; u < kOwnKeys<K>; ++u) now[u] = key[u];
            if (g + 1 < gcount) load_keys(hi);
#pragma unroll
            for (int u = 0; u < kOwnKeys<K>; ++u) {
                if (u * THREADS >= a.block_items) break;
                if (lo + u * THREADS + tid < hi) atomicAdd(&s_wave_hist[g & 1][wave][digit_of(now[u], a.shift, mask)], 1u);
            }
            sum_block(g);
        }
    } else {
        // the keys after a block's last whole vector, loaded a block ahead too (where
        // the blocks are whole vectors, only the array's last block has any)
        const bool tails = a.block_items % E != 0;
        K tail = K(0);
        auto load_tail = [&](int64_t first) {
            const int64_t end = block_end(first), q = end - (end - first) % E + tid;
            if (q < end) tail = keys[q];
        };
        if (last_vec >= 0) load_round(lo, block_end(lo));
        if (tails) load_tail(lo);
        for (int g = 0; g < gcount; ++g, lo += a.block_items) {
            const int64_t hi = block_end(lo);
            const int64_t v_end = hi - (hi - lo) % E;
            uint32_t* hist = s_wave_hist[g & 1][wave];
            const K last = tail;
            if (tails && g + 1 < gcount) load_tail(hi);
            for (int64_t base = lo; base < v_end; base += kVecs * kStride) {
                u32x4v now[kVecs];
#pragma unroll
                for (int u = 0; u < kVecs; ++u) now[u] = w[u];
                // the next round's vectors are in flight while this one is counted
                const bool full = base + kVecs * kStride <= v_end;
                const bool more = base + kVecs * kStride < v_end;
                if (more || g + 1 < gcount) load_round(more ? base + kVecs * kStride : hi, more ? v_end : block_end(hi));
#pragma unroll
                for (int u = 0; u < kVecs; ++u) {
                    if (full || base + u * kStride + tid * E < v_end) {
                        K k[E];
                        __builtin_memcpy(k, &now[u], 16);
#pragma unroll
                        for (int e = 0; e < E; ++e) atomicAdd(&hist[digit_of(k[e], a.shift, mask)], 1u);
                    }
                }
            }
            if (v_end + tid < hi) atomicAdd(&hist[digit_of(tails ? last : keys[v_end + tid], a.shift, mask)], 1u);
            sum_block(g);
        }
    }
    __syncthreads();

    // digit-major: for each digit, the G counts of this group's blocks
    const int dstep = THREADS / gcount, gstep = THREADS % gcount;
    int d = tid / gcount, g = tid % gcount;
    for (; d < digits; d += dstep, g += gstep) {
        if (g >= gcount) {
            g -= gcount;
            if (++d >= digits) break;
        }
        a.counts[int64_t(d) * a.num_blocks + b0 + g] = int64_t(entry(g, d));
    }
}

}  // namespace

hipError_t launch_digit_counts(const RadixArgs& a, hipStream_t stream)
{
    const int64_t groups = (a.num_blocks + a.group - 1) / a.group;
    const size_t table_bytes = size_t(a.group) * size_t(1 << a.bits) * sizeof(uint32_t);
    (void)hipGetLastError();
    const bool wide = groups <= kHistWideGroups && a.block_items >= kHistWideBytes / a.key_bytes;
    auto kernel = a.key_bytes == 4 ? (wide ? digit_count_kernel<uint32_t, kHistThreadsWide>
                                           : digit_count_kernel<uint32_t, kHistThreads>)
                                   : (wide ? digit_count_kernel<uint64_t, kHistThreadsWide>
                                           : digit_count_kernel<uint64_t, kHistThreads>);
    hipLaunchKernelGGL(kernel, dim3(unsigned(groups)), dim3(wide ? kHistThreadsWide : kHistThreads), table_bytes,
                       stream, a);
    return hipGetLastError();
}

}  // namespace lscan
