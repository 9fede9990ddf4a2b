// LSH index (Sec. 3.2): L hash tables of <key, id> pairs and the lookup of a query's L
// buckets, for gfx950.
//
// The paper fixes what a table holds (every vector's id under its key H_l(v)) and how a query
// uses it (fetch the L buckets H_1(u) .. H_L(u), evaluate the candidates), not a layout.  Here a
// table is the vector ids sorted by key (a stable sort of N <key, id> pairs, ids
// ascending inside a bucket; all tables are sorted together, by index_sort.hip or by the kernels below): a bucket is a contiguous run of the sorted ids, found by binary
// search of the sorted keys.  No chains, no resizing, 12 bytes per vector and table.
//
//   build      keys [N][L] -> per table: sorted keys [N], ids in key order [N]
//   probe      query keys [Q][L] -> per (query, table): first position and length of the bucket
//   candidates concatenation of a query's L buckets, all queries, at given offsets
//   nearest    processing of the candidates (Sec. 3.2, last paragraph): the candidate closest to
//              the query in l2, distances in fp32 over the full vectors; all candidates (the
//              exact version) or only the first max_candidates of the combined list (the
//              approximate version evaluates no more than 3L points)
#include <hip/hip_runtime.h>

#include <mutex>
#include <new>

#include "index_memory.h"
#include "index_sort.h"
#include "lsh.h"

struct lsh_index {
    uint64_t N = 0;
    uint32_t L = 0;
    int device = -1;
    uint64_t *d_keys = nullptr;  // [L][N] ascending per table
    uint32_t *d_ids = nullptr;   // [L][N] vector ids in key order (ascending within equal keys)
    lsh::IndexBlock tables;      // holds both
};

namespace {

// A group of LANES lanes per (query, table): lower and upper bound of the query's key in the table.
// A group reads LANES keys spread over its range at a time, which leaves one of LANES + 1 parts of
// it, and looks for the end of a bucket right behind its beginning first.  Few lookups are bound
// by the chain of dependent reads, many by the number of separate lines read, hence two sizes.
// Tables of 1e5 keys, one lane (halving, both ends from scratch) / 2 / 4 / 8 / 16 lanes: 512 lookups
// 7.1, 4.5, 4.0, 3.7, 3.7 us; 16384 lookups 13.5, 6.2, 5.3, 5.4, 6.5 us; 64000 lookups 24.7, 12.4, 14.5,
// 17.8, 20.2 us; 256000 lookups 87, 41, 49, 57, 67 us.
constexpr uint64_t kFewLookups = 16384;
constexpr uint32_t kFewLanes = 8, kManyLanes = 2;

// within positions [lo, hi) of an ascending table: the first one whose key is not below `key` (UPPER: is above it)
template <uint32_t LANES, bool UPPER>
__device__ __forceinline__ uint32_t group_bound(const uint64_t *__restrict__ table, uint32_t lo, uint32_t hi, uint64_t key) {
    constexpr uint64_t kMask = (1u << LANES) - 1;
    const uint32_t lane = threadIdx.x & (LANES - 1), first_lane = threadIdx.x & (63u & ~(LANES - 1));
    while (lo < hi) {
        const uint32_t len = hi - lo, part = len / (LANES + 1);
        auto at = [&](uint32_t i) { return lo + (part ? part * (i + 1) : i < len ? i : len - 1); };  // ascending, below hi
        const uint64_t have = table[at(lane)];
        const uint32_t before = __popcll((__ballot(UPPER ? have <= key : have < key) >> first_lane) & kMask);
        const uint32_t end = before < LANES ? at(before) : hi;
        if (before) lo = at(before - 1) + 1;
        hi = end;
    }
    return lo;
}

template <uint32_t LANES>
__device__ __forceinline__ void probe_item(const uint64_t *__restrict__ table, uint64_t N, uint64_t key, uint32_t *start,
                                           uint32_t *count) {
    constexpr uint64_t kMask = (1u << LANES) - 1;
    const uint32_t lane = threadIdx.x & (LANES - 1), first_lane = threadIdx.x & (63u & ~(LANES - 1));
    const uint32_t first = group_bound<LANES, false>(table, 0, (uint32_t)N, key);
    const bool same = first + lane < N && table[first + lane] == key;  // positions are below 2^31
    uint32_t end = first + __popcll((__ballot(same) >> first_lane) & kMask);
    if (end == first + LANES) end = group_bound<LANES, true>(table, end, (uint32_t)N, key);
    if (lane == 0) {
        *start = first;
        *count = end - first;
    }
}

template <uint32_t LANES>
__global__ __launch_bounds__(256) void probe_kernel(const uint64_t *__restrict__ sorted_keys, uint64_t N, uint32_t L,
                                                    const uint64_t *__restrict__ qkeys, uint64_t items,
                                                    uint32_t *__restrict__ start, uint32_t *__restrict__ count) {
    const uint64_t groups = (uint64_t)gridDim.x * (blockDim.x / LANES);
    for (uint64_t item = (blockIdx.x * (uint64_t)blockDim.x + threadIdx.x) / LANES; item < items; item += groups)
        probe_item<LANES>(sorted_keys + (item % L) * N, N, qkeys[item], start + item, count + item);
}

// The same table after table: what the lookups of a table read of it first, they find in an L2.  Eight tables at a time, one on
// every XCD, while there are eight; the lookups of those that are left go to all XCDs, one table after the other (with a table on
// each of some XCDs the others wait: 16000 queries in 11 tables of 4.8e4 13.1 us in turn, 16.8 so, 12.4 this way).
// For tables that two L2s do not hold and enough queries; us, in turn / table after table, tables in no cache: 1000 queries in 64
// tables of 1e5 20.3 / 19.7 (in a cache 15.1 / 10.7, between hashing and candidates 24.6 / 18), 4000 in 64 of 3e5 67 / 56,
// 16000 in 64 of 1e5 160 / 107.  In a cache, in turn : table after table, 500 to 64000 queries in 8 to 64 tables: of 4 MB
// together 0.92 to 1.28, of 5.6 MB 0.94 to 1.32, of 8.8 MB 0.99 to 1.47, of 10 MB 0.98 to 1.50, of 16 MB 1.01 to 1.62: queries and results are read and written in pieces.
constexpr uint64_t kTablesOfL2 = (4u << 20) / 8;  // keys
template <uint32_t LANES>
__global__ __launch_bounds__(256) void probe_tables_kernel(const uint64_t *__restrict__ sorted_keys, uint64_t N, uint32_t L,
                                                           const uint64_t *__restrict__ qkeys, uint32_t Q, uint32_t blocks,
                                                           uint32_t *__restrict__ start, uint32_t *__restrict__ count) {
    const uint32_t eights = L / 8 * 8, rest = blockIdx.x - eights * blocks;
    const bool dealt = blockIdx.x < eights * blocks;
    const uint32_t l = dealt ? blockIdx.x / 8 / blocks * 8 + blockIdx.x % 8 : eights + rest / blocks;
    const uint32_t q = ((dealt ? blockIdx.x / 8 : rest) % blocks * 256 + threadIdx.x) / LANES;
    if (q >= Q) return;
    const uint64_t item = (uint64_t)q * L + l;
    probe_item<LANES>(sorted_keys + l * N, N, qkeys[item], start + item, count + item);
}

// Exclusive prefix sum of 32-bit counts into 64-bit offsets, three small launches: (1) every
// block of kScanBlock counts adds up its own, (2) one block turns the block sums into block
// offsets in place, (3) every block scans its counts again on top of its offset.  `partial`
// holds one 64-bit word per block; every word is written by (1) before it is read, so the
// buffer needs no clearing between calls.
constexpr uint32_t kScanThreads = 256, kScanPerThread = 8, kScanBlock = kScanThreads * kScanPerThread;

// sum over the workgroup; every thread gets the total, `before` = sum over the threads below it
__device__ __forceinline__ uint64_t block_scan(uint64_t mine, uint64_t *wave_sums, uint64_t &before) {
    const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    uint64_t incl = mine;
    for (int d = 1; d < 64; d <<= 1) {
        const uint64_t up = __shfl_up(incl, d);
        if (lane >= (uint32_t)d) incl += up;
    }
    __syncthreads();  // wave_sums may still be read from an earlier call in the same kernel
    if (lane == 63) wave_sums[wave] = incl;
    __syncthreads();
    uint64_t below = 0, total = 0;
    for (uint32_t w = 0; w < kScanThreads / 64; ++w) {
        if (w < wave) below += wave_sums[w];
        total += wave_sums[w];
    }
    before = below + incl - mine;
    return total;
}

__global__ __launch_bounds__(kScanThreads) void scan_block_sums(const uint32_t *__restrict__ count, uint64_t items,
                                                                 uint64_t *__restrict__ partial) {
    __shared__ uint64_t wave_sums[kScanThreads / 64];
    const uint64_t first = (uint64_t)blockIdx.x * kScanBlock + (uint64_t)threadIdx.x * kScanPerThread;
    uint64_t mine = 0;
    for (uint32_t e = 0; e < kScanPerThread; ++e)
        if (first + e < items) mine += count[first + e];
    uint64_t before;
    const uint64_t total = block_scan(mine, wave_sums, before);
    if (threadIdx.x == 0) partial[blockIdx.x] = total;
}

// one workgroup: partial[b] <- sum of partial[0 .. b), for b < blocks, chunk after chunk
__global__ __launch_bounds__(kScanThreads) void scan_partials(uint64_t *__restrict__ partial, uint64_t blocks) {
    __shared__ uint64_t wave_sums[kScanThreads / 64];
    uint64_t carry = 0;
    for (uint64_t base = 0; base < blocks; base += kScanBlock) {
        const uint64_t first = base + (uint64_t)threadIdx.x * kScanPerThread;
        uint64_t v[kScanPerThread], mine = 0;
        for (uint32_t e = 0; e < kScanPerThread; ++e) {
            v[e] = first + e < blocks ? partial[first + e] : 0;
            mine += v[e];
        }
        uint64_t before;
        const uint64_t total = block_scan(mine, wave_sums, before);
        uint64_t run = carry + before;
        for (uint32_t e = 0; e < kScanPerThread; ++e) {
            if (first + e < blocks) partial[first + e] = run;
            run += v[e];
        }
        carry += total;
    }
}

// offsets[i] = sum of count[0 .. i) for i <= items (the last entry is the total)
__global__ __launch_bounds__(kScanThreads) void scan_offsets(const uint32_t *__restrict__ count, uint64_t items,
                                                              const uint64_t *__restrict__ partial,
                                                              uint64_t *__restrict__ offsets) {
    __shared__ uint64_t wave_sums[kScanThreads / 64];
    const uint64_t first = (uint64_t)blockIdx.x * kScanBlock + (uint64_t)threadIdx.x * kScanPerThread;
    uint32_t v[kScanPerThread];
    uint64_t mine = 0;
    for (uint32_t e = 0; e < kScanPerThread; ++e) {
        v[e] = first + e < items ? count[first + e] : 0;
        mine += v[e];
    }
    uint64_t before;
    block_scan(mine, wave_sums, before);
    uint64_t run = partial[blockIdx.x] + before;
    for (uint32_t e = 0; e < kScanPerThread; ++e) {
        if (first + e <= items) offsets[first + e] = run;  // element `items` receives the total
        run += v[e];
    }
}

// the three launches; partial must hold (items / kScanBlock + 1) words
int launch_offsets_scan(const uint32_t *d_count, uint64_t items, uint64_t *d_partial, uint64_t *d_offsets,
                        hipStream_t s) {
    const uint64_t blocks = items / kScanBlock + 1;  // covers element `items` too
    hipLaunchKernelGGL(scan_block_sums, dim3((uint32_t)blocks), dim3(kScanThreads), 0, s, d_count, items, d_partial);
    hipLaunchKernelGGL(scan_partials, dim3(1), dim3(kScanThreads), 0, s, d_partial, blocks);
    hipLaunchKernelGGL(scan_offsets, dim3((uint32_t)blocks), dim3(kScanThreads), 0, s, d_count, items, d_partial,
                       d_offsets);
    return hipGetLastError() == hipSuccess ? LSH_OK : LSH_ERR_HIP;
}

// Tables of more than 2^20 pairs (the others: index_sort.hip).
// Stable least-significant-digit radix sort of all L key columns at once (one grid row per
// table): eight passes of 8 bits.  A pass is three launches: per-tile digit histograms, an
// exclusive scan of every table's and digit's counts over the tiles, and the scatter.  A tile is 4096
// consecutive pairs; wave w of the workgroup owns pairs 1024 w ... 1024 w + 1023 of it, slot i
// of lane l being pair 64 i + l, so (wave, slot, lane) order is memory order and the ranks
// below keep equal keys in their original order (ids ascending inside a bucket).  The first
// pass takes the keys from where sort_columns put them and numbers the pairs itself.
constexpr uint32_t kSortThreads = 256, kSortSlots = 16, kSortTile = kSortThreads * kSortSlots;
constexpr uint32_t kSortWaves = kSortThreads / 64;

// What the first pass starts with: a workgroup takes up to 16 columns of a tile of the caller's rows, counts
// their first digits and writes the keys column by column, [L][N], so that a wave reads whole pieces of
// rows and the scatter whole pieces of columns.  (Both read a column of the caller's array before, 8 bytes out of
// every row: for 1e6 x 32 keys 329 us for the counts and 361 for the scatter; by rows, counts alone, 119.)
constexpr uint32_t kRowThreads = 1024, kRowColumns = 16, kRowStride = 257;  // a column's bins one bank on from the column before
constexpr uint32_t kRowLoads = 4, kRowBlock = kRowThreads * kRowLoads;      // keys turned at a time

__global__ __launch_bounds__(kRowThreads) void sort_columns(const uint64_t *__restrict__ keys, uint64_t N, uint32_t L,
                                                            uint32_t columns, uint32_t width, uint32_t tiles,
                                                            uint32_t *__restrict__ hist, uint64_t *__restrict__ out) {
    __shared__ uint32_t bins[kRowColumns * kRowStride];
    __shared__ uint64_t turned[kRowBlock + kRowColumns];  // [column][rows at a time + 1]
    const uint32_t tile = blockIdx.x, l0 = blockIdx.y * columns, here = L - l0 < columns ? L - l0 : columns;
    for (uint32_t b = threadIdx.x; b < kRowColumns * kRowStride; b += kRowThreads) bins[b] = 0;
    // width: a power of two, at least `columns` and at most 16
    const uint32_t column = threadIdx.x & (width - 1), row = threadIdx.x / width, step = kRowThreads / width;
    const uint32_t rows = kRowLoads * step;  // at a time; a tile is `width` times as many
    const uint64_t first = (uint64_t)tile * kSortTile, end = N - first < kSortTile ? N : first + kSortTile;
    const uint64_t *at = keys + l0 + (column < here ? column : 0);
    uint64_t key[kRowLoads];
    auto load = [&](uint64_t base) __attribute__((always_inline)) {
#pragma unroll
        for (uint32_t u = 0; u < kRowLoads; ++u) {
            const uint64_t i = base + row + u * step;
            key[u] = at[(i < end ? i : end - 1) * L];
        }
    };
    load(first);
    for (uint64_t base = first; base < end; base += rows) {
        __syncthreads();  // the keys before have been written out (and the bins are clear)
#pragma unroll
        for (uint32_t u = 0; u < kRowLoads; ++u) {
            turned[column * (rows + 1) + row + u * step] = key[u];
            if (column < here && base + row + u * step < end) atomicAdd(&bins[column * kRowStride + ((uint32_t)key[u] & 255u)], 1u);
        }
        __syncthreads();
        if (base + rows < end) load(base + rows);
        const uint32_t rows_here = end - base < rows ? (uint32_t)(end - base) : rows;
#pragma unroll
        for (uint32_t u = 0; u < kRowLoads; ++u) {
            const uint32_t e = threadIdx.x + u * kRowThreads, c = e / rows, r = e & (rows - 1);
            if (c < here && r < rows_here) out[(uint64_t)(l0 + c) * N + base + r] = turned[c * (rows + 1) + r];
        }
    }
    __syncthreads();
    for (uint32_t b = threadIdx.x; b < here * 256; b += kRowThreads)
        hist[((size_t)l0 * 256 + b) * tiles + tile] = bins[(b >> 8) * kRowStride + (b & 255u)];
}

// hist[(l * 256 + digit) * tiles + tile] = pairs of the tile with that digit.  Equal keys are neighbours once
// their lower digits are in order, and a wave that adds 64 of them to one word does so one after the other: the
// first lane of a run of equal digits adds its length.
__global__ __launch_bounds__(kSortThreads) void sort_histogram(const uint64_t *__restrict__ keys, uint64_t N,
                                                                uint32_t shift, uint32_t tiles,
                                                                uint32_t *__restrict__ hist) {
    __shared__ uint32_t bins[257];
    const uint32_t l = blockIdx.y, tile = blockIdx.x;
    const uint64_t first = (uint64_t)tile * kSortTile + threadIdx.x;
    uint32_t digit[kSortSlots];
#pragma unroll
    for (uint32_t e = 0; e < kSortSlots; ++e) {
        const uint64_t i = first + e * kSortThreads;
        digit[e] = i < N ? (uint32_t)(keys[(uint64_t)l * N + i] >> shift) & 255u : 256u;
    }
    bins[threadIdx.x] = 0;
    __syncthreads();
    const uint32_t lane = threadIdx.x & 63;
#pragma unroll
    for (uint32_t e = 0; e < kSortSlots; ++e) {
        const uint32_t before = (uint32_t)__builtin_amdgcn_update_dpp(-1, (int)digit[e], 0x138, 0xf, 0xf, false);  // wave_shr:1
        const uint64_t heads = __ballot(digit[e] != before), later = heads & ~((2ull << lane) - 1);
        const uint32_t stop = later ? (uint32_t)__builtin_ctzll(later) : 64u;
        if (digit[e] != before) atomicAdd(&bins[digit[e]], stop - lane);  // word 256 is not read
    }
    __syncthreads();
    hist[((size_t)l * 256 + threadIdx.x) * tiles + tile] = bins[threadIdx.x];
}

// One wave per (table, digit): its counts <- their exclusive prefix sum over the tiles, in place, and the
// sum of all of them to `total`; the scatter adds up the smaller digits' totals.  (One workgroup per table
// that scanned all 256 * tiles counts: 74 us a pass at 1e6 x 32, 32 workgroups on 256 CUs; this 6.)
__global__ __launch_bounds__(256) void sort_scan(uint32_t *__restrict__ hist, uint32_t tiles, uint32_t digits,
                                                 uint32_t *__restrict__ total) {
    const uint32_t lane = threadIdx.x & 63, digit = blockIdx.x * 4 + (threadIdx.x >> 6);  // of all tables
    if (digit >= digits) return;
    uint32_t *mine = hist + (size_t)digit * tiles;
    uint32_t carry = 0;  // below N < 2^31
    for (uint32_t base = 0; base < tiles; base += 256) {
        uint32_t v[4];
#pragma unroll
        for (uint32_t u = 0; u < 4; ++u) v[u] = base + u * 64 + lane < tiles ? mine[base + u * 64 + lane] : 0;
#pragma unroll
        for (uint32_t u = 0; u < 4; ++u) {
            uint32_t incl = v[u];
            for (uint32_t step = 1; step < 64; step <<= 1) {
                const uint32_t up = __shfl_up(incl, step);
                if (lane >= step) incl += up;
            }
            if (base + u * 64 + lane < tiles) mine[base + u * 64 + lane] = carry + incl - v[u];
            carry += __shfl(incl, 63);
        }
    }
    if (lane == 0) total[digit] = carry;
}

// The scatter of a pass.  A pair's place in the output is (pairs of smaller digits in its
// table) + (pairs of its digit in earlier tiles) + (pairs of its digit before it in its tile);
// the first two come from the totals and the scanned histograms, the third from wave ballots in memory order.
// The tile is first put in that order in LDS and then written out by consecutive threads:
// pairs of one digit are then neighbours in LDS and in memory, so the stores of a wave are a
// few runs instead of 64 separate 8-byte writes (about three times faster than scattering from the
// registers on this part).
template <bool FIRST>
__global__ __launch_bounds__(kSortThreads) void sort_scatter(const uint64_t *__restrict__ keys,
                                                              const uint32_t *__restrict__ ids, uint64_t N,
                                                              uint32_t shift, uint32_t tiles,
                                                              const uint32_t *__restrict__ offsets,
                                                              const uint32_t *__restrict__ total,
                                                              uint64_t *__restrict__ out_keys,
                                                              uint32_t *__restrict__ out_ids) {
    __shared__ uint32_t counter[kSortWaves][256];  // per wave: pairs seen so far per digit, then its first place in the tile's order
    __shared__ uint32_t delta[256];                // per digit: first output position minus first place in the tile's order
    __shared__ uint32_t wave_total[2][kSortWaves];
    __shared__ uint64_t tile_keys[kSortTile];
    __shared__ uint32_t tile_ids[kSortTile];
    const uint32_t l = blockIdx.y, tile = blockIdx.x;
    const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    for (uint32_t w = 0; w < kSortWaves; ++w) counter[w][threadIdx.x] = 0;
    __syncthreads();
    const uint64_t tile_first = (uint64_t)tile * kSortTile;
    const uint64_t first = tile_first + (uint64_t)wave * (kSortSlots * 64) + lane;
    const uint64_t below = (1ull << lane) - 1;
    uint64_t key[kSortSlots];
    uint32_t id[kSortSlots];
    uint32_t rank[kSortSlots];
    volatile uint32_t *mine = counter[wave];
    // All loads first: behind the ordered LDS accesses of the ranking they go out one slot at a time (a pass over
    // 1e6 x 32 pairs 334 -> 219 us, 3.5 TB/s).
#pragma unroll
    for (uint32_t i = 0; i < kSortSlots; ++i) {
        const uint64_t at = first + (uint64_t)i * 64;
        key[i] = keys[(uint64_t)l * N + (at < N ? at : N - 1)];
        id[i] = FIRST ? (uint32_t)at : ids[(uint64_t)l * N + (at < N ? at : N - 1)];
    }
    const uint32_t tile_offset = offsets[((size_t)l * 256 + threadIdx.x) * tiles + tile], digit_total = total[l * 256 + threadIdx.x];
#pragma unroll
    for (uint32_t i = 0; i < kSortSlots; ++i) {
        const bool valid = first + (uint64_t)i * 64 < N;
        const uint32_t digit = (uint32_t)(key[i] >> shift) & 255u;
        // lanes of the wave that hold the same digit in this slot
        uint64_t peers = __ballot(valid);
#pragma unroll
        for (uint32_t bit = 0; bit < 8; ++bit) {
            const uint64_t set = __ballot((digit >> bit) & 1u);
            peers &= ((digit >> bit) & 1u) ? set : ~set;
        }
        const uint32_t seen = mine[digit];
        rank[i] = seen + (uint32_t)__popcll(peers & below);
        __builtin_amdgcn_wave_barrier();
        if (valid && (peers & below) == 0) mine[digit] = seen + (uint32_t)__popcll(peers);  // the first of the peers
        __builtin_amdgcn_wave_barrier();
    }
    __syncthreads();
    {   // thread d: the tile's pairs of digit d, their first place in the tile's order (an exclusive
        // scan over the digits) and, per wave, the first place of that wave's pairs of the digit
        uint32_t per_wave[kSortWaves], in_tile = 0;
        for (uint32_t w = 0; w < kSortWaves; ++w) {
            per_wave[w] = counter[w][threadIdx.x];
            in_tile += per_wave[w];
        }
        // inclusive scans over the 64 digits of this wave, then over the waves: of the tile, of the table
        uint32_t incl = in_tile, incl_table = digit_total;
#pragma unroll
        for (uint32_t step = 1; step < 64; step <<= 1) {
            const uint32_t up = __shfl_up(incl, step), up_table = __shfl_up(incl_table, step);
            if (lane >= step) incl += up, incl_table += up_table;
        }
        if (lane == 63) wave_total[0][wave] = incl, wave_total[1][wave] = incl_table;
        __syncthreads();
        uint32_t start = incl - in_tile, table_start = incl_table - digit_total;
        for (uint32_t w = 0; w < wave; ++w) start += wave_total[0][w], table_start += wave_total[1][w];
        delta[threadIdx.x] = table_start + tile_offset - start;
        for (uint32_t w = 0; w < kSortWaves; ++w) {
            counter[w][threadIdx.x] = start;
            start += per_wave[w];
        }
    }
    __syncthreads();
#pragma unroll
    for (uint32_t i = 0; i < kSortSlots; ++i) {
        const uint64_t at = first + (uint64_t)i * 64;
        if (at >= N) continue;
        const uint32_t digit = (uint32_t)(key[i] >> shift) & 255u;
        const uint32_t place = counter[wave][digit] + rank[i];
        tile_keys[place] = key[i];
        tile_ids[place] = id[i];
    }
    __syncthreads();
    const uint32_t pairs = (uint32_t)(N - tile_first < kSortTile ? N - tile_first : kSortTile);
    for (uint32_t place = threadIdx.x; place < pairs; place += kSortThreads) {
        const uint64_t k64 = tile_keys[place];
        const uint64_t pos = (uint64_t)l * N + (uint32_t)(delta[(uint32_t)(k64 >> shift) & 255u] + place);
        out_keys[pos] = k64;
        out_ids[pos] = tile_ids[place];
    }
}

// Scratch of lsh_index_candidate_offsets_static: the block sums of the scan, for callers that
// must not allocate.  One copy per GPU, held until the process ends; its device address is
// looked up once per device (the name below is only a host-side handle of the symbol).
constexpr uint64_t kStaticScanItems = 1ull << 22;
constexpr uint64_t kStaticScanWords = kStaticScanItems / kScanBlock + 1;
static __device__ __align__(256) uint64_t scratch[kStaticScanWords];

constexpr int kMaxDevices = 64;
std::mutex scratch_mutex;
uint64_t *scratch_of_device[kMaxDevices] = {};

// device address of `scratch` on the current device (null on failure)
uint64_t *static_scratch() {
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return nullptr;
    std::lock_guard<std::mutex> lock(scratch_mutex);
    if (!scratch_of_device[dev]) {
        void *ptr = nullptr;
        if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess) {
            (void)hipGetLastError();
            return nullptr;
        }
        scratch_of_device[dev] = static_cast<uint64_t *>(ptr);
    }
    return scratch_of_device[dev];
}

// one wave per (query, table): copies the bucket's ids to the output run of that item
__global__ void candidates_kernel(const uint32_t *__restrict__ sorted_ids, uint64_t N, uint32_t L,
                                  const uint32_t *__restrict__ start, const uint32_t *__restrict__ count,
                                  const uint64_t *__restrict__ offsets, uint64_t items, uint32_t *__restrict__ out) {
    const uint32_t lane = threadIdx.x & 63;
    const uint64_t waves = ((uint64_t)gridDim.x * blockDim.x) >> 6;
    for (uint64_t item = (blockIdx.x * (uint64_t)blockDim.x + threadIdx.x) >> 6; item < items; item += waves) {
        const uint32_t l = (uint32_t)(item % L);
        const uint32_t *src = sorted_ids + (uint64_t)l * N + start[item];
        uint32_t *dst = out + offsets[item];
        for (uint32_t i = lane; i < count[item]; i += 64) dst[i] = src[i];
    }
}

// One workgroup per query: squared l2 distance of every distinct candidate of its L buckets,
// minimum with ties to the smaller id.
// INNER: the score is the inner product with the query instead and the largest one wins
// (maximum inner product search; internally the negated product is minimised).
// The work is reading the candidates' vectors, so the kernel first lays out which ones: the
// positions of the combined list are dealt to all threads (a prefix sum over the bucket lengths
// says which bucket a position is in), and an id goes on the list in LDS unless it is among those
// met before (a table of 2048 slots in LDS; an id that finds no slot in a few tries is simply
// evaluated again, which changes nothing).  The list is then evaluated by groups of lanes, as many
// as a vector has pieces of VEC coordinates (at most a wave), four candidates in flight in each.
// VEC = 4 (16-byte loads) for vectors and queries on 16-byte boundaries with n a multiple of 4.
// QUERY_IN_LDS up to kQueryInLds coordinates (all of the LDS used stays below 64 KB).
// 1000 queries against 1e5 vectors of 960 dimensions, every candidate of 64 buckets: 1028 -> 70 us
// (one wave a candidate, 4-byte loads, one in flight, repeats evaluated again -> this).
constexpr uint32_t kListIds = 1024, kSeenSlots = 2048, kSeenTries = 4, kBucketsAtOnce = 256, kQueryInLds = 11264;
constexpr uint32_t kNearestThreads = 1024, kNoId = 0xFFFFFFFFu;

template <int VEC>
struct Piece {
    float x[VEC];
};

template <int VEC>
__device__ __forceinline__ Piece<VEC> read_piece(const float *at) {
    Piece<VEC> r;
    if constexpr (VEC == 4) {
        const float4 v = *reinterpret_cast<const float4 *>(at);
        r.x[0] = v.x, r.x[1] = v.y, r.x[2] = v.z, r.x[3] = v.w;
    } else {
        r.x[0] = *at;
    }
    return r;
}

template <bool INNER, int VEC, bool QUERY_IN_LDS>
__global__ __launch_bounds__(kNearestThreads) void nearest_kernel(
    const uint32_t *__restrict__ sorted_ids, uint64_t N, uint32_t L, const float *__restrict__ data,
    const float *__restrict__ queries, uint32_t n, uint32_t group_lanes, const uint32_t *__restrict__ start,
    const uint32_t *__restrict__ count, uint32_t max_candidates, uint32_t *__restrict__ best_id,
    float *__restrict__ best_dist) {
    extern __shared__ __align__(16) float query_lds[];  // [n] when QUERY_IN_LDS
    __shared__ uint64_t bucket_end[kBucketsAtOnce];     // positions up to the end of the bucket, from the first of these buckets
    __shared__ uint32_t bucket_first[kBucketsAtOnce];
    __shared__ uint64_t wave_sums[kBucketsAtOnce / 64];
    __shared__ uint32_t seen[kSeenSlots];
    __shared__ uint32_t list[kListIds];
    __shared__ uint32_t listed;
    __shared__ float wave_d[kNearestThreads / 64];
    __shared__ uint32_t wave_id[kNearestThreads / 64];
    const uint64_t q = blockIdx.x;
    const uint32_t tid = threadIdx.x, threads = blockDim.x, lane = tid & 63, wave = tid >> 6;
    const float *query = queries + q * n;
    if constexpr (QUERY_IN_LDS) {
        for (uint32_t c = tid * VEC; c < n; c += threads * VEC) {
            const Piece<VEC> p = read_piece<VEC>(query + c);
#pragma unroll
            for (int e = 0; e < VEC; ++e) query_lds[c + e] = p.x[e];
        }
    }
    for (uint32_t i = tid; i < kSeenSlots; i += threads) seen[i] = kNoId;
    if (tid == 0) listed = 0;
    float mine_d = INFINITY;
    uint32_t mine_id = kNoId;
    uint64_t left = max_candidates;  // of the combined list, still to be looked at
    for (uint32_t l0 = 0; l0 < L && left; l0 += kBucketsAtOnce) {
        uint64_t incl = 0;
        if (tid < kBucketsAtOnce) {
            const uint32_t l = l0 + tid;
            incl = l < L ? count[q * L + l] : 0;
            bucket_first[tid] = l < L ? start[q * L + l] : 0;
            for (int d = 1; d < 64; d <<= 1) {
                const uint64_t up = __shfl_up(incl, d);
                if (lane >= (uint32_t)d) incl += up;
            }
            if (lane == 63) wave_sums[wave] = incl;
        }
        __syncthreads();
        if (tid < kBucketsAtOnce) {
            for (uint32_t w = 0; w < wave; ++w) incl += wave_sums[w];
            bucket_end[tid] = incl;
        }
        __syncthreads();
        const uint64_t all = bucket_end[kBucketsAtOnce - 1], total = all < left ? all : left;
        for (uint64_t base = 0; base < total; base += kListIds) {
            const uint64_t stop = total - base < kListIds ? total : base + kListIds;
            for (uint64_t pos = base + tid; pos < stop; pos += threads) {
                uint32_t b = 0;  // first bucket that ends behind pos
                for (uint32_t half = kBucketsAtOnce / 2; half; half >>= 1)
                    if (bucket_end[b + half - 1] <= pos) b += half;
                const uint64_t before = b ? bucket_end[b - 1] : 0;
                const uint32_t id = sorted_ids[(uint64_t)(l0 + b) * N + bucket_first[b] + (pos - before)];
                bool fresh = true;
                uint32_t slot = (id * 0x9E3779B1u) >> 21;
                for (uint32_t t = 0; t < kSeenTries; ++t) {
                    const uint32_t was = atomicCAS(&seen[slot], kNoId, id);
                    if (was == id) fresh = false;
                    if (was == id || was == kNoId) break;
                    slot = (slot + 1) & (kSeenSlots - 1);
                }
                if (fresh) list[atomicAdd(&listed, 1u)] = id;
            }
            __syncthreads();
            const uint32_t have = listed;
            const uint32_t groups = threads / group_lanes, group = tid / group_lanes, piece0 = tid & (group_lanes - 1);
            for (uint32_t e0 = group; e0 < have; e0 += 4 * groups) {
                uint32_t id[4];
                const float *v[4];
                float acc[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (uint32_t u = 0; u < 4; ++u) {
                    const uint32_t e = e0 + u * groups;
                    id[u] = list[e < have ? e : have - 1];
                    v[u] = data + (uint64_t)id[u] * n;
                }
                for (uint32_t c = piece0 * VEC; c < n; c += group_lanes * VEC) {
                    Piece<VEC> x[4];
#pragma unroll
                    for (uint32_t u = 0; u < 4; ++u) x[u] = read_piece<VEC>(v[u] + c);
                    const Piece<VEC> y = read_piece<VEC>((QUERY_IN_LDS ? query_lds : query) + c);
#pragma unroll
                    for (uint32_t u = 0; u < 4; ++u)
#pragma unroll
                        for (int e = 0; e < VEC; ++e) {
                            if constexpr (INNER) {
                                acc[u] = fmaf(-x[u].x[e], y.x[e], acc[u]);
                            } else {
                                const float d = x[u].x[e] - y.x[e];
                                acc[u] = fmaf(d, d, acc[u]);
                            }
                        }
                }
#pragma unroll
                for (uint32_t u = 0; u < 4; ++u) {
                    for (uint32_t s = group_lanes / 2; s > 0; s >>= 1) acc[u] += __shfl_xor(acc[u], s);
                    if (acc[u] < mine_d || (acc[u] == mine_d && id[u] < mine_id)) {  // the last one again: no change
                        mine_d = acc[u];
                        mine_id = id[u];
                    }
                }
            }
            __syncthreads();  // the list has been read
            if (tid == 0) listed = 0;
            __syncthreads();
        }
        left -= total;
    }
    for (uint32_t s = 32; s > 0; s >>= 1) {
        const float d = __shfl_xor(mine_d, s);
        const uint32_t id = __shfl_xor(mine_id, s);
        if (d < mine_d || (d == mine_d && id < mine_id)) {
            mine_d = d;
            mine_id = id;
        }
    }
    if (lane == 0) {
        wave_d[wave] = mine_d;
        wave_id[wave] = mine_id;
    }
    __syncthreads();
    if (tid == 0) {
        for (uint32_t w = 1; w < threads / 64; ++w)
            if (wave_d[w] < mine_d || (wave_d[w] == mine_d && wave_id[w] < mine_id)) {
                mine_d = wave_d[w];
                mine_id = wave_id[w];
            }
        best_id[q] = mine_id;
        best_dist[q] = INNER ? -mine_d : mine_d;  // no candidate: +inf distance, -inf inner product
    }
}

template <bool INNER>
void launch_nearest(const lsh_index *ix, const float *d_data, const float *d_queries, uint32_t n, const uint32_t *d_start,
                    const uint32_t *d_count, uint64_t Q, uint32_t limit, uint32_t *d_best_id, float *d_best_score,
                    hipStream_t s) {
    const bool pieces4 = n % 4 == 0 && ((reinterpret_cast<uintptr_t>(d_data) | reinterpret_cast<uintptr_t>(d_queries)) & 15) == 0;
    const uint32_t pieces = pieces4 ? n / 4 : n;
    uint32_t group_lanes = 8;
    while (group_lanes < 64 && group_lanes < pieces) group_lanes *= 2;
    // Up to a query for each of the 256 CUs: a workgroup as large as can be for each.  Up to three a CU, as many as run
    // at a time: half of that.  Beyond four a CU, the most of a quarter that run at a time: a quarter, because what a workgroup
    // spends around its candidates weighs most when they are few, and how many there are is on the device.  Between the two a
    // quarter where it fits all: limits that a query is soon done with, and vectors of whole waves.  With 256, 512,
    // 1024 threads, us: about 480 candidates a query of 960 dimensions, 128 queries 35, 21, 17; 400: 41, 32, 36; 900: 61, 65, 72;
    // 1300: 92, 85, 105; 4000: 228, 224, 271; 42 of them, few distinct, 4096: 25, 46; 96 candidates of 128 dimensions, 512:
    // 12.3, 12.6, 15.0; 1024: 14, 20, 30; 4000: 40, 57, 103; about 900 of them, 400: 94, 53, 54; 900: 113, 89, 92; 4000: 250, 228, 330.
    const bool soon_done = (uint64_t)limit * n <= 1u << 16, whole_waves = group_lanes == 64;
    const uint32_t threads = Q <= 256 ? kNearestThreads
                             : Q <= 768 || (Q <= 1024 && !soon_done && !whole_waves) ? kNearestThreads / 2 : kNearestThreads / 4;
    auto launch = [&](auto kernel, uint32_t lds) {
        hipLaunchKernelGGL(kernel, dim3((uint32_t)Q), dim3(threads), lds, s, ix->d_ids, ix->N, ix->L, d_data, d_queries, n,
                           group_lanes, d_start, d_count, limit, d_best_id, d_best_score);
    };
    const bool in_lds = n <= kQueryInLds;
    if (pieces4 && in_lds) launch(nearest_kernel<INNER, 4, true>, n * 4);
    else if (pieces4) launch(nearest_kernel<INNER, 4, false>, 0);
    else if (in_lds) launch(nearest_kernel<INNER, 1, true>, n * 4);
    else launch(nearest_kernel<INNER, 1, false>, 0);
}

int on_index_device(const lsh_index *ix) {
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess) return LSH_ERR_HIP;
    return dev == ix->device ? LSH_OK : LSH_ERR_INVALID_ARG;
}

}  // namespace

extern "C" {

int lsh_index_build(const uint64_t *d_keys, uint64_t N, uint32_t L, void *stream, lsh_index_t **out) {
    if (!out) return LSH_ERR_INVALID_ARG;
    *out = nullptr;
    if (!d_keys || !N || !L || N >= (1ull << 31) || L > 65535) return LSH_ERR_INVALID_ARG;  // positions are 32-bit, tables a grid row
    int count = 0;
    if (hipGetDeviceCount(&count) != hipSuccess || count <= 0) {
        (void)hipGetLastError();
        return LSH_ERR_NO_DEVICE;
    }
    // the (tile, table) workgroups of a pass are counted in 32 bits
    if (((N + kSortTile - 1) / kSortTile) * L >= (1ull << 31)) return LSH_ERR_UNSUPPORTED;
    lsh_index *ix = new (std::nothrow) lsh_index;
    if (!ix) return LSH_ERR_ALLOC;
    ix->N = N;
    ix->L = L;
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    const uint32_t tiles = (uint32_t)((N + kSortTile - 1) / kSortTile);
    const size_t pairs = (size_t)L * N;
    const bool by_buckets = lsh::bucket_sort_takes(N, L);
    // scratch: the other half of the ping-pong, and the (digit, tile) counts of every table
    const size_t scratch_bytes = by_buckets ? lsh::bucket_sort_scratch(N, L) : pairs * 12 + (size_t)L * 256 * (tiles + 1) * 4;
    lsh::IndexBlock scratch;
    uint64_t *tmp_keys = nullptr;
    uint32_t *tmp_ids = nullptr, *hist = nullptr, *total = nullptr;
    int rc = LSH_OK;
    if (hipGetDevice(&ix->device) != hipSuccess) {
        delete ix;
        return LSH_ERR_HIP;
    }
    lsh::index_memory_enter(ix->device);
    if (!lsh::index_memory_take(ix->device, pairs * 12, false, s, ix->tables)) rc = LSH_ERR_ALLOC;
    if (rc == LSH_OK && !lsh::index_memory_take(ix->device, scratch_bytes, true, s, scratch))
        rc = LSH_ERR_ALLOC;
    if (rc == LSH_OK) {
        ix->d_keys = static_cast<uint64_t *>(ix->tables.ptr);
        ix->d_ids = reinterpret_cast<uint32_t *>(ix->d_keys + pairs);
        tmp_keys = static_cast<uint64_t *>(scratch.ptr);
        tmp_ids = reinterpret_cast<uint32_t *>(tmp_keys + pairs);
        hist = tmp_ids + pairs;
        total = hist + (size_t)L * 256 * tiles;
    }
    if (rc == LSH_OK && by_buckets) {
        lsh::launch_bucket_sort(d_keys, N, L, scratch.ptr, ix->d_keys, ix->d_ids, s);
        if (hipGetLastError() != hipSuccess) rc = LSH_ERR_HIP;
    } else if (rc == LSH_OK) {
        const dim3 grid(tiles, L), block(kSortThreads);
        // eight passes; odd passes write the index's own arrays, so the last one ends there
        for (uint32_t pass = 0; pass < 8; ++pass) {
            const uint32_t shift = 8 * pass;
            const uint64_t *src_keys = (pass & 1) ? tmp_keys : ix->d_keys;
            const uint32_t *src_ids = (pass & 1) ? tmp_ids : ix->d_ids;
            uint64_t *dst_keys = (pass & 1) ? ix->d_keys : tmp_keys;
            uint32_t *dst_ids = (pass & 1) ? ix->d_ids : tmp_ids;
            if (pass == 0) {
                const uint32_t groups = (L + kRowColumns - 1) / kRowColumns, columns = (L + groups - 1) / groups;
                uint32_t width = 1;
                while (width < columns) width *= 2;
                hipLaunchKernelGGL(sort_columns, dim3(tiles, groups), dim3(kRowThreads), 0, s, d_keys, N, L, columns, width, tiles,
                                   hist, ix->d_keys);
            } else {
                hipLaunchKernelGGL(sort_histogram, grid, block, 0, s, src_keys, N, shift, tiles, hist);
            }
            hipLaunchKernelGGL(sort_scan, dim3(L * 64), dim3(256), 0, s, hist, tiles, L * 256, total);
            auto scatter = pass == 0 ? sort_scatter<true> : sort_scatter<false>;
            hipLaunchKernelGGL(scatter, grid, block, 0, s, src_keys, src_ids, N, shift, tiles, hist, total, dst_keys, dst_ids);
        }
        if (hipGetLastError() != hipSuccess) rc = LSH_ERR_HIP;
    }
    lsh::index_memory_give_scratch(ix->device, scratch, s);
    if (rc != LSH_OK) {
        (void)hipStreamSynchronize(s);
        (void)hipGetLastError();
        lsh_index_destroy(ix);
        return rc;
    }
    *out = ix;
    return LSH_OK;
}

void lsh_index_destroy(lsh_index_t *ix) {
    if (!ix) return;
    int prev = -1;  // the tables live on the device the index was built on
    const bool switched = ix->device >= 0 && hipGetDevice(&prev) == hipSuccess && prev != ix->device &&
                          hipSetDevice(ix->device) == hipSuccess;
    // work on any stream may still read the tables: wait for the device, as hipFree does
    if (lsh::index_memory_wait()) lsh::index_memory_give(ix->device, ix->tables);
    else (void)hipFree(ix->tables.ptr);
    lsh::index_memory_leave(ix->device);
    if (switched) (void)hipSetDevice(prev);
    delete ix;
}

int lsh_index_tables(const lsh_index_t *ix, uint64_t *N, uint32_t *L, const uint64_t **d_sorted_keys,
                     const uint32_t **d_sorted_ids) {
    if (!ix) return LSH_ERR_INVALID_ARG;
    if (N) *N = ix->N;
    if (L) *L = ix->L;
    if (d_sorted_keys) *d_sorted_keys = ix->d_keys;
    if (d_sorted_ids) *d_sorted_ids = ix->d_ids;
    return LSH_OK;
}

int lsh_index_probe(const lsh_index_t *ix, const uint64_t *d_qkeys, uint64_t Q, uint32_t *d_start, uint32_t *d_count,
                    void *stream) {
    if (!ix) return LSH_ERR_INVALID_ARG;
    if (Q == 0) return LSH_OK;
    if (!d_qkeys || !d_start || !d_count) return LSH_ERR_INVALID_ARG;
    int rc = on_index_device(ix);
    if (rc != LSH_OK) return rc;
    const uint64_t items = Q * ix->L;
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    auto launch = [&](auto kernel, uint32_t lanes) {
        const uint64_t wanted = (items * lanes + 255) / 256;  // one group per item, up to 2^20 workgroups
        hipLaunchKernelGGL(kernel, dim3((uint32_t)(wanted < (1u << 20) ? wanted : (1u << 20))), dim3(256), 0, s, ix->d_keys,
                           ix->N, ix->L, d_qkeys, items, d_start, d_count);
    };
    const uint64_t blocks = (Q * kManyLanes + 255) / 256;
    if (items <= kFewLookups) {
        launch(probe_kernel<kFewLanes>, kFewLanes);
    } else if (ix->N * ix->L > 2 * kTablesOfL2 && Q >= 128 && ix->L >= 8 && Q < (1u << 24) && blocks * ix->L < (1u << 24)) {
        hipLaunchKernelGGL(probe_tables_kernel<kManyLanes>, dim3((uint32_t)(blocks * ix->L)), dim3(256), 0, s, ix->d_keys, ix->N,
                           ix->L, d_qkeys, (uint32_t)Q, (uint32_t)blocks, d_start, d_count);
    } else {
        launch(probe_kernel<kManyLanes>, kManyLanes);
    }
    return hipGetLastError() == hipSuccess ? LSH_OK : LSH_ERR_HIP;
}

int lsh_index_candidate_offsets(const uint32_t *d_count, uint64_t items, uint64_t *d_offsets, void *stream) {
    if (!d_offsets || (items && !d_count) || items >= (1ull << 31)) return LSH_ERR_INVALID_ARG;
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    uint64_t *partial = nullptr;
    int rc = LSH_OK;
    if (hipMalloc(&partial, (items / kScanBlock + 1) * sizeof(uint64_t)) != hipSuccess) rc = LSH_ERR_ALLOC;
    if (rc == LSH_OK) rc = launch_offsets_scan(d_count, items, partial, d_offsets, s);
    if (rc == LSH_OK && hipStreamSynchronize(s) != hipSuccess) rc = LSH_ERR_HIP;
    if (partial) (void)hipFree(partial);
    if (rc != LSH_OK) (void)hipGetLastError();
    return rc;
}

int lsh_index_candidate_offsets_static(const uint32_t *d_count, uint64_t items, uint64_t *d_offsets, void *stream) {
    if (!d_offsets || (items && !d_count)) return LSH_ERR_INVALID_ARG;
    if (items > kStaticScanItems) return LSH_ERR_UNSUPPORTED;
    uint64_t *partial = static_scratch();
    if (!partial) return LSH_ERR_HIP;
    return launch_offsets_scan(d_count, items, partial, d_offsets, reinterpret_cast<hipStream_t>(stream));
}

int lsh_index_candidates(const lsh_index_t *ix, const uint32_t *d_start, const uint32_t *d_count,
                         const uint64_t *d_offsets, uint64_t Q, uint32_t *d_out, void *stream) {
    if (!ix) return LSH_ERR_INVALID_ARG;
    if (Q == 0) return LSH_OK;
    if (!d_start || !d_count || !d_offsets || !d_out) return LSH_ERR_INVALID_ARG;
    int rc = on_index_device(ix);
    if (rc != LSH_OK) return rc;
    const uint64_t items = Q * ix->L;
    const uint64_t wanted = (items * 64 + 255) / 256;  // one wave per item, up to 2^20 workgroups
    hipLaunchKernelGGL(candidates_kernel, dim3((uint32_t)(wanted < (1u << 20) ? wanted : (1u << 20))), dim3(256), 0,
                       reinterpret_cast<hipStream_t>(stream), ix->d_ids, ix->N, ix->L, d_start, d_count, d_offsets, items,
                       d_out);
    return hipGetLastError() == hipSuccess ? LSH_OK : LSH_ERR_HIP;
}

static int best_candidate(bool inner, const lsh_index_t *ix, const float *d_data, const float *d_queries, uint32_t n,
                          const uint32_t *d_start, const uint32_t *d_count, uint64_t Q, uint32_t max_candidates,
                          uint32_t *d_best_id, float *d_best_score, void *stream) {
    if (!ix || !n) return LSH_ERR_INVALID_ARG;
    if (Q == 0) return LSH_OK;
    if (!d_data || !d_queries || !d_start || !d_count || !d_best_id || !d_best_score) return LSH_ERR_INVALID_ARG;
    if (Q >= (1ull << 31)) return LSH_ERR_INVALID_ARG;
    if ((uint64_t)n * 4 + 64 > 64 * 1024) return LSH_ERR_UNSUPPORTED;
    int rc = on_index_device(ix);
    if (rc != LSH_OK) return rc;
    const uint32_t limit = max_candidates ? max_candidates : 0xFFFFFFFFu;
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    if (inner) launch_nearest<true>(ix, d_data, d_queries, n, d_start, d_count, Q, limit, d_best_id, d_best_score, s);
    else launch_nearest<false>(ix, d_data, d_queries, n, d_start, d_count, Q, limit, d_best_id, d_best_score, s);
    return hipGetLastError() == hipSuccess ? LSH_OK : LSH_ERR_HIP;
}

int lsh_index_nearest(const lsh_index_t *ix, const float *d_data, const float *d_queries, uint32_t n,
                      const uint32_t *d_start, const uint32_t *d_count, uint64_t Q, uint32_t max_candidates,
                      uint32_t *d_best_id, float *d_best_dist, void *stream) {
    return best_candidate(false, ix, d_data, d_queries, n, d_start, d_count, Q, max_candidates, d_best_id, d_best_dist,
                          stream);
}

int lsh_index_best_inner_product(const lsh_index_t *ix, const float *d_data, const float *d_queries, uint32_t n,
                                 const uint32_t *d_start, const uint32_t *d_count, uint64_t Q,
                                 uint32_t max_candidates, uint32_t *d_best_id, float *d_best_ip, void *stream) {
    return best_candidate(true, ix, d_data, d_queries, n, d_start, d_count, Q, max_candidates, d_best_id, d_best_ip,
                          stream);
}

}  // extern "C"
