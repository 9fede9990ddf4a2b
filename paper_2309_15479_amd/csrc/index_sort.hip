// The tables of an index: every column of the keys [N][L] sorted, with the row numbers.
//
//   sort_splitters  per table: a sample of its keys, sorted; every 16th is a splitter between two buckets
//   sort_tiles      per tile of 4096 rows and table: the pairs in the order of their buckets, to scratch in one
//                   piece, with the place where each bucket begins
//   sort_buckets    per bucket: its runs from all tiles, in the order of the tiles, sorted in LDS and written
//                   (sort_medium_buckets, sort_large_buckets: those that are too much for that)
//
// A pair is read twice and written twice, where the radix sort by eight digits (index.hip) reads it sixteen times and
// writes it eight times.  The buckets need neither a count of the whole table before they are filled nor
// room kept free: they stay spread over the tiles until the launch that reads them, to which the tiles'
// offsets also say where a bucket begins in the table (the sum over the tiles of the pairs ahead of it).
// Splitters from a sample, not the keys' top bits: keys of few functions, or of one, differ in their low bits
// only.  A key that fills a bucket of the sample is kept from its neighbours by a second splitter right
// above it.  How well the sample was met costs time only: a bucket that LDS does not hold is sorted part by part.
// Measured, the radix sort -> this, us: 1e6 x 32 keys of the SIFT shape 2630 -> 890 (splitters 49, tiles 206, buckets 585 at 61 % of
// the issue slots, the larger ones 31), random keys 1e6 x 2 227 -> 132, 1e5 x 64 625 -> 224, 1e4 x 32 214 -> 74, 1000 x 64
// 169 -> 55, one key 1e6 times x 32 2160 -> 462.  Up to 2^20 pairs a table (1048576 x 8: 670 -> 285): beyond that a tile has more
// buckets, or a bucket more pairs, than a workgroup has room for, and the radix sort stays (1.1e6 x 8: 765).
#include "index_sort.h"

#include <utility>

namespace lsh {
namespace {

// Tiles: 4096 rows, so that a row's number in its tile takes 16 bits.  Four tables a workgroup: pieces of 32 bytes of a
// row, all loaded before the first is ranked.  Eight rows a thread: with four, and twice the threads, some of their keys do
// not fit the 64 registers (219 us instead of 206, and 65 MB of scratch memory written).
constexpr uint32_t kTileThreads = 512, kTileSlots = 8, kTileRows = kTileThreads * kTileSlots, kTileColumns = 4;
// Buckets: 2048 pairs and less on average, up to 4096 in LDS, three workgroups a CU.  A workgroup of four waves: what a pass
// costs beside the ranking of the pairs, it costs once a wave.  (256 buckets of twice the size, two workgroups of 16 waves: 95
// registers' worth of pairs in 64.)
constexpr uint32_t kMaxBuckets = 512, kBucketMean = 2048, kBucketThreads = 256, kSlots = 16;
constexpr uint32_t kBucketCap = kBucketThreads * kSlots;
constexpr uint32_t kLargeThreads = 1024, kLargeSlots = 8, kLargeCap = kLargeThreads * kLargeSlots;  // those that are more
constexpr uint32_t kMaxTiles = kMaxBuckets * kBucketMean / kTileRows;
// The sample: 16 keys a bucket, as many as one workgroup sorts.
constexpr uint32_t kSampleThreads = 1024, kSampleSlots = 8, kSamples = kSampleThreads * kSampleSlots / kMaxBuckets;
static_assert(kSamples >= 2 && kSamples <= kBucketThreads, "a sample of more rows than there are");
static_assert(kMaxTiles == 256 && kBucketThreads >= 256 && kTileRows <= 65536, "runs of a bucket: a thread each; numbers in a tile: 16 bits");

struct Plan {
    uint32_t tiles, buckets;
    uint64_t stride;
};

Plan plan_of(uint64_t N, uint32_t L) {
    Plan p;
    p.tiles = (uint32_t)((N + kTileRows - 1) / kTileRows);
    p.buckets = 1;
    while ((uint64_t)p.buckets * kBucketMean < N) p.buckets *= 2;
    // few tables: smaller buckets, down to a pair a thread, until every CU has some
    while (p.buckets < kMaxBuckets && (uint64_t)p.buckets * L < 512 && (uint64_t)p.buckets * 2 * kBucketThreads <= N) p.buckets *= 2;
    p.stride = (N + 7) & ~7ull;
    return p;
}

// What sort_tiles leaves: [L][stride] keys and row numbers within their tiles, where each bucket begins in each tile
// ([L][tiles][buckets + 1]), and the splitters it went by ([L][buckets]; bucket b ends below cuts[b]).
struct SortedTiles {
    uint64_t *keys;
    uint16_t *ids, *offsets;
    uint64_t *cuts;
    uint64_t N, stride;  // pairs of a table; from one table to the next
    uint32_t tiles, buckets;
};

__device__ __forceinline__ uint32_t lane_id() { return threadIdx.x & 63; }
__device__ __forceinline__ uint32_t wave_id() { return threadIdx.x >> 6; }
__device__ __forceinline__ uint32_t uniform(uint32_t x) { return __builtin_amdgcn_readfirstlane(x); }

// Orders a wave's LDS accesses as written; no instruction.
__device__ __forceinline__ void wave_order() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

__device__ __forceinline__ uint32_t spread_bit(uint32_t x, uint32_t b) {
#ifdef __HIP_DEVICE_COMPILE__
    uint32_t r = (uint32_t)__builtin_amdgcn_sbfe((int)x, b, 1);
    asm("" : "+v"(r));  // (the compiler would test the bit a second time, in place, for the ballot)
    return r;
#else
    return 0u - ((x >> b) & 1u);
#endif
}

// Lanes among `valid` whose low `bits` (up to MOST) bits of `digit` are this lane's.  Four instructions a bit: the bit
// spread over a word, its ballot, and either half of the lanes taken where ballot and bit agree.
template <uint32_t MOST>
__device__ __forceinline__ uint64_t same_digit(uint32_t digit, uint32_t bits, uint64_t valid) {
    uint32_t low = (uint32_t)valid, high = (uint32_t)(valid >> 32);
#pragma unroll
    for (uint32_t b = 0; b < MOST; ++b) {
        if (b < bits) {
            const uint32_t mine = spread_bit(digit, b);
            const uint64_t set = __ballot(mine != 0);
            low &= ~((uint32_t)set ^ mine);
            high &= ~((uint32_t)(set >> 32) ^ mine);
        }
    }
    return (uint64_t)high << 32 | low;
}

// Per digit and wave: pairs seen so far, then the place of the first.  An odd number of words from one digit to the next: a wave's
// lanes, each at its digit, and the threads that add up a digit's waves, two at a time, hit different banks.
template <uint32_t WAVES, uint32_t DIGITS>
struct Counters {
    static constexpr uint32_t kStride = WAVES + 2, kWaves = WAVES, kDigits = DIGITS, kThreads = WAVES * 64;
    static_assert(WAVES % 4 == 0 && DIGITS % 64 == 0 && DIGITS <= kThreads, "");
    __align__(8) uint16_t of[DIGITS * kStride];
    uint32_t total[DIGITS / 64];

    __device__ __forceinline__ uint16_t &mine(uint32_t digit) { return of[digit * kStride + wave_id()]; }

    // Number of this lane's pair among its wave's pairs of the same digit, in the order of slots and lanes; adds the
    // slot's pairs to the wave's counters.  (Ranks from ballots: equal digits, which equal keys have, cost no more.)
    template <uint32_t MOST>
    __device__ __forceinline__ uint32_t rank(uint32_t digit, uint32_t bits, bool valid) {
        const uint64_t peers = same_digit<MOST>(digit, bits, __ballot(valid));
        const uint32_t before = __builtin_amdgcn_mbcnt_hi((uint32_t)(peers >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)peers, 0));
        uint16_t &counter = mine(digit);
        const uint32_t seen = counter;
        wave_order();
        if (valid && before == 0) counter = (uint16_t)(seen + (uint32_t)__popcll(peers));
        wave_order();
        __builtin_amdgcn_sched_barrier(0);
        return seen + before;
    }

    // by all threads, with a barrier after
    __device__ __forceinline__ void clear() {
        uint32_t *const words = reinterpret_cast<uint32_t *>(of);
#pragma unroll
        for (uint32_t e = threadIdx.x; e < DIGITS * kStride / 2; e += kThreads) words[e] = 0;
    }

    // Inclusive sum over the first DIGITS threads; all threads call it.
    __device__ __forceinline__ uint32_t scan(uint32_t mine) {
        uint32_t incl = mine;
        if (threadIdx.x < DIGITS) {
#pragma unroll
            for (uint32_t step = 1; step < 64; step <<= 1) {
                const uint32_t up = __shfl_up(incl, step);
                if (lane_id() >= step) incl += up;
            }
            if (lane_id() == 63) total[wave_id()] = incl;
        }
        __syncthreads();
        if (threadIdx.x < DIGITS)
            for (uint32_t w = 0; w < wave_id(); ++w) incl += total[w];
        return incl;
    }

    // Pairs per digit and wave -> place of the first of them; for thread d < DIGITS the place of the digit's first pair.
    // The counters are complete (barrier before); barrier at the end.
    __device__ __forceinline__ uint32_t to_places() {
        uint32_t *const two = reinterpret_cast<uint32_t *>(of + (threadIdx.x & (DIGITS - 1)) * kStride);
        uint32_t pairs[WAVES / 2], here = 0;
        if (threadIdx.x < DIGITS) {
#pragma unroll
            for (uint32_t w = 0; w < WAVES / 2; ++w) {
                pairs[w] = two[w];
                here += (pairs[w] & 0xFFFF) + (pairs[w] >> 16);
            }
        }
        const uint32_t start = scan(here) - here;
        if (threadIdx.x < DIGITS) {
            uint32_t at = start;
#pragma unroll
            for (uint32_t w = 0; w < WAVES / 2; ++w) {
                const uint32_t next = at + (pairs[w] & 0xFFFF);
                two[w] = at | next << 16;
                at = next + (pairs[w] >> 16);
            }
        }
        __syncthreads();
        return start;
    }
};

// The pairs of a workgroup: `slots` each thread, pair `slot` of a lane being number
// wave * slots * 64 + slot * 64 + lane.
struct Share {
    uint32_t first, slots;
    int left;
    __device__ Share(uint32_t count, uint32_t threads)
        : first(0), slots((count + threads - 1) / threads), left(0) {
        first = wave_id() * slots * 64 + lane_id();
        const int of_wave = (int)(slots * 64 - lane_id()), of_all = (int)count - (int)first;
        left = of_wave < of_all ? of_wave : of_all;
    }
    __device__ __forceinline__ uint32_t number(uint32_t slot) const { return first + slot * 64; }
    __device__ __forceinline__ bool has(uint32_t slot) const { return (int)(slot * 64) < left; }
};

// Cells that sort leaves out of order: kListed pairs at most.
constexpr uint32_t kListed = 512, kOnList = 0x80000000u;

// A workgroup's sort of up to THREADS * SLOTS pairs.
template <uint32_t THREADS, uint32_t SLOTS>
struct Sorter {
    static constexpr uint32_t kWaves = THREADS / 64;
    uint64_t words[THREADS * SLOTS];  // keys on their way from one order to the next
    uint16_t from[THREADS * SLOTS];   // and which pair each was
    union {
        Counters<kWaves, 256> counter;
        struct {  // pairs of cells out of order, between two uses of the counters
            uint64_t key[kListed];
            uint16_t place[kListed], to[kListed];
        } list;
    };
    uint32_t dirty[256];  // a bit for every 8192nd cell
    uint32_t flag, listed;

    // Smallest and largest of what the threads bring.  Barriers in front of the exchange and behind it.
    __device__ __forceinline__ void range(uint64_t &low, uint64_t &high) {
#pragma unroll
        for (uint32_t step = 32; step > 0; step >>= 1) {
            const uint64_t a = __shfl_xor(low, step), b = __shfl_xor(high, step);
            low = a < low ? a : low;
            high = b > high ? b : high;
        }
        __syncthreads();
        if (lane_id() == 0) words[wave_id()] = low, words[kWaves + wave_id()] = high;
        __syncthreads();
        for (uint32_t w = 0; w < kWaves; ++w) {
            low = words[w] < low ? words[w] : low;
            high = words[kWaves + w] > high ? words[kWaves + w] : high;
        }
        low = (uint64_t)uniform((uint32_t)(low >> 32)) << 32 | uniform((uint32_t)low);
        high = (uint64_t)uniform((uint32_t)(high >> 32)) << 32 | uniform((uint32_t)high);
        __syncthreads();
    }

    // Sorts the workgroup's pairs by key, stably, all keys being in [low, high]; order[]: which pair has come to be where.
    // Keys that span no more than 24 bits: a pass for every 8.  Others: the lowest 8 bits, then those from 32 up, or the top 16
    // where these are fewer.  Keys of one bucket differ at random from one another, or, where all functions of the
    // table but the last agree, by a small number, or by 2^32 less a small number (an id enters a key as 32 unsigned bits); what is
    // still out of order after that are a few cells of equal top bits, whose pairs are put in order by
    // counting.  If those are more than kListed, all digits are sorted.  (1e6 x 32 keys of the SIFT shape, 1950 a bucket, four passes:
    // 26 pairs in 1 bucket of 6, more than kListed in 1 of 1000.  Digits from the top alone, two: 95 cells of 2900 pairs in 3900.)
    // Barrier before the call where the counters were in use; at the end `words` and `from` are free.
    template <bool ORDER>
    __device__ __forceinline__ void sort(const Share share, uint64_t low, uint64_t high, uint64_t (&key)[SLOTS],
                                         uint32_t (&order)[SLOTS]) {
        if constexpr (ORDER) {
#pragma unroll
            for (uint32_t i = 0; i < SLOTS; ++i) order[i] = share.number(i);
        }
        if (low >= high) return;
        const int bits = 64 - __clzll((long long)(high - low));
        bool part = bits > 24;
        const int cell = bits > 48 ? 32 : bits - 16;  // part: keys of one cell differ below this bit
        counter.clear();
        __syncthreads();
#pragma unroll
        for (uint32_t i = 0; i < SLOTS; ++i) key[i] -= low;
        for (int shift = 0; shift < bits; shift = part && shift == 0 ? cell : shift + 8) {
            uint32_t place[SLOTS];
#pragma unroll
            for (uint32_t i = 0; i < SLOTS; ++i)
                if (i < share.slots) place[i] = counter.template rank<8>((uint32_t)(key[i] >> shift) & 255u, 8, share.has(i));
            if (threadIdx.x < 256) dirty[threadIdx.x] = 0;
            if (threadIdx.x == 0) flag = listed = 0;
            __syncthreads();
            counter.to_places();
#pragma unroll
            for (uint32_t i = 0; i < SLOTS; ++i)
                if (share.has(i)) {
                    place[i] += counter.mine((uint32_t)(key[i] >> shift) & 255u);
                    words[place[i]] = key[i];
                    if constexpr (ORDER) from[place[i]] = (uint16_t)order[i];
                }
            __syncthreads();
            if (part && shift + 8 >= bits) {
                // cells are in order; a key below its neighbour shows a cell that is not in order itself
                bool out_of_order = false;
#pragma unroll
                for (uint32_t i = 0; i < SLOTS; ++i)
                    if (share.has(i) && place[i] > 0 && words[place[i] - 1] > key[i]) {
                        const uint32_t bit = (uint32_t)(key[i] >> cell) & 8191u;
                        atomicOr(&dirty[bit >> 5], 1u << (bit & 31));
                        out_of_order = true;
                    }
                if (out_of_order) atomicOr(&flag, 1u);
                __syncthreads();
                if (uniform(flag)) {
                    // the pairs of such cells on a list, and each one's place from a walk through it
#pragma unroll
                    for (uint32_t i = 0; i < SLOTS; ++i)
                        if (share.has(i)) {
                            const uint32_t bit = (uint32_t)(key[i] >> cell) & 8191u;
                            if (dirty[bit >> 5] >> (bit & 31) & 1u) {
                                const uint32_t e = atomicAdd(&listed, 1u);
                                if (e < kListed) list.key[e] = key[i], list.place[e] = (uint16_t)place[i];
                                place[i] = kOnList | e;
                            }
                        }
                    __syncthreads();
                    const uint32_t entries = uniform(listed);
                    if (entries > kListed) {  // all digits, from the keys as they stood before this pass
                        __syncthreads();
                        counter.clear();
                        __syncthreads();
                        part = false;
                        shift = -8;
                        continue;  // the loop adds 8
                    }
                    for (uint32_t own = threadIdx.x; own < entries; own += THREADS) {
                        const uint64_t mine = list.key[own], begin = mine >> cell << cell, end = begin | ((1ull << cell) - 1);
                        const uint32_t at = list.place[own];
                        uint32_t to = at;
#pragma unroll 4
                        for (uint32_t e = 0; e < entries; ++e) {
                            const uint64_t k = list.key[e];
                            const bool ahead = list.place[e] < at, same = k >= begin && k <= end;
                            to += same && (k < mine || (k == mine && ahead)) ? 1u : 0u;
                            to -= same && ahead ? 1u : 0u;
                        }
                        list.to[own] = (uint16_t)to;
                    }
                    __syncthreads();
#pragma unroll
                    for (uint32_t i = 0; i < SLOTS; ++i)
                        if (share.has(i) && (place[i] & kOnList)) {
                            const uint32_t to = list.to[place[i] & ~kOnList];
                            words[to] = key[i];
                            if constexpr (ORDER) from[to] = (uint16_t)order[i];
                        }
                    __syncthreads();
                }
            }
            counter.clear();
#pragma unroll
            for (uint32_t i = 0; i < SLOTS; ++i)
                if (share.has(i)) {
                    key[i] = words[share.number(i)];
                    if constexpr (ORDER) order[i] = from[share.number(i)];
                }
            __syncthreads();
        }
#pragma unroll
        for (uint32_t i = 0; i < SLOTS; ++i) key[i] += low;
    }
};

// One workgroup per table: cuts[l][b] for b < buckets - 1 ascending; bucket b holds the keys from cuts[b - 1] on, below
// cuts[b].
__global__ __launch_bounds__(kSampleThreads) void sort_splitters(const uint64_t *__restrict__ keys, uint64_t N, uint32_t L,
                                                                 uint32_t buckets, uint64_t *__restrict__ cuts) {
    __shared__ Sorter<kSampleThreads, kSampleSlots> sh;
    const uint32_t l = blockIdx.x, count = buckets * kSamples;  // more rows than that: plan_of leaves 256 and more a bucket
    const Share share(count, kSampleThreads);
    uint64_t key[kSampleSlots], low = ~0ull, high = 0;
    uint32_t unused[kSampleSlots];
#pragma unroll
    for (uint32_t i = 0; i < kSampleSlots; ++i)
        if (i < share.slots) {  // one row of every count-th part of the table, at a place that follows no pattern of the rows
            const uint64_t j = share.number(i) < count ? share.number(i) : count - 1;
            const uint64_t first = j * N / count, room = (j + 1) * N / count - first;
            const uint32_t mixed = ((uint32_t)j * 0x9E3779B1u ^ 0x85EBCA6Bu) * 0xC2B2AE35u;
            key[i] = keys[(first + (((mixed ^ mixed >> 15) * (uint64_t)room) >> 32)) * L + l];
        }
#pragma unroll
    for (uint32_t i = 0; i < kSampleSlots; ++i)
        if (share.has(i)) {
            low = key[i] < low ? key[i] : low;
            high = key[i] > high ? key[i] : high;
        }
    sh.range(low, high);
    sh.sort<false>(share, low, high, key, unused);
#pragma unroll
    for (uint32_t i = 0; i < kSampleSlots; ++i)
        if (share.has(i)) sh.words[share.number(i)] = key[i];
    __syncthreads();
    constexpr uint32_t half = kSamples / 2;
    for (uint32_t b = threadIdx.x + 1; b < buckets; b += kSampleThreads) {
        const uint32_t at = b * kSamples;
        const uint64_t cut = sh.words[at];
        // A key met at the splitter before too: it has a bucket of its own, which ends here.  One that lies more ahead of
        // this place than behind it goes to the bucket ahead.
        const bool again = b > 1 && sh.words[at - kSamples] == cut;
        const bool ahead = sh.words[at - half] == cut && sh.words[at + half] != cut;
        cuts[(uint64_t)l * buckets + b - 1] = (again || ahead) && cut != ~0ull ? cut + 1 : cut;
    }
}

// The buckets that are more pairs than the launch in front of this one sorts; those of one key in parts of kLargeCap.
struct BucketList {
    uint32_t count, unused;
    struct {
        uint32_t bucket, part;
    } entry[1];
};
// entries: every bucket once, and once more for every kLargeCap pairs of its table
size_t list_bytes(uint64_t N, uint32_t L, uint32_t buckets) { return 8 + (size_t)L * (buckets + N / kLargeCap) * 8; }

// One workgroup per tile and four tables.  Bound by what it moves (8 bytes in, 10 out a pair) and by the search
// and the ranking, some 100 vector instructions a pair; the loads of all four columns are in flight before
// the first is ranked.  The workgroups of a tile run on the same XCD: they read the same lines.
template <bool PAIRS>
__global__ __launch_bounds__(kTileThreads, 4) void sort_tiles(const uint64_t *__restrict__ keys, uint32_t L, uint32_t groups,
                                                              uint32_t bucket_bits, const SortedTiles out,
                                                              BucketList *__restrict__ medium,
                                                              BucketList *__restrict__ large) {
    __shared__ uint64_t cut[kTileColumns][kMaxBuckets];
    __shared__ Counters<kTileThreads / 64, kMaxBuckets> counter;
    __shared__ __align__(16) uint64_t out_keys[kTileRows];
    __shared__ __align__(16) uint16_t out_ids[kTileRows];
    const uint32_t tile = blockIdx.x / (8 * groups) * 8 + (blockIdx.x & 7), l0 = (blockIdx.x / 8) % groups * kTileColumns;
    if (blockIdx.x == 0 && threadIdx.x == 0) medium->count = large->count = 0;
    if (tile >= out.tiles) return;
    const uint32_t here = L - l0 < kTileColumns ? L - l0 : kTileColumns, buckets = 1u << bucket_bits;
    const uint64_t first = (uint64_t)tile * kTileRows;
    const uint32_t rows = (uint32_t)(out.N - first < kTileRows ? out.N - first : kTileRows);
    const uint32_t row0 = wave_id() * (kTileSlots * 64) + lane_id();
    uint64_t key[kTileSlots][kTileColumns];
#pragma unroll
    for (uint32_t i = 0; i < kTileSlots; ++i) {
        const uint32_t row = row0 + i * 64;
        const uint64_t *at = keys + (first + (row < rows ? row : rows - 1)) * L + l0;
        if constexpr (PAIRS) {
#pragma unroll
            for (uint32_t c = 0; c < kTileColumns; c += 2) {
                const ulonglong2 two = *reinterpret_cast<const ulonglong2 *>(at + (c < here ? c : 0));
                key[i][c] = two.x;
                key[i][c + 1] = two.y;
            }
        } else {
#pragma unroll
            for (uint32_t c = 0; c < kTileColumns; ++c) key[i][c] = at[c < here ? c : 0];
        }
    }
    for (uint32_t e = threadIdx.x; e < here * kMaxBuckets; e += kTileThreads) {
        const uint32_t c = e / kMaxBuckets, b = e % kMaxBuckets;
        // node b of a search tree, node 1 its root, the children of b 2 b and 2 b + 1: the nodes of a level, which the lanes read
        // at the same time, lie side by side (in ascending order they are a power of two apart, in one bank)
        const uint32_t level = 31 - __builtin_clz(b | 1), step = buckets >> level;
        if (b > 0 && b < buckets) cut[c][b] = out.cuts[(uint64_t)(l0 + c) * buckets + (b - (1u << level)) * step + step / 2 - 1];
    }
    counter.clear();
#pragma unroll
    for (uint32_t c = 0; c < kTileColumns; ++c) {
        if (c >= here) break;
        __syncthreads();  // the cuts are there, the counters are clear, the column before has been written out
        uint32_t bucket[kTileSlots], place[kTileSlots];
#pragma unroll
        for (uint32_t i = 0; i < kTileSlots; ++i) bucket[i] = 1;
#pragma unroll 1
        for (uint32_t level = 0; level < bucket_bits; ++level) {
#pragma unroll
            for (uint32_t i = 0; i < kTileSlots; ++i) bucket[i] = 2 * bucket[i] + (cut[c][bucket[i]] <= key[i][c] ? 1 : 0);
        }
#pragma unroll
        for (uint32_t i = 0; i < kTileSlots; ++i) bucket[i] -= buckets;
#pragma unroll
        for (uint32_t i = 0; i < kTileSlots; ++i) place[i] = counter.template rank<9>(bucket[i], bucket_bits, row0 + i * 64 < rows);
        __syncthreads();
        const uint32_t start = counter.to_places();
        const uint32_t l = l0 + c;
        uint16_t *const to = out.offsets + ((uint64_t)l * out.tiles + tile) * (buckets + 1);
        if (threadIdx.x < buckets) to[threadIdx.x] = (uint16_t)start;
        if (threadIdx.x == 0) to[buckets] = (uint16_t)rows;
#pragma unroll
        for (uint32_t i = 0; i < kTileSlots; ++i)
            if (row0 + i * 64 < rows) {
                place[i] += counter.mine(bucket[i]);
                out_keys[place[i]] = key[i][c];
                out_ids[place[i]] = (uint16_t)(row0 + i * 64);
            }
        __syncthreads();
        counter.clear();
        // whole pieces of 16 bytes: the arrays have room for them behind the last pair of a table
        const uint64_t at = l * out.stride + first;
#pragma unroll 1
        for (uint32_t e = threadIdx.x * 2; e < rows; e += kTileThreads * 2)
            *reinterpret_cast<ulonglong2 *>(out.keys + at + e) = *reinterpret_cast<const ulonglong2 *>(out_keys + e);
        for (uint32_t e = threadIdx.x * 8; e < rows; e += kTileThreads * 8)
            *reinterpret_cast<uint4 *>(out.ids + at + e) = *reinterpret_cast<const uint4 *>(out_ids + e);
    }
}

// The runs of a bucket in the tiles: pair p of the bucket, in run t, is pair p + ahead[t] of the table's tiles; run t begins at
// pair begin[t], the runs of no tile behind all pairs.
struct Runs {
    uint32_t begin[kMaxTiles], ahead[kMaxTiles], count, of_smaller;

    __device__ __forceinline__ uint32_t run_of(uint32_t p) const {
        uint32_t t = 0;
#pragma unroll
        for (uint32_t half = 128; half > 0; half >>= 1)
            if (begin[t + half] <= p) t += half;
        return t;
    }
};

struct Bucket {
    const uint64_t *keys;
    const uint16_t *ids;
    uint64_t out, low, high;  // its first place in the sorted tables; its keys are in [low, high]
    uint32_t count;
};

template <class COUNTERS>
__device__ __forceinline__ Bucket find_bucket(Runs &runs, COUNTERS &scratch, const SortedTiles &in, uint32_t item) {
    const uint32_t l = item / in.buckets, b = item - l * in.buckets;
    uint32_t from = 0, length = 0;
    if (threadIdx.x < in.tiles) {
        const uint16_t *at = in.offsets + ((uint64_t)l * in.tiles + threadIdx.x) * (in.buckets + 1) + b;
        from = at[0];
        length = at[1] - from;
    }
    const uint64_t *const cuts = in.cuts + (uint64_t)l * in.buckets;
    const uint64_t low = b ? cuts[b - 1] : 0, high = b + 1 < in.buckets ? cuts[b] - 1 : ~0ull;
    const uint32_t end = scratch.scan(length);
    __syncthreads();
    const uint32_t smaller = scratch.scan(from);
    if (threadIdx.x < 256) {
        runs.begin[threadIdx.x] = threadIdx.x < in.tiles ? end - length : ~0u;
        runs.ahead[threadIdx.x] = threadIdx.x * kTileRows + from - (end - length);
        if (threadIdx.x == 255) runs.count = end, runs.of_smaller = smaller;
    }
    __syncthreads();
    return {in.keys + l * in.stride, in.ids + l * in.stride, (uint64_t)l * in.N + uniform(runs.of_smaller), low, high,
            uniform(runs.count)};
}

// A workgroup sorts a bucket, or puts it on the list of larger ones.
template <uint32_t THREADS, uint32_t SLOTS>
__device__ __forceinline__ void sort_bucket(Sorter<THREADS, SLOTS> &sh, const Runs &runs, const Bucket &bucket, uint32_t item,
                                            BucketList *__restrict__ larger, uint64_t *__restrict__ sorted_keys,
                                            uint32_t *__restrict__ sorted_ids) {
    if (bucket.count == 0) return;
    if (bucket.count > THREADS * SLOTS) {
        if (threadIdx.x == 0) {
            const uint32_t parts = bucket.low == bucket.high ? (bucket.count + kLargeCap - 1) / kLargeCap : 1;
            const uint32_t at = atomicAdd(&larger->count, parts);
            for (uint32_t p = 0; p < parts; ++p) larger->entry[at + p] = {item, p};
        }
        return;
    }
    const Share share(bucket.count, THREADS);
    uint64_t key[SLOTS];
    uint32_t id[SLOTS], order[SLOTS];
    constexpr uint32_t kTogether = 4;  // searches of as many pairs side by side: each is a chain of eight reads
#pragma unroll
    for (uint32_t i0 = 0; i0 < SLOTS; i0 += kTogether)
        if (i0 < share.slots) {
            uint32_t p[kTogether], t[kTogether] = {};
#pragma unroll
            for (uint32_t u = 0; u < kTogether; ++u) p[u] = share.has(i0 + u) ? share.number(i0 + u) : bucket.count - 1;
#pragma unroll
            for (uint32_t half = kMaxTiles / 2; half > 0; half >>= 1)
#pragma unroll
                for (uint32_t u = 0; u < kTogether; ++u)
                    if (runs.begin[t[u] + half] <= p[u]) t[u] += half;
#pragma unroll
            for (uint32_t u = 0; u < kTogether; ++u) {
                const uint32_t at = p[u] + runs.ahead[t[u]];
                key[i0 + u] = bucket.keys[at];
                id[i0 + u] = bucket.ids[at] + t[u] * kTileRows;
            }
        }
    sh.template sort<true>(share, bucket.low, bucket.high, key, order);
    uint32_t *const ids = reinterpret_cast<uint32_t *>(sh.words);
#pragma unroll
    for (uint32_t i = 0; i < SLOTS; ++i)
        if (share.has(i)) {
            sorted_keys[bucket.out + share.number(i)] = key[i];
            ids[share.number(i)] = id[i];
        }
    __syncthreads();
#pragma unroll
    for (uint32_t i = 0; i < SLOTS; ++i)
        if (share.has(i)) sorted_ids[bucket.out + share.number(i)] = ids[order[i]];
}

// One workgroup per bucket.
__global__ __launch_bounds__(kBucketThreads, 3) void sort_buckets(const SortedTiles in, uint32_t items, uint32_t items_of_xcd,
                                                                  BucketList *__restrict__ medium,
                                                                  uint64_t *__restrict__ sorted_keys,
                                                                  uint32_t *__restrict__ sorted_ids) {
    __shared__ Sorter<kBucketThreads, kSlots> sh;
    __shared__ Runs runs;
    // neighbouring buckets run at the same time on one XCD: their runs share lines
    const uint32_t item = (blockIdx.x & 7) * items_of_xcd + (blockIdx.x >> 3);
    if (item >= items) return;
    const Bucket bucket = find_bucket(runs, sh.counter, in, item);
    sort_bucket(sh, runs, bucket, item, medium, sorted_keys, sorted_ids);
}

// Those of up to twice as many pairs (keys that are met in one splitter only, with their neighbours), and those of one key.
__global__ __launch_bounds__(kLargeThreads) void sort_medium_buckets(const SortedTiles in, const BucketList *__restrict__ medium,
                                                                     BucketList *__restrict__ large,
                                                                     uint64_t *__restrict__ sorted_keys,
                                                                     uint32_t *__restrict__ sorted_ids) {
    __shared__ Sorter<kLargeThreads, kLargeSlots> sh;
    __shared__ Runs runs;
    const uint32_t listed = medium->count;
    for (uint32_t entry = blockIdx.x; entry < listed; entry += gridDim.x) {
        __syncthreads();  // the bucket before has left the LDS
        const Bucket bucket = find_bucket(runs, sh.counter, in, medium->entry[entry].bucket);
        if (bucket.low < bucket.high) {
            sort_bucket(sh, runs, bucket, medium->entry[entry].bucket, large, sorted_keys, sorted_ids);
            continue;
        }
        const uint32_t first = medium->entry[entry].part * kLargeCap;
#pragma unroll 4
        for (uint32_t i = 0; i < kLargeSlots; ++i) {
            const uint32_t p = first + i * kLargeThreads + threadIdx.x;
            if (p < bucket.count) {
                const uint32_t t = runs.run_of(p);
                sorted_keys[bucket.out + p] = bucket.low;
                sorted_ids[bucket.out + p] = bucket.ids[p + runs.ahead[t]] + t * kTileRows;
            }
        }
    }
}

// The rest, which the sample met badly.  Range after range of the keys, each read
// off all runs.
__global__ __launch_bounds__(kLargeThreads) void sort_large_buckets(const SortedTiles in, const BucketList *__restrict__ large,
                                                                     uint64_t *__restrict__ sorted_keys,
                                                                     uint32_t *__restrict__ sorted_ids) {
    __shared__ Sorter<kLargeThreads, kLargeSlots> sh;
    __shared__ Runs runs;
    uint32_t *const words32 = reinterpret_cast<uint32_t *>(sh.words);
    const uint32_t listed = large->count;
    for (uint32_t entry = blockIdx.x; entry < listed; entry += gridDim.x) {
        __syncthreads();  // the runs of the bucket before have been read
        const Bucket bucket = find_bucket(runs, sh.counter, in, large->entry[entry].bucket);
        const uint32_t count = bucket.count;
        // where pair p of the bucket is
        auto at = [&](uint32_t p, uint32_t &tile) __attribute__((always_inline)) {
            tile = runs.run_of(p);
            return p + runs.ahead[tile];
        };
        // the pairs with keys in [low, high], in order: put(number among them, key, id)
        auto sweep = [&](uint64_t low, uint64_t high, auto put) __attribute__((always_inline)) {
            uint32_t base = 0;
            for (uint32_t p0 = 0; p0 < count; p0 += kLargeThreads) {
                const uint32_t p = p0 + threadIdx.x;
                uint32_t tile = 0, where = 0;
                uint64_t k = 0;
                bool taken = false;
                if (p < count) {
                    where = at(p, tile);
                    k = bucket.keys[where];
                    taken = k >= low && k <= high;
                }
                const uint64_t those = __ballot(taken);
                __syncthreads();  // the totals of the step before have been read
                if (lane_id() == 0) sh.dirty[wave_id()] = (uint32_t)__popcll(those);
                __syncthreads();
                uint32_t mine = base + (uint32_t)__popcll(those & ((1ull << lane_id()) - 1));
                for (uint32_t w = 0; w < kLargeThreads / 64; ++w) {
                    if (w < wave_id()) mine += sh.dirty[w];
                    base += sh.dirty[w];
                }
                if (taken) put(mine, k, bucket.ids[where] + tile * kTileRows);
            }
            __syncthreads();
        };
        uint64_t low = ~0ull, last = 0;
        for (uint32_t p = threadIdx.x; p < count; p += kLargeThreads) {
            uint32_t tile;
            const uint64_t k = bucket.keys[at(p, tile)];
            low = k < low ? k : low;
            last = k > last ? k : last;
        }
        sh.range(low, last);
        if (low == last) {  // one key: its pairs are in order
            for (uint32_t p = threadIdx.x; p < count; p += kLargeThreads) {
                uint32_t tile;
                const uint32_t where = at(p, tile);
                sorted_keys[bucket.out + p] = low;
                sorted_ids[bucket.out + p] = bucket.ids[where] + tile * kTileRows;
            }
            continue;
        }
        for (uint32_t done = 0; done < count;) {  // pairs of keys below `low` are out; every turn puts out at least one key's
            uint32_t take = 0;
            uint64_t high = last;
            bool one_key = false;
            while (!take) {  // [low, high] holds pairs; a turn without a result leaves 8 bits fewer between its ends
                const int bits = high > low ? 64 - __clzll((long long)(high - low)) : 0, shift = bits > 8 ? bits - 8 : 0;
                uint32_t *const cells = sh.dirty;
                if (threadIdx.x < 256) cells[threadIdx.x] = 0;
                __syncthreads();
                for (uint32_t p = threadIdx.x; p < count; p += kLargeThreads) {
                    uint32_t tile;
                    const uint64_t k = bucket.keys[at(p, tile)];
                    if (k >= low && k <= high) atomicAdd(&cells[(uint32_t)((k - low) >> shift)], 1u);
                }
                __syncthreads();
                const uint32_t upto = sh.counter.scan(threadIdx.x < 256 ? cells[threadIdx.x] : 0);
                if (threadIdx.x < 256) cells[threadIdx.x] = upto;
                __syncthreads();
                uint32_t fit = 0;  // leading cells that LDS holds together
                for (uint32_t half = 128; half > 0; half >>= 1)
                    if (cells[fit + half - 1] <= kLargeCap) fit += half;
                if (fit == 255 && cells[255] <= kLargeCap) fit = 256;
                fit = uniform(fit);
                take = fit ? uniform(cells[fit - 1]) : 0;
                const uint32_t next = fit < 256 ? uniform(cells[fit]) : 0;
                __syncthreads();
                if (take) {
                    if (fit < 256) high = low + ((uint64_t)fit << shift) - 1;
                    continue;
                }
                low += (uint64_t)fit << shift;  // cell `fit` alone is too much: into it
                if (shift == 0) {
                    high = low;
                    take = next;
                    one_key = true;
                    continue;
                }
                const uint64_t cell = (1ull << shift) - 1;
                if (high - low > cell) high = low + cell;
            }
            const uint64_t out = bucket.out + done;
            if (one_key) {
                sweep(low, high, [&](uint32_t number, uint64_t k, uint32_t i) {
                    sorted_keys[out + number] = k;
                    sorted_ids[out + number] = i;
                });
            } else {
                const Share share(take, kLargeThreads);
                uint64_t key[kLargeSlots];
                uint32_t order[kLargeSlots];
                sweep(low, high, [&](uint32_t number, uint64_t k, uint32_t) { sh.words[number] = k; });
#pragma unroll
                for (uint32_t i = 0; i < kLargeSlots; ++i)
                    if (share.has(i)) key[i] = sh.words[share.number(i)];
                __syncthreads();
                sh.sort<true>(share, low, high, key, order);
                sweep(low, high, [&](uint32_t number, uint64_t, uint32_t i) { words32[number] = i; });
#pragma unroll
                for (uint32_t i = 0; i < kLargeSlots; ++i)
                    if (share.has(i)) {
                        sorted_keys[out + share.number(i)] = key[i];
                        sorted_ids[out + share.number(i)] = words32[order[i]];
                    }
                __syncthreads();
            }
            done += take;
            low = high + 1;
        }
    }
}

size_t align16(size_t bytes) { return (bytes + 15) & ~size_t(15); }

}  // namespace

bool bucket_sort_takes(uint64_t N, uint32_t L) {
    return N <= (uint64_t)kMaxBuckets * kBucketMean && (uint64_t)L * kMaxBuckets < (1u << 31);
}

size_t bucket_sort_scratch(uint64_t N, uint32_t L) {
    const Plan p = plan_of(N, L);
    return align16((size_t)L * p.stride * 8) + align16((size_t)L * p.stride * 2) + align16((size_t)L * p.buckets * 8) +
           align16((size_t)L * p.tiles * (p.buckets + 1) * 2) + 2 * align16(list_bytes(N, L, p.buckets));
}

void launch_bucket_sort(const uint64_t *d_keys, uint64_t N, uint32_t L, void *scratch, uint64_t *d_out_keys,
                        uint32_t *d_out_ids, hipStream_t s) {
    const Plan p = plan_of(N, L);
    char *at = static_cast<char *>(scratch);
    auto piece = [&](size_t bytes) { return std::exchange(at, at + align16(bytes)); };
    SortedTiles t;
    t.keys = reinterpret_cast<uint64_t *>(piece((size_t)L * p.stride * 8));
    t.ids = reinterpret_cast<uint16_t *>(piece((size_t)L * p.stride * 2));
    t.cuts = reinterpret_cast<uint64_t *>(piece((size_t)L * p.buckets * 8));
    t.offsets = reinterpret_cast<uint16_t *>(piece((size_t)L * p.tiles * (p.buckets + 1) * 2));
    BucketList *const medium = reinterpret_cast<BucketList *>(piece(list_bytes(N, L, p.buckets)));
    BucketList *const large = reinterpret_cast<BucketList *>(piece(list_bytes(N, L, p.buckets)));
    t.N = N, t.stride = p.stride, t.tiles = p.tiles, t.buckets = p.buckets;
    uint32_t bucket_bits = 0;
    while ((1u << bucket_bits) < p.buckets) ++bucket_bits;
    if (p.buckets > 1) hipLaunchKernelGGL(sort_splitters, dim3(L), dim3(kSampleThreads), 0, s, d_keys, N, L, p.buckets, t.cuts);
    const uint32_t groups = (L + kTileColumns - 1) / kTileColumns;
    const bool pairs = L % 2 == 0 && (reinterpret_cast<uintptr_t>(d_keys) & 15) == 0;
    hipLaunchKernelGGL(pairs ? sort_tiles<true> : sort_tiles<false>, dim3((p.tiles + 7) / 8 * 8 * groups), dim3(kTileThreads), 0,
                       s, d_keys, L, groups, bucket_bits, t, medium, large);
    const uint32_t items = L * p.buckets, items_of_xcd = (items + 7) / 8;
    hipLaunchKernelGGL(sort_buckets, dim3(items_of_xcd * 8), dim3(kBucketThreads), 0, s, t, items, items_of_xcd, medium, d_out_keys,
                       d_out_ids);
    if (N <= kBucketCap) return;
    hipLaunchKernelGGL(sort_medium_buckets, dim3(items < 256 ? items : 256), dim3(kLargeThreads), 0, s, t, medium, large,
                       d_out_keys, d_out_ids);
    if (N <= kLargeCap) return;
    hipLaunchKernelGGL(sort_large_buckets, dim3(items < 256 ? items : 256), dim3(kLargeThreads), 0, s, t, large, d_out_keys,
                       d_out_ids);
}

}  // namespace lsh
