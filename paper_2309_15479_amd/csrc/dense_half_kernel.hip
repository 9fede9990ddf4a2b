// Dense E2LSH projections (Sec. 2.2, Eq. 1) on the fp16 matrix cores of gfx950 with fp32 accuracy,
// for sums of 128 terms and more: P = V A^T from two-way fp16 splits of both operands scaled by
// powers of two, and three products.
//
// Arithmetic.  x 2^e = x1 + x2 + r with x1 = fp16(x 2^e), x2 = fp16(x 2^e - x1), round to nearest:
// two 11-bit significands and the sign of the second hold 23 bits, |r| <= 2^-23 of x (2^-25 absolute
// where x2 is subnormal).  The products a1 v1 + a1 v2 + a2 v1 are exact in fp32, a2 v2 (below 2^-22 of
// the term) is left out.  Against 64 bits the split is off by 7e-8 (2-norm) at any length, and the
// accumulation rounds half as often as over the six bf16 products of dense_split_wide_kernel.hip,
// where every product is added to the same accumulators.  Both together, modelled with one rounding a
// product of 16 terms, fp16 / bf16: 8.5e-8 / 6.3e-8 at 30 terms, 1.07e-7 / 1.18e-7 at 128, 1.9e-7 /
// 2.5e-7 at 512, 2.5e-7 / 3.5e-7 at 960.  Measured, fp16 / bf16: normal coordinates 1.53e-7 / 1.74e-7 at 132 terms, 1.93 /
// 2.40 at 256, 3.5 / 4.7 at 960; whole numbers below 256, of which two of the bf16 terms are zero, 1.14 / 1.13 at 132, 1.211 /
// 1.208 at 160, 1.263 / 1.270 at 176, 2.8 / 3.0 at 960.  kHalfMinTerms is where the fp16 product is the more accurate
// one, but for those whole numbers, where they are even up to 170 terms (1 % apart at most).  Below 1e-36, where bf16 terms
// are lost, it is the only one that keeps to 1e-5 of sum |a_i v_i|.
//
// Scales.  e is a function's (on the host, from its largest coefficient: [2^14, 2^15) after scaling)
// or a vector's.  A vector's comes from 80 of its coordinates, the three stages that start the
// contraction and two further on.  If eight of them are at least an eighth of the largest, the largest goes to
// [2^5, 2^6), and any other coordinate may be a thousand times larger before it leaves fp16; if eight are at least a 128th,
// to [2^9, 2^10), with room for 64 times more.  Eight coordinates are 4 and more then, and what any
// coordinate loses below 2^-24, at most 2^-25, is nothing beside their products.  Such a vector is regular, unless a
// coordinate leaves fp16.
//
// Odd vectors.  In any other vector (sparse, or of coordinates of very different sizes) a few coordinates may
// carry the sum, and where a function has small coefficients at those, what the others lost would be more than the 1e-5
// of sum |a_i v_i| that a projection may be off.  Their results come from the exact bf16 splits instead, the
// same numbers as dense_split_wide_kernel.hip gives: a workgroup puts the odd vectors of kSegment tiles by
// and contracts them together (dense_wide_tile.h).  Tiles of nearly only odd vectors are not contracted in
// fp16 at all; their few regular ones are put by, too.  A coordinate that leaves fp16 is met in the contraction, which
// then was for nothing; a workgroup to which that has happened with half a tile looks at the same place of its later
// tiles first.  Which way a vector goes, and its scale, depend on the vector alone.
// N = 2e5, n = 960, k = 1024, us, this kernel / the six bf16 products for all vectors: normal coordinates 1240 / 1980,
// 30 % of them not zero 1150 / 1890, 10 % (half of the vectors odd) 1930 / 1790, 2 % 1790 / 1710, one per vector 1700 / 1630,
// ratios of two normal ones 1530 / 2000, columns of sizes from 1 to 10^6 1240 / 1990, one column 10^4 times as large
// 2140 / 1960 if it is looked at, 2630 / 1980 if not (seven vectors in ten odd, none known before the contraction).
//
//   V [N][n] fp32 row-major; A split on the host into two fp16 planes in the order of use:
//   [function tile of 256][stage of 16 coordinates][plane][row][coordinate] (zero rows up to a multiple
//   of 256, zero columns up to a multiple of 16), the functions' exponents behind them.
//
// Workgroup, tile, placement and the three LDS stages are those of dense_split_wide_kernel.hip: 4 waves,
// 256 functions x 256 vectors, 4 x 4 blocks of 32 x 32 a wave, everything that is not an MFMA dealt out
// behind the MFMAs.  A stage is 48 MFMAs a wave here (96 there), which leaves half as many places for
// 8 global loads, 12 LDS writes, 16 LDS reads and the split of 16 vector elements; it takes 1.25 us of
// which the matrix pipe is busy 0.8.  The rest is the issue of those instructions by a wave that is alone on
// its SIMD, and 14 us a tile of first loads, scales and results.
// Measured against the six bf16 products (same job): 9230 -> 5570 us at N = 1e6, n = 960, k = 1024;
// 14150 -> 8030 at 2e5, 4096, 2048; 429 -> 217 at 1e4, 4096, 512; 114 -> 64 at 1000, 960, 1024; 77 -> 58 at
// 1e5, 132, 256; 467 -> 321 at 3e5, 300, 250.  What gave how much at 1e6 x 960: the arithmetic 5930; LDS accesses
// kept away from the barrier and smaller pieces of work behind the MFMAs 5800; results through LDS into whole
// lines 5570.  Two and three register sets for the vector and coefficient loads, and the next tile's first loads
// ahead of the results, cost more in registers spilled around the loop than they hide (6000 to 6500).
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstring>
#include <type_traits>
#include <utility>
#include <vector>

#include "dense_wide_tile.h"
#include "lsh_internal.h"

namespace lsh {
namespace {

typedef _Float16 halfx8 __attribute__((ext_vector_type(8)));
typedef _Float16 halfx4 __attribute__((ext_vector_type(4)));
typedef _Float16 halfx2 __attribute__((ext_vector_type(2)));
typedef float floatx2 __attribute__((ext_vector_type(2)));
typedef int intx4 __attribute__((ext_vector_type(4)));

// the tile of dense_wide_tile.h
using wide::floatx16;
using wide::floatx4;
using wide::uintx4;
using wide::TF;
using wide::TVW;
using wide::NB;
using wide::KB;
using wide::ROWB;
using wide::A_PLANE;
using wide::V_PLANE;
constexpr int STAGE = 2 * (A_PLANE + V_PLANE);  // 32768 bytes
constexpr int kThreadsH = 256;
constexpr int kStagePlanes = 2 * TF * KB;  // fp16 elements of one function tile's two planes in one stage
constexpr int kVectorScales = 3 * STAGE;   // LDS offset of the tile's 256 vector exponents
constexpr uint32_t kSegment = 16;          // tiles after which the odd vectors put by are contracted
constexpr int kOddList = wide::kLdsBytes;  // LDS offset of their numbers in the segment, 16 bits each
constexpr int kOddCount = kOddList + (int)kSegment * TVW * 2;  // of the words below
constexpr int kLdsBytesH = kOddCount + 24;
constexpr uint32_t kFewRegular = 48;       // a tile of so few regular vectors is not contracted (94 us): they are put by, too, for few_block (1.6 us each)
constexpr uint32_t kFewOdd = 64;           // up to so many by blocks of 32 x 32 (80 us at n = 960), more by tiles (150 us)
constexpr int kResultRow = 144;            // bytes of a vector's 32 results in LDS on their way out: conflict-free both ways
constexpr uint32_t kHalfMinTerms = 128;
constexpr float kLargestHalf = 65504.f;
constexpr int kFunctionTop = 14;                  // exponent of a function's largest coefficient after scaling
constexpr int kEvenTop = 5, kUnevenTop = 9;       // of a vector's largest looked-at coordinate, see vector_scale
constexpr uint32_t kRegularCount = 8;             // looked-at coordinates of 2^2 and more after scaling that make a vector regular
constexpr float kRegularLeast = 1.17549435e-38f;  // 2^-126, which the largest scale, 2^126, takes to 1
constexpr int kOdd = 4096;                        // added to the exponent of an odd vector

struct HalfArgs {
    const float *data;       // [N][n]
    const uint16_t *planes;  // [kpad / 256][npad / 16][2][256][16] fp16 bit patterns
    const int *fexp;         // [kpad] exponents the functions were scaled by
    const float *off;        // [>= kpad]
    uint64_t N;
    uint32_t n, npad, k, kpad;
    float w, inv_w;
    void *out;               // [N][k]
    const uint16_t *exact_planes;  // the bf16 planes, as in wide::Args

    __device__ wide::Args exact() const { return {data, exact_planes, off, N, n, npad, k, kpad, w, inv_w, out}; }
};

// exponent e that takes a value's leading bit to 2^top; 2^e is a normal float
__device__ __forceinline__ int scale_exponent(float largest, int top) {
    const int biased = (int)((__float_as_uint(largest) >> 23) & 255u);
    const int e = top + 127 - biased;
    return largest == 0.f ? 0 : e > 126 ? 126 : e;  // at least top - 128
}

__device__ __forceinline__ float power_of_two(int e) { return __uint_as_float((uint32_t)(e + 127) << 23); }

__device__ __forceinline__ float largest_of(floatx4 v, float so_far) {
    return fmaxf(fmaxf(fmaxf(fabsf(v[0]), fabsf(v[1])), so_far), fmaxf(fabsf(v[2]), fabsf(v[3])));
}

// how many are at least an eighth of the largest of all, and in the upper half how many at least a 128th
__device__ __forceinline__ uint32_t count_large(floatx4 v, float largest) {
    uint32_t count = 0;
#pragma unroll
    for (int e = 0; e < 4; ++e)
        count += (fabsf(v[e]) >= largest * 0x1p-3f ? 1u : 0u) + (fabsf(v[e]) >= largest * 0x1p-7f ? 0x10000u : 0u);
    return count;
}

// The exponent for a vector from its largest looked-at coordinate and their count; kOdd is added if it is odd.
__device__ __forceinline__ int vector_scale(float largest, uint32_t count) {
    const bool even = (count & 0xFFFFu) >= kRegularCount, uneven = (count >> 16) >= kRegularCount;
    return scale_exponent(largest, even ? kEvenTop : kUnevenTop) + (uneven && largest >= kRegularLeast ? 0 : kOdd);
}

// vectors put by: a list of their numbers in the tiles tile, tile + step, ...
struct Listed {
    const uint16_t *list;
    uint64_t tile, step;
    uint32_t last, first = 0;
    __device__ uint64_t wanted(uint32_t i) const {
        const uint32_t in = list[first + i];
        return (tile + in / TVW * step) * TVW + in % TVW;
    }
    __device__ uint64_t any(uint32_t i) const { return wanted(first + i < last ? i : last - first); }
};

// two elements, scaled and split: hi + lo = x 2^e to 23 bits
__device__ __forceinline__ void split2(float x0, float x1, float scale, halfx2 &hi, halfx2 &lo) {
    const floatx2 y = {x0 * scale, x1 * scale};
    hi = __builtin_convertvector(y, halfx2);
    const floatx2 r = {__builtin_fmaf(x0, scale, -(float)hi[0]), __builtin_fmaf(x1, scale, -(float)hi[1])};
    lo = __builtin_convertvector(r, halfx2);
}

// PROJ: raw projections instead of bucket ids.  POW2: w is a power of two (fma(p, 1/w, b/w) is
// then the same float as (p + b) / w).  VEC: k is a multiple of 4 (16-byte stores).
//
// The same product for few vectors, where tiles of 256 x 256 leave most of the chip idle and each of them
// still walks all stages.  A wave takes 32 functions x 32 vectors with its operands straight from memory, the
// planes in the order they are stored in and the vectors split in registers: no LDS, no barrier, the
// loads of kFewSets stages on their way.  Scales, products and their order are those of the tile kernel below,
// and so are the results, bit for bit.  Bound by the chain of a stage (three dependent MFMAs, the split) and by 4 KB
// of loads for every 3 MFMAs, which is why it loses where there are tiles enough.  Tiles / this kernel, by the
// number of its waves: 8 x 960 x 1024 (32) 60.5 / 14.2 us; 100 x 16000 x 250 (32) 805 / 275; 1000 x 4096 x 512 (512)
// 211 / 74; 1000 x 960 x 1024 (1024) 64.5 / 21.7; 1e4 x 300 x 250 (2504) 39.0 / 23.5; 4000 x 960 x 1024 (4000) 66 / 79; 8000 x
// 4096 x 512 (4000) 214 / 291; 3e4 x 132 x 256 (7504) 28.6 / 33.7.  The line is three waves for every SIMD.
constexpr int kFewSets = 4;
constexpr uint64_t kFewWaves = 3072;

// Functions j0 ... j0 + 31 (j0 a multiple of 32 below k) against 32 vectors: lanes l and l + 32 take vector `row` and
// store its results if `store`.
template <bool PROJ, bool POW2, bool VEC>
__device__ __forceinline__ void few_block(const HalfArgs &a, uint32_t thread, uint32_t j0, uint64_t row, bool store) {
    const uint32_t lane = thread & 63, lr = lane & 31, lh = lane >> 5;
    const uint32_t stages = a.npad / KB;
    const uint16_t *arow = a.planes + (size_t)(j0 / TF) * stages * kStagePlanes + (j0 % TF + lr) * KB + lh * 8;
    const float *vrow = a.data + row * a.n + lh * 8;
    // as in the tile kernel: coordinates beyond n read the vector's first ones, stages beyond the last the last one
    auto load_v = [&](uint32_t s, floatx4 (&v)[2]) __attribute__((always_inline)) {
#pragma unroll
        for (int h = 0; h < 2; ++h)
            v[h] = *reinterpret_cast<const floatx4 *>(vrow + h * 4 + (s * KB + lh * 8 + h * 4 < a.n ? s * KB : 0u));
    };
    auto load_a = [&](uint32_t s, halfx8 (&c)[2]) __attribute__((always_inline)) {
        const uint32_t ka = s < stages ? s : stages - 1;
#pragma unroll
        for (int p = 0; p < 2; ++p) c[p] = *reinterpret_cast<const halfx8 *>(arow + (size_t)ka * kStagePlanes + p * (TF * KB));
    };
    floatx4 v[kFewSets][2];
    halfx8 c[kFewSets][2];
    float largest = 0.f;
    int vexp;
    bool odd;
    {
        floatx4 looked[5][2];
        const uint32_t at[5] = {0, 1, 2, stages / 3, stages * 2 / 3};
#pragma unroll
        for (int t = 0; t < 5; ++t) load_v(at[t], looked[t]);
#pragma unroll
        for (int t = 0; t < 5; ++t) largest = largest_of(looked[t][1], largest_of(looked[t][0], largest));
        largest = fmaxf(largest, __shfl_xor(largest, 32));  // the two lanes of a vector
        uint32_t count = 0;
#pragma unroll
        for (int t = 0; t < 5; ++t) count += count_large(looked[t][0], largest) + count_large(looked[t][1], largest);
        count += __shfl_xor(count, 32);
        vexp = vector_scale(largest, count);
        odd = vexp >= kOdd / 2;
        if (odd) vexp = 0;
    }
    floatx16 acc;
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[e] = 0.f;
    if (__any(!odd)) {
        const float scale = power_of_two(vexp);
#pragma unroll
        for (int d = 0; d < kFewSets; ++d) {
            load_v(d, v[d]);
            load_a(d, c[d]);
        }
        for (uint32_t s0 = 0; s0 < stages; s0 += kFewSets) {
#pragma unroll
            for (int d = 0; d < kFewSets; ++d) {
                if (s0 + d < stages) {
                    halfx8 v1, v2;
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        halfx2 hi, lo;
                        split2(v[d][e / 2][e % 2 * 2], v[d][e / 2][e % 2 * 2 + 1], scale, hi, lo);
                        v1[2 * e] = hi[0], v1[2 * e + 1] = hi[1];
                        v2[2 * e] = lo[0], v2[2 * e + 1] = lo[1];
                    }
                    largest = largest_of(v[d][1], largest_of(v[d][0], largest));
                    acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(c[d][0], v2, acc, 0, 0, 0);
                    acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(c[d][0], v1, acc, 0, 0, 0);
                    acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(c[d][1], v1, acc, 0, 0, 0);
                }
                load_v(s0 + d + kFewSets, v[d]);
                load_a(s0 + d + kFewSets, c[d]);
            }
        }
        largest = fmaxf(largest, __shfl_xor(largest, 32));
        odd |= largest * scale > kLargestHalf;
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const uint32_t j = j0 + 8 * q + 4 * lh;  // < kpad
        const intx4 fe = *reinterpret_cast<const intx4 *>(a.fexp + j);
        floatx4 b4 = {0.f, 0.f, 0.f, 0.f};
        if constexpr (!PROJ) {
            b4 = *reinterpret_cast<const floatx4 *>(a.off + j);
            if constexpr (POW2) b4 *= a.inv_w;
        }
        uintx4 r;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float p = __builtin_ldexpf(acc[4 * q + e], -(fe[e] + vexp));
            if constexpr (PROJ) {
                r[e] = __float_as_uint(p);
            } else {
                const float h = POW2 ? fmaf(p, a.inv_w, b4[e]) : (p + b4[e]) / a.w;
                r[e] = (uint32_t)(int)floorf(h);
            }
        }
        if (store) {
            uint32_t *dst = reinterpret_cast<uint32_t *>(a.out) + row * a.k + j;
            if constexpr (VEC) {
                if (j < a.k) *reinterpret_cast<uintx4 *>(dst) = r;
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (j + e < a.k) dst[e] = r[e];
            }
        }
    }
    odd = odd && store;
    if (__any(odd)) wide::block<PROJ, POW2, VEC>(a.exact(), thread, j0, row, odd);  // the same lane stores over its results
}

template <bool PROJ, bool POW2, bool VEC>
__global__ __launch_bounds__(256) void dense_half_few_kernel(const HalfArgs a) {
    const uint32_t j0 = (blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6)) * 32;  // the wave's functions
    const uint64_t vec = (uint64_t)blockIdx.y * 32 + (threadIdx.x & 31);
    if (j0 < a.k) few_block<PROJ, POW2, VEC>(a, threadIdx.x, j0, vec < a.N ? vec : a.N - 1, vec < a.N);
}

template <bool PROJ, bool POW2, bool VEC>
__global__ __launch_bounds__(kThreadsH) void dense_half_kernel(const HalfArgs a) {
    extern __shared__ __align__(16) char lds_h[];  // 3 stages x ([2][256][32] coefficients, [2][256][32] vectors), exponents; odd vectors
    int *const vector_exp = reinterpret_cast<int *>(lds_h + kVectorScales);
    uint16_t *const odd_list = reinterpret_cast<uint16_t *>(lds_h + kOddList);
    volatile uint32_t *const odd_count = reinterpret_cast<uint32_t *>(lds_h + kOddCount);  // from the front of the list
    volatile uint32_t *const few_count = odd_count + 1;    // regular vectors of tiles with few of them, from its back
    volatile uint32_t *const regular_count = odd_count + 2;  // in a tile; two, taken in turn
    volatile uint32_t *const left_count = odd_count + 4;   // vectors of a tile of which a coordinate left fp16
    volatile uint32_t *const left_stage = odd_count + 5;   // where one did, of the last tile with many

    // which (function tile, vector tile) pairs this workgroup takes
    const uint32_t F = a.kpad / TF;
    const uint64_t Vt = (a.N + TVW - 1) / TVW;
    const uint32_t x = blockIdx.x & 7, i = blockIdx.x >> 3, per_xcd = gridDim.x >> 3;
    uint32_t ft_first, ft_step, reps, rep;
    if (F >= 8) {
        ft_first = x; ft_step = 8; reps = 1; rep = 0;
    } else {
        ft_first = x % F; ft_step = F;  // one function tile per XCD
        reps = (8 - ft_first + F - 1) / F;  // XCDs that share it
        rep = x / F;
    }

    const uint32_t stages = a.npad / KB;

    // as in dense_split_wide_kernel: the function tiles of a vector tile side by side on one XCD
    const bool by_vector = per_xcd % F == 0 && F <= per_xcd;
    uint64_t vt_first = (uint64_t)i * reps + rep, vt_step = (uint64_t)per_xcd * reps;
    if (by_vector) {
        ft_first = i % F;
        ft_step = F;  // one function tile per workgroup
        const uint32_t groups = per_xcd / F;
        vt_first = x + 8ull * (i / F);
        vt_step = 8ull * groups;
    }
    const bool whole_lines = a.k % 32 == 0;  // non-temporal stores then; of partial lines they are slower (341 against 302 us at k = 252)
    if (threadIdx.x < 6) odd_count[threadIdx.x] = 0;
    lds_barrier();
    uint32_t turn = 0;  // of the two counts
    for (uint32_t ft = ft_first; ft < F; ft += ft_step) {
        uint32_t tiles = 0;  // since the odd vectors were last contracted
        for (uint64_t vt = vt_first; vt < Vt; vt += vt_step) {
            uint32_t thread = threadIdx.x;
            asm volatile("" : "+v"(thread));  // or every address made from it would be held through all tiles, in memory
            const uint32_t lane = thread & 63, wave = __builtin_amdgcn_readfirstlane(thread >> 6);
            const uint32_t lr = lane & 31, lh = lane >> 5;
            const uint32_t fw = wave & 1, vw = wave >> 1;  // the wave's half of the functions, half of the vectors
            // loading roles: 16 bytes of the vector tile and of each coefficient plane per stage
            const uint32_t vr = thread >> 2, vq = thread & 3;  // vector rows vr + 64 h (h < 4), 4-coordinate piece
            const uint32_t ar = thread >> 1, ah = thread & 1;  // coefficient rows ar and ar + 128, 8-coordinate half

            // operand read and write offsets inside a stage (half h of row r sits at 16 * (h ^ bit 3 of r))
            const uint32_t rd_a = (fw * 32 * NB + lr) * ROWB + ((lh ^ ((lr >> 3) & 1)) << 4);                // + rb * 32 rows + plane
            const uint32_t rd_v = 2 * A_PLANE + (vw * 32 * NB + lr) * ROWB + ((lh ^ ((lr >> 3) & 1)) << 4);  // + cb * 32 rows + plane
            const uint32_t wr_a = ar * ROWB + ((ah ^ ((ar >> 3) & 1)) << 4);
            const uint32_t wr_v = 2 * A_PLANE + vr * ROWB + (((vq >> 1) ^ ((vr >> 3) & 1)) << 4) + ((vq & 1) << 3);
            // thread t: 16 bytes at 16 t of rows 0-127 of a plane, and of rows 128-255
            const uint16_t *arow = a.planes + (size_t)ft * stages * kStagePlanes + thread * 8;
            const float *vrow[4];
#pragma unroll
            for (int h = 0; h < 4; ++h) {
                uint64_t row = vt * TVW + vr + h * 64;
                row = row < a.N ? row : a.N - 1;  // rows beyond the data repeat the last vector (never stored)
                vrow[h] = a.data + row * a.n + vq * 4;
            }
            // Every load is issued unconditionally (the compiler can then count the loads in flight
            // exactly and wait for the oldest only).  Coordinates beyond n read the vector's first ones
            // instead: the coefficients are zero there.  Stages beyond the last are read and written to
            // LDS like others and never contracted.
            auto load_v = [&](uint32_t s, int h) __attribute__((always_inline)) {
                const uint32_t k0 = s * KB;
                return *reinterpret_cast<const floatx4 *>(vrow[h] + (k0 + vq * 4 < a.n ? k0 : 0u));
            };
            auto load_a = [&](uint32_t s, int h, int p) __attribute__((always_inline)) {
                const uint32_t ka = s < stages ? s : stages - 1;
                return *reinterpret_cast<const uintx4 *>(arow + (size_t)ka * kStagePlanes + p * (TF * KB) + h * 128 * KB);
            };
            floatx16 acc[NB][NB];
            float scale[4], largest[4];
            bool contracted;
            {
                // stages 0 to 2 and the coordinates the scales are taken from: all in flight at once
                floatx4 gv[3][4];
                uintx4 ga[3][2][2];
#pragma unroll
                for (int t = 0; t < 3; ++t) {
#pragma unroll
                    for (int h = 0; h < 4; ++h) gv[t][h] = load_v(t, h);
#pragma unroll
                    for (int h = 0; h < 2; ++h)
#pragma unroll
                        for (int p = 0; p < 2; ++p) ga[t][h][p] = load_a(t, h, p);
                }
                floatx4 far_v[2][4];
#pragma unroll
                for (int t = 0; t < 2; ++t)
#pragma unroll
                    for (int h = 0; h < 4; ++h) far_v[t][h] = load_v(stages * (t + 1) / 3, h);
                float there[4] = {0.f, 0.f, 0.f, 0.f};  // where many of an earlier tile's vectors left fp16: they turn out odd at once
                const uint32_t before = __builtin_amdgcn_readfirstlane(*left_stage);
                if (before) {
#pragma unroll
                    for (int h = 0; h < 4; ++h) there[h] = largest_of(load_v(before, h), 0.f);
#pragma unroll
                    for (int h = 0; h < 4; ++h) {
                        there[h] = fmaxf(there[h], __shfl_xor(there[h], 1));
                        there[h] = fmaxf(there[h], __shfl_xor(there[h], 2));
                    }
                }
                // The largest of two halves of a thread's coordinates: if the least of a vector's eight is an eighth of
                // their largest, as it nearly always is, nothing needs counting (2 % of the time at n = 300).
                uint32_t count[4];
                bool sure = true;
#pragma unroll
                for (int h = 0; h < 4; ++h) {
                    float half[2] = {0.f, 0.f};
#pragma unroll
                    for (int p = 0; p < 2; ++p) {
#pragma unroll
                        for (int t = 0; t < 3; ++t) half[p] = fmaxf(fmaxf(fabsf(gv[t][h][2 * p]), fabsf(gv[t][h][2 * p + 1])), half[p]);
#pragma unroll
                        for (int t = 0; t < 2; ++t) half[p] = fmaxf(fmaxf(fabsf(far_v[t][h][2 * p]), fabsf(far_v[t][h][2 * p + 1])), half[p]);
                    }
                    float top = fmaxf(half[0], half[1]), least = fminf(half[0], half[1]);
                    top = fmaxf(top, __shfl_xor(top, 1));  // the four threads of a vector are neighbours
                    least = fminf(least, __shfl_xor(least, 1));
                    top = fmaxf(top, __shfl_xor(top, 2));
                    least = fminf(least, __shfl_xor(least, 2));
                    largest[h] = top;
                    count[h] = kRegularCount | kRegularCount << 16;
                    sure = sure && least >= top * 0x1p-3f;
                }
                if (!__all(sure)) {
#pragma unroll
                    for (int h = 0; h < 4; ++h) {
                        count[h] = 0;
#pragma unroll
                        for (int t = 0; t < 3; ++t) count[h] += count_large(gv[t][h], largest[h]);
#pragma unroll
                        for (int t = 0; t < 2; ++t) count[h] += count_large(far_v[t][h], largest[h]);
                        count[h] += __shfl_xor(count[h], 1);
                        count[h] += __shfl_xor(count[h], 2);
                    }
                }
                uint32_t regular = 0;
#pragma unroll
                for (int h = 0; h < 4; ++h) {
                    int e = vector_scale(largest[h], count[h]);
                    if (e < kOdd / 2 && there[h] * power_of_two(e) > kLargestHalf) e += kOdd;
                    regular += __popcll(__ballot(vq == 0 && e < kOdd / 2));
                    scale[h] = power_of_two(e < kOdd / 2 ? e : 0);
                    if (vq == 0) vector_exp[vr + h * 64] = e;
                }
                if (lane == 0) atomicAdd(const_cast<uint32_t *>(regular_count) + turn, regular);
                if (thread == 0) *left_count = 0;
#pragma unroll
                for (int t = 0; t < 2; ++t) {
                    char *stage = lds_h + t * STAGE;
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        halfx2 hi[2], lo[2];
                        split2(gv[t][r][0], gv[t][r][1], scale[r], hi[0], lo[0]);
                        split2(gv[t][r][2], gv[t][r][3], scale[r], hi[1], lo[1]);
                        *reinterpret_cast<halfx4 *>(stage + wr_v + r * 64 * ROWB) = halfx4{hi[0][0], hi[0][1], hi[1][0], hi[1][1]};
                        *reinterpret_cast<halfx4 *>(stage + wr_v + r * 64 * ROWB + V_PLANE) = halfx4{lo[0][0], lo[0][1], lo[1][0], lo[1][1]};
                    }
#pragma unroll
                    for (int r = 0; r < 2; ++r)
#pragma unroll
                        for (int p = 0; p < 2; ++p) *reinterpret_cast<uintx4 *>(stage + wr_a + r * 128 * ROWB + p * A_PLANE) = ga[t][r][p];
                }
                floatx4 v_set[4];
                uintx4 c_set[2][2];
#pragma unroll
                for (int h = 0; h < 4; ++h) v_set[h] = gv[2][h];
#pragma unroll
                for (int h = 0; h < 2; ++h)
#pragma unroll
                    for (int p = 0; p < 2; ++p) c_set[h][p] = ga[2][h][p];
#pragma unroll
                for (int rb = 0; rb < NB; ++rb)
#pragma unroll
                    for (int cb = 0; cb < NB; ++cb)
#pragma unroll
                        for (int e = 0; e < 16; ++e) acc[rb][cb][e] = 0.f;
                lds_barrier();

                // operand registers of the stage being contracted: fa[block][plane], fv[block][plane]
                halfx8 fa[NB][2], fv[NB][2];
                auto read_a1 = [&](const char *stage, int b, int p) __attribute__((always_inline)) {
                    fa[b][p] = *reinterpret_cast<const halfx8 *>(stage + rd_a + b * 32 * ROWB + p * A_PLANE);
                };
                auto read_v1 = [&](const char *stage, int b, int p) __attribute__((always_inline)) {
                    fv[b][p] = *reinterpret_cast<const halfx8 *>(stage + rd_v + b * 32 * ROWB + p * V_PLANE);
                };
#pragma unroll
                for (int b = 0; b < NB; ++b) {
                    read_v1(lds_h, b, 1);
                    read_a1(lds_h, b, 0);
                    read_v1(lds_h, b, 0);
                }

                // One stage.  LDS holds three: s (in the operand registers, but for the low coefficients), s + 1
                // (written during the previous iteration, read into the freed operand registers during this one)
                // and s + 2 (written during this one from the load registers, which then take the loads of
                // stage s + 3).  Products a1 v2 by columns, a1 v1 by rows, a2 v1 by columns: an operand is
                // refilled when its last product has been issued, 16 MFMAs or more before its first one in the
                // next stage; a2 is used in every column of the last product and is read during the first one.
                auto iteration = [&](uint32_t s) __attribute__((always_inline)) {
                    const char *cur = lds_h + (s % 3) * STAGE;
                    const char *nxt = lds_h + ((s + 1) % 3) * STAGE;
                    char *far = lds_h + ((s + 2) % 3) * STAGE;  // last read before the barrier of the iteration before
                    halfx2 hi[2], lo[2];  // a vector row on its way
                    // a quarter of the split of row r: two elements to their high or, after that, their low halves
                    auto split_quarter = [&](int r, int quarter) __attribute__((always_inline)) {
                        const int e = quarter / 2;
                        const float x0 = v_set[r][2 * e], x1 = v_set[r][2 * e + 1];
                        if (quarter % 2 == 0) {
                            hi[e] = __builtin_convertvector((floatx2{x0 * scale[r], x1 * scale[r]}), halfx2);
                            largest[r] = fmaxf(fmaxf(fabsf(x0), fabsf(x1)), largest[r]);
                        } else {
                            lo[e] = __builtin_convertvector((floatx2{__builtin_fmaf(x0, scale[r], -(float)hi[e][0]),
                                                                     __builtin_fmaf(x1, scale[r], -(float)hi[e][1])}), halfx2);
                        }
                    };
                    auto write_v = [&](int r, int p) __attribute__((always_inline)) {
                        *reinterpret_cast<halfx4 *>(far + wr_v + r * 64 * ROWB + p * V_PLANE) =
                            p == 0 ? halfx4{hi[0][0], hi[0][1], hi[1][0], hi[1][1]} : halfx4{lo[0][0], lo[0][1], lo[1][0], lo[1][1]};
                    };
                    auto coefficient = [&](int at, bool load) __attribute__((always_inline)) {
                        const int r = at / 2, p = at % 2;
                        if (load) c_set[r][p] = load_a(s + 3, r, p);
                        else *reinterpret_cast<uintx4 *>(far + wr_a + r * 128 * ROWB + p * A_PLANE) = c_set[r][p];
                    };
                    // What goes out after MFMA j (0..15) of product k (0..2): one memory instruction at most, or two
                    // LDS reads, and a quarter of the split of a vector row beside it.  The LDS accesses that the
                    // barrier behind product 0 waits for are issued three MFMAs before it or earlier.
                    auto after = [&](auto K_, auto I_) __attribute__((always_inline)) {
                        constexpr int k = decltype(K_)::value, j = decltype(I_)::value;
                        if constexpr (k == 0) {
                            if constexpr (j < 4) { read_a1(cur, j, 1); split_quarter(0, j); }
                            if constexpr (j == 4 || j == 5) write_v(0, j - 4);
                            if constexpr (j == 6) v_set[0] = load_v(s + 3, 0);
                            if constexpr (j >= 7 && j < 11) split_quarter(1, j - 7);
                            if constexpr (j == 11 || j == 12) write_v(1, j - 11);
                            if constexpr (j == 14) v_set[1] = load_v(s + 3, 1);
                        } else if constexpr (k == 1) {
                            if constexpr (j % 4 == 3) read_a1(nxt, j / 4, 0);
                            if constexpr (j < 4) { read_v1(nxt, j, 1); split_quarter(2, j); }
                            if constexpr (j == 4 || j == 5) write_v(2, j - 4);
                            if constexpr (j == 6) v_set[2] = load_v(s + 3, 2);
                            if constexpr (j == 8 || j == 10) coefficient(j / 2 - 4, false);
                            if constexpr (j == 9 || j == 12) coefficient(j / 3 - 3, true);
                            if constexpr (j == 13) coefficient(2, false);
                            if constexpr (j == 14) coefficient(2, true);
                        } else {
                            if constexpr (j % 4 == 3) read_v1(nxt, j / 4, 0);
                            if constexpr (j < 4) split_quarter(3, j);
                            if constexpr (j == 4 || j == 5) write_v(3, j - 4);
                            if constexpr (j == 6) v_set[3] = load_v(s + 3, 3);
                            if constexpr (j == 8) coefficient(3, false);
                            if constexpr (j == 9) coefficient(3, true);
                        }
                    };
                    auto product = [&](auto K_, auto PA_, auto PV_, auto BY_ROW_) __attribute__((always_inline)) {
                        constexpr int pa = decltype(PA_)::value, pv = decltype(PV_)::value;
                        constexpr bool by_row = decltype(BY_ROW_)::value;
                        [&]<int... I>(std::integer_sequence<int, I...>) __attribute__((always_inline)) {
                            (([&] {
                                constexpr int rb = by_row ? I / 4 : I % 4, cb = by_row ? I % 4 : I / 4;
                                acc[rb][cb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(fa[rb][pa], fv[cb][pv], acc[rb][cb], 0, 0, 0);
                                __builtin_amdgcn_sched_barrier(0);
                                after(K_, std::integral_constant<int, I>{});
                                __builtin_amdgcn_sched_barrier(0);
                            }()), ...);
                        }(std::make_integer_sequence<int, 16>{});
                    };
                    using std::integral_constant;
                    __builtin_amdgcn_sched_barrier(0);
                    product(integral_constant<int, 0>{}, integral_constant<int, 0>{}, integral_constant<int, 1>{}, std::false_type{});
                    lds_barrier();  // stage s + 1 is complete in LDS (the product before touched stage s and the free slot only)
                    __builtin_amdgcn_sched_barrier(0);
                    product(integral_constant<int, 1>{}, integral_constant<int, 0>{}, integral_constant<int, 0>{}, std::true_type{});
                    product(integral_constant<int, 2>{}, integral_constant<int, 1>{}, integral_constant<int, 0>{}, std::false_type{});
                };
                contracted = __builtin_amdgcn_readfirstlane(regular_count[turn]) > kFewRegular;
                bool mine = false;  // a coordinate that this thread brings in of row vr left fp16
                if (contracted) {
                    for (uint32_t s = 0; s < stages; ++s) iteration(s);
                    mine = largest[0] * scale[0] > kLargestHalf;
                    uint32_t left = 0;
#pragma unroll
                    for (int h = 0; h < 4; ++h) {
                        largest[h] = fmaxf(largest[h], __shfl_xor(largest[h], 1));
                        largest[h] = fmaxf(largest[h], __shfl_xor(largest[h], 2));
                        const bool leaves = vq == 0 && largest[h] * scale[h] > kLargestHalf;
                        if (leaves) vector_exp[vr + h * 64] = kOdd;
                        left += __popcll(__ballot(leaves));
                    }
                    if (lane == 0 && left) atomicAdd(const_cast<uint32_t *>(left_count), left);
                }
                lds_barrier();  // also: the next prologue writes stages that the last iterations read
                if (contracted && __builtin_amdgcn_readfirstlane(*left_count) >= TVW / 2 && __any(mine)) {
                    for (uint32_t s = 3; s < stages; s += 4) {
                        floatx4 w[4];
#pragma unroll
                        for (int u = 0; u < 4; ++u) w[u] = load_v(s + u, 0);
#pragma unroll
                        for (int u = 0; u < 4; ++u)
                            if (mine && s + u < stages && largest_of(w[u], 0.f) * scale[0] > kLargestHalf) *left_stage = s + u;
                    }
                }
            }
            turn ^= 1;
            if (thread == 0) regular_count[turn] = 0;  // added to again behind the barrier that ends this tile
            if (vt * TVW + thread < a.N) {
                const uint16_t in = (uint16_t)(tiles * TVW + thread);
                if (vector_exp[thread] >= kOdd / 2) odd_list[atomicAdd(const_cast<uint32_t *>(odd_count), 1u)] = in;
                else if (!contracted) odd_list[kSegment * TVW - 1 - atomicAdd(const_cast<uint32_t *>(few_count), 1u)] = in;
            }

            // Epilogue (odd vectors' results are stored over later): register 4q + e of block (rb, cb) is function 8q + 4 (l / 32) + e of the
            // block's 32, vector l % 32.  A block passes through a wave-private piece of LDS (the stages are
            // free now), from which eight neighbouring lanes take the 32 results of one vector, 128 bytes.
            if (contracted) {
                int ve[NB];
#pragma unroll
                for (int cb = 0; cb < NB; ++cb) ve[cb] = vector_exp[vw * 32 * NB + cb * 32 + lr];
                char *const block = lds_h + wave * (32 * kResultRow);
#pragma unroll
                for (int rb = 0; rb < NB; ++rb) {
                    const uint32_t j0 = ft * TF + fw * 32 * NB + rb * 32;
                    const uint32_t j = j0 + 4 * (lane & 7);  // of the results this lane stores
                    intx4 fe[4];
                    floatx4 b4[4];
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        fe[q] = *reinterpret_cast<const intx4 *>(a.fexp + j0 + 8 * q + 4 * lh);  // below kpad
                        if constexpr (!PROJ) {
                            b4[q] = *reinterpret_cast<const floatx4 *>(a.off + j0 + 8 * q + 4 * lh);
                            if constexpr (POW2) b4[q] *= a.inv_w;
                        }
                    }
#pragma unroll
                    for (int cb = 0; cb < NB; ++cb) {
#pragma unroll
                        for (int q = 0; q < 4; ++q) {
                            uintx4 v;
#pragma unroll
                            for (int e = 0; e < 4; ++e) {
                                const float p = __builtin_ldexpf(acc[rb][cb][4 * q + e], -(fe[q][e] + ve[cb]));
                                if constexpr (PROJ) {
                                    v[e] = __float_as_uint(p);
                                } else {
                                    const float h = POW2 ? fmaf(p, a.inv_w, b4[q][e]) : (p + b4[q][e]) / a.w;
                                    v[e] = (uint32_t)(int)floorf(h);
                                }
                            }
                            *reinterpret_cast<uintx4 *>(block + lr * kResultRow + q * 32 + lh * 16) = v;
                        }
                        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
                        __builtin_amdgcn_wave_barrier();
                        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
                        const uint64_t vec0 = vt * TVW + vw * 32 * NB + cb * 32;
#pragma unroll
                        for (int q = 0; q < 4; ++q) {
                            const uint32_t r = q * 8 + (lane >> 3);
                            const uintx4 v = *reinterpret_cast<const uintx4 *>(block + r * kResultRow + (lane & 7) * 16);
                            if (vec0 + r < a.N) {
                                uint32_t *dst = reinterpret_cast<uint32_t *>(a.out) + (vec0 + r) * a.k + j;
                                if constexpr (VEC) {
                                    if (j < a.k) {
                                        if (whole_lines) __builtin_nontemporal_store(v, reinterpret_cast<uintx4 *>(dst));
                                        else *reinterpret_cast<uintx4 *>(dst) = v;
                                    }
                                } else {
#pragma unroll
                                    for (int e = 0; e < 4; ++e)
                                        if (j + e < a.k) dst[e] = v[e];
                                }
                            }
                        }
                        __builtin_amdgcn_wave_barrier();
                    }
                }
            }
            lds_barrier();  // the exponents and the results have been read
            if (++tiles < kSegment && vt + vt_step < Vt) continue;
            const uint32_t odd = __builtin_amdgcn_readfirstlane(*odd_count), few = __builtin_amdgcn_readfirstlane(*few_count);
            if (odd + few) {
                __syncthreads();  // what the waves stored for odd vectors is where it belongs, and gets stored over
                uint32_t thread = threadIdx.x;
                asm volatile("" : "+v"(thread));  // as above
                const wide::Args x = a.exact();
                const Listed listed{odd_list, vt - (tiles - 1) * vt_step, vt_step, odd - 1};
                auto blocks = [&](uint32_t first, uint32_t count, auto run) {  // 32 functions x 32 vectors a wave
                    for (uint32_t b = thread >> 6; b < (count + 31) / 32 * 8; b += 4) {
                        const uint32_t j0 = __builtin_amdgcn_readfirstlane(ft * TF + (b & 7) * 32), at = (b >> 3) * 32 + (thread & 31);
                        if (j0 < a.k) run(j0, listed.wanted(first + (at < count ? at : count - 1)), at < count);
                    }
                };
                blocks(kSegment * TVW - few, few, [&](uint32_t j0, uint64_t row, bool store) { few_block<PROJ, POW2, VEC>(a, thread, j0, row, store); });
                if (odd <= kFewOdd) {
                    blocks(0, odd, [&](uint32_t j0, uint64_t row, bool store) { wide::block<PROJ, POW2, VEC>(x, thread, j0, row, store); });
                } else {
                    for (Listed rows = listed; rows.first < odd; rows.first += TVW)
                        wide::tile<PROJ, POW2, VEC>(x, lds_h, thread, ft, rows, odd - rows.first);
                }
                __syncthreads();
                if (threadIdx.x == 0) *odd_count = 0, *few_count = 0;
                lds_barrier();
            }
            tiles = 0;
        }
    }
}

}  // namespace

namespace {

// the fp16 nearest to x (ties to even), |x| below 2^15, and its value: bit arithmetic, since the host's own
// conversion is a library call per number
uint16_t to_half(float x, float &value) {
    uint32_t u;
    std::memcpy(&u, &x, 4);
    const uint32_t sign = u & 0x80000000u, mag = u ^ sign;
    uint32_t h, rounded;
    if (mag >= 0x38800000u) {  // 2^-14: 13 bits of the significand are rounded off
        rounded = (mag + 0xFFFu + ((mag >> 13) & 1u)) & ~0x1FFFu;
        h = (rounded >> 13) - (112u << 10);
    } else {  // a multiple of 2^-24, the spacing of floats at 1/2: the sum rounds to it
        float s;
        std::memcpy(&s, &mag, 4);
        s += 0.5f;
        std::memcpy(&h, &s, 4);
        h -= 0x3F000000u;
        s -= 0.5f;
        std::memcpy(&rounded, &s, 4);
    }
    rounded |= sign;
    std::memcpy(&value, &rounded, 4);
    return (uint16_t)(h | (sign >> 16));
}

}  // namespace

// Only where every function takes all n coordinates.  A vector's scale comes from all of them, so with m < n (a
// sampled object under LSH_DENSE_MATRIX) a large coordinate that a function does not sample would push the ones it
// samples below fp16's range; the bf16 splits have fp32's range and such a coordinate meets coefficient 0.
bool dense_half_used(const lsh_params *p) { return p->m == p->n && p->m >= kHalfMinTerms; }

// The two fp16 planes of a coefficient matrix [k][n] in the order the kernel reads them,
// [function tile of 256][stage of 16 coordinates][plane][row][coordinate], zeros beyond k and n, and
// behind them the exponent (32 bits) of every function.
void build_half_planes(const float *a, uint32_t k, uint32_t n, uint32_t kpad, uint32_t npad, std::vector<uint16_t> &planes) {
    const size_t elements = (size_t)2 * kpad * npad;
    planes.assign(elements + (size_t)2 * kpad, 0);
    const uint32_t stages = npad / KB;
    for (uint32_t j = 0; j < k; ++j) {
        float top = 0.f;
        for (uint32_t c = 0; c < n; ++c) {
            const float x = std::fabs(a[(size_t)j * n + c]);
            top = x > top ? x : top;
        }
        int32_t e = top > 0.f && std::isfinite(top) ? kFunctionTop - std::ilogb(top) : 0;
        if (e > 126) e = 126;  // 2^e is a normal float
        std::memcpy(planes.data() + elements + (size_t)2 * j, &e, 4);
        const float scale = std::ldexp(1.0f, e);
        for (uint32_t c = 0; c < n; ++c) {
            const float x = a[(size_t)j * n + c] * scale;
            float hi, lo;
            const size_t at = ((size_t)(j / TF) * stages + c / KB) * kStagePlanes + (size_t)(j % TF) * KB + c % KB;
            planes[at] = to_half(x, hi);
            planes[at + TF * KB] = to_half(x - hi, lo);
        }
    }
}

int launch_dense_half(const lsh_params *p, bool proj, const float *d_data, uint64_t N, void *d_out, void *stream) {
    HalfArgs a;
    a.data = d_data;
    a.planes = static_cast<const uint16_t *>(p->d_half_planes);
    a.exact_planes = static_cast<const uint16_t *>(p->d_dense_planes);
    a.off = p->d_off;
    a.N = N;
    a.n = p->n;
    a.npad = (p->n + KB - 1) / KB * KB;
    a.k = p->k;
    a.kpad = (p->k + TF - 1) / TF * TF;
    a.fexp = reinterpret_cast<const int *>(a.planes + (size_t)2 * a.kpad * a.npad);
    a.w = p->w;
    a.inv_w = 1.0f / p->w;
    a.out = d_out;
    int exp2 = 0;
    const bool pw = proj || std::frexp(p->w, &exp2) == 0.5f;
    const bool vec = p->k % 4 == 0;
    const uint64_t waves = (N + 31) / 32 * ((p->k + 31) / 32);
    const bool few = waves <= kFewWaves;
    // one workgroup per CU (152 KB of LDS, all registers), a multiple of 8 so that every XCD gets the same number
    uint32_t wgs = (uint32_t)(p->num_cus > 0 ? p->num_cus : 256) / 8 * 8;
    if (wgs < 8) wgs = 8;
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
#define LSH_HALF_CASE(P_, W_, V_) \
    if (proj == P_ && pw == W_ && vec == V_ && few) { \
        hipLaunchKernelGGL((dense_half_few_kernel<P_, W_, V_>), dim3((p->k + 127) / 128, (uint32_t)((N + 31) / 32)), dim3(256), 0, s, a); \
    } else if (proj == P_ && pw == W_ && vec == V_) { \
        auto fn = &dense_half_kernel<P_, W_, V_>; \
        if (ensure_lds_limit(reinterpret_cast<const void *>(fn), kLdsBytesH) != LSH_OK) return LSH_ERR_HIP; \
        hipLaunchKernelGGL(fn, dim3(wgs), dim3(kThreadsH), kLdsBytesH, s, a); \
    }
    LSH_HALF_CASE(false, true, true) LSH_HALF_CASE(false, false, true) LSH_HALF_CASE(true, true, true)
    LSH_HALF_CASE(false, true, false) LSH_HALF_CASE(false, false, false) LSH_HALF_CASE(true, true, false)
#undef LSH_HALF_CASE
    return hipGetLastError() == hipSuccess ? LSH_OK : LSH_ERR_HIP;
}

}  // namespace lsh
