// The dense product from exact three-way bf16 splits (see dense_split_kernel.hip for the arithmetic, and
// dense_split_wide_kernel.hip for the tile and why it looks like this): one tile of 256 functions x 256
// vectors by a workgroup of four waves, and one block of 32 x 32 by a wave.  A result is the same number from either.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>
#include <type_traits>
#include <utility>

#include "device_utils.h"

namespace lsh {
namespace wide {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef uint32_t uintx4 __attribute__((ext_vector_type(4)));
typedef float floatx4 __attribute__((ext_vector_type(4)));

constexpr int TF = 256;    // functions per tile
constexpr int TVW = 256;   // vectors per tile
constexpr int NB = 4;      // 32 x 32 blocks of a wave along either axis: a wave owns 128 functions x 128 vectors
constexpr int KB = 16;     // coordinates per stage = one MFMA step
constexpr int ROWB = 32;   // bytes per row and plane in a stage: two 16-byte halves, swapped in rows with bit 3 set
constexpr int A_PLANE = TF * ROWB, V_PLANE = TVW * ROWB;
constexpr int STAGE = 3 * (A_PLANE + V_PLANE);  // 49152 bytes
constexpr int kThreads = 256;
constexpr int kStagePlanes = 3 * TF * KB;  // bf16 elements of one function tile's three planes in one stage
constexpr int kLdsBytes = 3 * STAGE;

struct Args {
    const float *data;       // [N][n]
    const uint16_t *planes;  // [kpad / 256][npad / 16][3][256][16] bf16 bit patterns
    const float *off;        // [>= kpad]
    uint64_t N;
    uint32_t n, npad, k, kpad;
    float w, inv_w;
    void *out;               // [N][k]
};

// x = x1 + x2 + x3 exactly, each a bf16 (round to nearest even)
__device__ __forceinline__ void split3(float x, __bf16 &x1, __bf16 &x2, __bf16 &x3) {
    x1 = (__bf16)x;
    const float r1 = x - (float)x1;
    x2 = (__bf16)r1;
    x3 = (__bf16)(r1 - (float)x2);
}

// PROJ: raw projections instead of bucket ids.  POW2: w is a power of two (fma(p, 1/w, b/w) is
// then the same float as (p + b) / w).
template <bool PROJ, bool POW2>
__device__ __forceinline__ uint32_t result(const Args &a, float p, float b) {  // b: offset, times 1/w if POW2
    if constexpr (PROJ) return __float_as_uint(p);
    return (uint32_t)(int)floorf(POW2 ? fmaf(p, a.inv_w, b) : (p + b) / a.w);
}

// Function tile ft against 256 vectors, of which the first `count` are wanted.  rows.wanted(i): the number of the
// vector, i below count; rows.any(i): the same, and of any vector for i from count on.  VEC: k is a multiple of 4
// (16-byte stores).  lds: kLdsBytes; free for other use by all waves after a barrier.  thread: threadIdx.x.
template <bool PROJ, bool POW2, bool VEC, typename Rows>
__device__ __forceinline__ void tile(const Args &a, char *lds, uint32_t thread, uint32_t ft, const Rows &rows, uint32_t count) {
    const uint32_t lane = thread & 63, wave = __builtin_amdgcn_readfirstlane(thread >> 6);
    const uint32_t lr = lane & 31, lh = lane >> 5;
    const uint32_t fw = wave & 1, vw = wave >> 1;  // the wave's half of the functions, half of the vectors

    // loading roles: 16 bytes of the vector tile and of each coefficient plane per stage
    const uint32_t vr = thread >> 2, vq = thread & 3;  // vector rows vr + 64 h (h < 4), 4-coordinate piece
    const uint32_t ar = thread >> 1, ah = thread & 1;  // coefficient rows ar and ar + 128, 8-coordinate half
    const uint32_t stages = a.npad / KB;

    // operand read and write offsets inside a stage (half h of row r sits at 16 * (h ^ bit 3 of r))
    const uint32_t rd_a = (fw * 32 * NB + lr) * ROWB + ((lh ^ ((lr >> 3) & 1)) << 4);                // + rb * 32 rows + plane
    const uint32_t rd_v = 3 * A_PLANE + (vw * 32 * NB + lr) * ROWB + ((lh ^ ((lr >> 3) & 1)) << 4);  // + cb * 32 rows + plane
    const uint32_t wr_a = ar * ROWB + ((ah ^ ((ar >> 3) & 1)) << 4);
    const uint32_t wr_v = 3 * A_PLANE + vr * ROWB + (((vq >> 1) ^ ((vr >> 3) & 1)) << 4) + ((vq & 1) << 3);
    // the planes are stored stage by stage: [function tile][stage][plane][256 rows][16 coordinates],
    // so the 64 lanes of a load read 1 KB in one piece (thread t: 16 bytes at 16 t of rows 0-127)
    const uint16_t *arow = a.planes + (size_t)ft * stages * kStagePlanes + thread * 8;
    const float *vrow[4];
#pragma unroll
    for (int h = 0; h < 4; ++h) {
        vrow[h] = a.data + rows.any(vr + h * 64) * a.n + vq * 4;
    }

    // the registers of the global loads: the stage on its way to LDS
    floatx4 gv[4];
    uintx4 ga[2][3];
    // Every load is issued unconditionally (the compiler can then count the loads in flight
    // exactly and wait for the oldest only): stages beyond the last read the last stage's
    // coefficients against zeros.
    auto gload = [&](uint32_t s, floatx4 (&v)[4], uintx4 (&c)[2][3]) __attribute__((always_inline)) {
        const uint32_t k0 = s * KB;
        // coordinates beyond n read the row's first ones instead; lstore() replaces them by zeros
#pragma unroll
        for (int h = 0; h < 4; ++h) v[h] = *reinterpret_cast<const floatx4 *>(vrow[h] + (k0 + vq * 4 < a.n ? k0 : 0u));
        const uint32_t ka = s < stages ? s : stages - 1;  // stage
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int p = 0; p < 3; ++p)
                c[h][p] = *reinterpret_cast<const uintx4 *>(arow + (size_t)ka * kStagePlanes + p * (TF * KB) + h * 128 * KB);
    };
    auto lstore = [&](char *stage, uint32_t s, const floatx4 (&v)[4], const uintx4 (&c)[2][3]) __attribute__((always_inline)) {
        const bool inside = s * KB + vq * 4 < a.n;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            bf16x4 h[3];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                __bf16 x1, x2, x3;
                split3(inside ? v[r][e] : 0.f, x1, x2, x3);
                h[0][e] = x1;
                h[1][e] = x2;
                h[2][e] = x3;
            }
#pragma unroll
            for (int p = 0; p < 3; ++p) *reinterpret_cast<bf16x4 *>(stage + wr_v + r * 64 * ROWB + p * V_PLANE) = h[p];
        }
#pragma unroll
        for (int r = 0; r < 2; ++r)
#pragma unroll
            for (int p = 0; p < 3; ++p) *reinterpret_cast<uintx4 *>(stage + wr_a + r * 128 * ROWB + p * A_PLANE) = c[r][p];
    };

    floatx16 acc[NB][NB];
#pragma unroll
    for (int rb = 0; rb < NB; ++rb)
#pragma unroll
        for (int cb = 0; cb < NB; ++cb)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[rb][cb][e] = 0.f;

    // Operand registers of the stage being contracted: fa[block][plane], fv[block][plane].
    // A plane's registers are read again, for the next stage, as soon as the last product
    // that uses them has been issued.
    bf16x8 fa[NB][3], fv[NB][3];
    auto read_a = [&](const char *stage, int p) __attribute__((always_inline)) {
#pragma unroll
        for (int b = 0; b < NB; ++b)
            fa[b][p] = *reinterpret_cast<const bf16x8 *>(stage + rd_a + b * 32 * ROWB + p * A_PLANE);
    };
    auto read_v = [&](const char *stage, int p) __attribute__((always_inline)) {
#pragma unroll
        for (int b = 0; b < NB; ++b)
            fv[b][p] = *reinterpret_cast<const bf16x8 *>(stage + rd_v + b * 32 * ROWB + p * V_PLANE);
    };
    auto read_a1 = [&](const char *stage, int b, int p) __attribute__((always_inline)) {
        fa[b][p] = *reinterpret_cast<const bf16x8 *>(stage + rd_a + b * 32 * ROWB + p * A_PLANE);
    };
    auto read_v1 = [&](const char *stage, int b, int p) __attribute__((always_inline)) {
        fv[b][p] = *reinterpret_cast<const bf16x8 *>(stage + rd_v + b * 32 * ROWB + p * V_PLANE);
    };
    // single loads of the next stage's operands, small enough to go out in the shadow of one MFMA
    auto load_v_row = [&](uint32_t s, int h, floatx4 (&v)[4]) __attribute__((always_inline)) {
        const uint32_t k0 = s * KB;
        v[h] = *reinterpret_cast<const floatx4 *>(vrow[h] + (k0 + vq * 4 < a.n ? k0 : 0u));
    };
    auto load_a_piece = [&](uint32_t s, int h, int p, uintx4 (&c)[2][3]) __attribute__((always_inline)) {
        const uint32_t ka = s < stages ? s : stages - 1;  // stage
        c[h][p] = *reinterpret_cast<const uintx4 *>(arow + (size_t)ka * kStagePlanes + p * (TF * KB) + h * 128 * KB);
    };

    // One stage.  LDS holds three stages: s (in the operand registers by now), s + 1 (written
    // during the previous iteration, read into the freed operand registers during this one)
    // and s + 2 (written during this one from the load registers, which then take the loads
    // of stage s + 3).  A wave is alone on its SIMD, so everything that is not an MFMA is cut
    // into pieces that go out one after each MFMA: an operand register is refilled right
    // after the last MFMA that reads it, the stores to LDS and the global loads ride along.
    auto iteration = [&](uint32_t s, floatx4 (&v_set)[4], uintx4 (&c_set)[2][3]) __attribute__((always_inline)) {
        const char *cur = lds + (s % 3) * STAGE;
        const char *nxt = lds + ((s + 1) % 3) * STAGE;
        char *far = lds + ((s + 2) % 3) * STAGE;  // last read two iterations ago: free since the barrier before this one
        const bool inside = (s + 2) * KB + vq * 4 < a.n;
        bf16x4 h[3];  // a vector row on its way: split in one product, written during the next
        auto split_element = [&](int r, int e) __attribute__((always_inline)) {
            __bf16 x1, x2, x3;
            split3(inside ? v_set[r][e] : 0.f, x1, x2, x3);
            h[0][e] = x1;
            h[1][e] = x2;
            h[2][e] = x3;
        };
        auto write_plane = [&](int r, int pl) __attribute__((always_inline)) {
            *reinterpret_cast<bf16x4 *>(far + wr_v + r * 64 * ROWB + pl * V_PLANE) = h[pl];
        };
        auto store_a = [&](int r, int pl) __attribute__((always_inline)) {
            *reinterpret_cast<uintx4 *>(far + wr_a + r * 128 * ROWB + pl * A_PLANE) = c_set[r][pl];
        };
        // What goes out after MFMA i (0..15) of product k (0..5) of the stage: at most one
        // memory instruction, or the split of one vector element.  Products 0, 1, 2 and 5 run
        // row by row, 3 and 4 column by column, so that after every fourth MFMA one operand
        // register has been read for the last time and is refilled from the next stage.
        auto after = [&](auto K_, auto I_) __attribute__((always_inline)) {
            constexpr int k = decltype(K_)::value, i = decltype(I_)::value;
            if constexpr (i % 4 == 3) {
                constexpr int q = i / 4;
                if constexpr (k == 0) read_v1(cur, q, 2);  // read in every row of the stage before's last product
                if constexpr (k == 1) read_a1(nxt, q, 1);
                if constexpr (k == 2) read_a1(nxt, q, 2);
                if constexpr (k == 3) read_v1(nxt, q, 1);
                if constexpr (k == 4) read_v1(nxt, q, 0);
                if constexpr (k == 5) read_a1(nxt, q, 0);
            } else if constexpr (k == 0 || k == 5) {  // the two coefficient rows: store, then load again
                constexpr int r = k == 0 ? 0 : 1;
                if constexpr (i < 3) store_a(r, i);
                if constexpr (i >= 4 && i < 7) load_a_piece(s + 3, r, i - 4, c_set);
                if constexpr (k == 0 && i >= 8 && i < 13) split_element(0, i < 11 ? i - 8 : 3);
            } else {  // products 1..4: write vector row k - 1, load it again, split row k
                if constexpr (i < 3) write_plane(k - 1, i);
                if constexpr (i == 4) load_v_row(s + 3, k - 1, v_set);
                if constexpr (k < 4 && (i == 5 || i == 6 || i == 8 || i == 9)) split_element(k, i < 7 ? i - 5 : i - 6);
            }
        };
        auto product = [&](auto K_, auto PA_, auto PV_, auto BY_ROW_) __attribute__((always_inline)) {
            constexpr int pa = decltype(PA_)::value, pv = decltype(PV_)::value;
            constexpr bool by_row = decltype(BY_ROW_)::value;
            [&]<int... I>(std::integer_sequence<int, I...>) __attribute__((always_inline)) {
                (([&] {
                    constexpr int rb = by_row ? I / 4 : I % 4, cb = by_row ? I % 4 : I / 4;
                    acc[rb][cb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[rb][pa], fv[cb][pv], acc[rb][cb], 0, 0, 0);
                    __builtin_amdgcn_sched_barrier(0);
                    after(K_, std::integral_constant<int, I>{});
                    __builtin_amdgcn_sched_barrier(0);
                }()), ...);
            }(std::make_integer_sequence<int, 16>{});
        };
        using std::integral_constant;
        __builtin_amdgcn_sched_barrier(0);
        product(integral_constant<int, 0>{}, integral_constant<int, 1>{}, integral_constant<int, 1>{}, std::true_type{});
        lds_barrier();  // stage s + 1 is complete in LDS (the product before touched stage s and the free slot only)
        __builtin_amdgcn_sched_barrier(0);
        product(integral_constant<int, 1>{}, integral_constant<int, 1>{}, integral_constant<int, 0>{}, std::true_type{});
        product(integral_constant<int, 2>{}, integral_constant<int, 2>{}, integral_constant<int, 0>{}, std::true_type{});
        product(integral_constant<int, 3>{}, integral_constant<int, 0>{}, integral_constant<int, 1>{}, std::false_type{});
        product(integral_constant<int, 4>{}, integral_constant<int, 0>{}, integral_constant<int, 0>{}, std::false_type{});
        product(integral_constant<int, 5>{}, integral_constant<int, 0>{}, integral_constant<int, 2>{}, std::true_type{});
    };

    // prologue: stages 0 and 1 to LDS, stage 2 on its way
    gload(0, gv, ga);
    lstore(lds, 0, gv, ga);
    gload(1, gv, ga);
    lstore(lds + STAGE, 1, gv, ga);
    gload(2, gv, ga);
    __syncthreads();
    read_a(lds, 1);  // in the order of the refills
    read_a(lds, 2);
    read_v(lds, 1);
    read_v(lds, 0);
    read_a(lds, 0);
    read_v(lds, 2);
    for (uint32_t s = 0; s < stages; ++s) iteration(s, gv, ga);
    __syncthreads();  // the next tile's prologue writes stages that the last iterations read

    // epilogue: register 4q + e of block (rb, cb) is function 8q + 4 (l / 32) + e of the
    // block's 32, vector l % 32
#pragma unroll
    for (int rb = 0; rb < NB; ++rb)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const uint32_t j = ft * TF + fw * 32 * NB + rb * 32 + 8 * q + 4 * lh;  // < kpad
            float b4[4] = {0.f, 0.f, 0.f, 0.f};
            if constexpr (!PROJ) {
                const floatx4 t = *reinterpret_cast<const floatx4 *>(a.off + j);
#pragma unroll
                for (int e = 0; e < 4; ++e) b4[e] = POW2 ? t[e] * a.inv_w : t[e];
            }
#pragma unroll
            for (int cb = 0; cb < NB; ++cb) {
                uintx4 v;
#pragma unroll
                for (int e = 0; e < 4; ++e) v[e] = result<PROJ, POW2>(a, acc[rb][cb][4 * q + e], b4[e]);
                const uint32_t at = vw * 32 * NB + cb * 32 + lr;
                if (at < count) {
                    uint32_t *dst = reinterpret_cast<uint32_t *>(a.out) + rows.wanted(at) * a.k + j;
                    if constexpr (VEC) {
                        if (j < a.k) *reinterpret_cast<uintx4 *>(dst) = v;
                    } else {
#pragma unroll
                        for (int e = 0; e < 4; ++e)
                            if (j + e < a.k) dst[e] = v[e];
                    }
                }
            }
        }
}

// Functions j0 ... j0 + 31 (j0 a multiple of 32 below k) against 32 vectors by one wave, operands straight from memory:
// lanes l and l + 32 take vector `row` and store its results if `store`.  No LDS, no barrier.  For few
// vectors: bound by the chain of six MFMAs and the split a stage (about 0.35 us), it takes a wave 20 us at n = 960.
template <bool PROJ, bool POW2, bool VEC>
__device__ __forceinline__ void block(const Args &a, uint32_t thread, uint32_t j0, uint64_t row, bool store) {
    constexpr int kSets = 2;
    const uint32_t lane = thread & 63, lr = lane & 31, lh = lane >> 5;
    const uint32_t stages = a.npad / KB;
    const uint16_t *arow = a.planes + (size_t)(j0 / TF) * stages * kStagePlanes + (j0 % TF + lr) * KB + lh * 8;
    const float *vrow = a.data + row * a.n + lh * 8;
    floatx4 v[kSets][2];
    bf16x8 c[kSets][3];
    // as in tile(): coordinates beyond n read the vector's first ones and count as zeros
    auto load = [&](uint32_t s, int d) __attribute__((always_inline)) {
#pragma unroll
        for (int h = 0; h < 2; ++h)
            v[d][h] = *reinterpret_cast<const floatx4 *>(vrow + h * 4 + (s * KB + lh * 8 + h * 4 < a.n ? s * KB : 0u));
        const uint32_t ka = s < stages ? s : stages - 1;
#pragma unroll
        for (int p = 0; p < 3; ++p) c[d][p] = *reinterpret_cast<const bf16x8 *>(arow + (size_t)ka * kStagePlanes + p * (TF * KB));
    };
    floatx16 acc;
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[e] = 0.f;
#pragma unroll
    for (int d = 0; d < kSets; ++d) load(d, d);
    for (uint32_t s0 = 0; s0 < stages; s0 += kSets) {
#pragma unroll
        for (int d = 0; d < kSets; ++d) {
            const uint32_t s = s0 + d;
            if (s < stages) {
                bf16x8 x[3];
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    __bf16 x1, x2, x3;
                    split3(s * KB + lh * 8 + e / 4 * 4 < a.n ? v[d][e / 4][e % 4] : 0.f, x1, x2, x3);
                    x[0][e] = x1;
                    x[1][e] = x2;
                    x[2][e] = x3;
                }
                // the products in the order of tile()
                acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(c[d][1], x[1], acc, 0, 0, 0);
                acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(c[d][1], x[0], acc, 0, 0, 0);
                acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(c[d][2], x[0], acc, 0, 0, 0);
                acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(c[d][0], x[1], acc, 0, 0, 0);
                acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(c[d][0], x[0], acc, 0, 0, 0);
                acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(c[d][0], x[2], acc, 0, 0, 0);
            }
            load(s + kSets, d);
        }
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const uint32_t j = j0 + 8 * q + 4 * lh;  // < kpad
        floatx4 b4 = {0.f, 0.f, 0.f, 0.f};
        if constexpr (!PROJ) {
            b4 = *reinterpret_cast<const floatx4 *>(a.off + j);
            if constexpr (POW2) b4 *= a.inv_w;
        }
        uintx4 r;
#pragma unroll
        for (int e = 0; e < 4; ++e) r[e] = result<PROJ, POW2>(a, acc[4 * q + e], b4[e]);
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
}

}  // namespace wide
}  // namespace lsh
