// Dense E2LSH projections (Sec. 2.2, Eq. 1) for any dimension n on the bf16 matrix cores of
// gfx950, with fp32 accuracy: P = V A^T from exact three-way bf16 splits of both operands and
// the six products of weight >= 2^-16 (see dense_split_kernel.hip for the arithmetic and its
// error: what is left out is below 2^-23 of each term |a_i v_i|).  The fp32 MFMA runs at a
// sixteenth of the bf16 rate, so six bf16 products are 16/6 of its speed at best.
//
//   V [N][n] fp32 row-major; A already split on the host into three bf16 planes, stored in the
//   order of use: [function tile of 256][stage of 16 coordinates][plane][row][coordinate]
//   (zero rows up to a multiple of 256, zero columns up to a multiple of 16).
//
// Workgroup = 4 waves, one per SIMD; tile = 256 functions x 256 vectors, contraction in stages
// of 16 coordinates.  A wave owns 128 functions x 128 vectors: 4 x 4 blocks of
// v_mfma_f32_32x32x16_bf16, 256 accumulator registers (functions are the row operand, so an
// accumulator lane holds runs of four consecutive functions of one vector).  The large tile is
// what counts: the time of this kernel follows the instructions that bring operands in (global
// loads, LDS writes, LDS reads) per multiply-add, and a 128 x 128 wave tile needs half as many
// as a 64 x 64 one.  Per stage a thread brings 16 bytes of four vector rows (4 fp32 each,
// split here on their way to LDS) and 16 bytes of each plane of two coefficient rows (8 bf16);
// LDS holds three stages, [plane][row][32 bytes], the two 16-byte halves of a row swapped in
// rows whose number has bit 3 set, which makes the 16-byte operand reads of 32 consecutive rows
// (and the writes) conflict-free without padding.  While stage s is contracted, the operand
// registers it has finished with are refilled from stage s + 1, stage s + 2 is written to LDS
// and the loads of stage s + 3 go out into the registers just stored (one set: a stage is 96
// MFMAs per wave, about 1.8 us).  With one wave per SIMD nothing else hides what a wave
// issues between two MFMAs, so the stage is written out MFMA by MFMA with at most one memory
// instruction or the split of one vector element after each (scheduling barriers keep that
// order); one LDS-only barrier per stage.
//
// The tile itself is in dense_wide_tile.h; dense_half_kernel.hip uses it, too.
//
// Placement: workgroup g runs on XCD g % 8.  XCD x takes the vector tiles x, x + 8, ...; the
// F function tiles of a vector tile go to F workgroups of that XCD, which walk the stages in
// step, so a vector stage is fetched into the XCD's L2 once and the other F - 1 workgroups hit
// there; a workgroup keeps its function tile for all its vector tiles, and the workgroups of
// an XCD that have the same one (workgroups per XCD / F of them) share its stages in L2, too.
// (With a number of function tiles that does not divide the workgroups of an XCD: function
// tiles dealt to the XCDs, every XCD walking all vectors.)
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstring>
#include <vector>

#include "dense_wide_tile.h"
#include "lsh_internal.h"

namespace lsh {
namespace {

using wide::TF;
using wide::TVW;
using wide::KB;
using wide::kStagePlanes;

struct Neighbours {
    uint64_t first, last;
    __device__ uint64_t wanted(uint32_t i) const { return first + i; }
    __device__ uint64_t any(uint32_t i) const { return first + i < last ? first + i : last; }
};

// PROJ, POW2, VEC: as in dense_wide_tile.h
template <bool PROJ, bool POW2, bool VEC>
__global__ __launch_bounds__(wide::kThreads) void dense_split_wide_kernel(const wide::Args a) {
    extern __shared__ __align__(16) char lds_w[];  // 3 stages x ([3][256][32] coefficients, [3][256][32] vectors)
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

    // When the number of function tiles divides an XCD's workgroups (the usual case), XCD x
    // takes the vector tiles x, x + 8, ... and F of its workgroups contract one of them at the
    // same time, each with its own function tile: the vector tile is then fetched into that
    // XCD's L2 once instead of once per XCD.
    const bool by_vector = per_xcd % F == 0 && F <= per_xcd;
    uint64_t vt_first = (uint64_t)i * reps + rep, vt_step = (uint64_t)per_xcd * reps;
    if (by_vector) {
        ft_first = i % F;
        ft_step = F;  // one function tile per workgroup
        const uint32_t groups = per_xcd / F;
        vt_first = x + 8ull * (i / F);
        vt_step = 8ull * groups;
    }
    for (uint32_t ft = ft_first; ft < F; ft += ft_step) {
        for (uint64_t vt = vt_first; vt < Vt; vt += vt_step) {
            const uint64_t left = a.N - vt * TVW;
            uint32_t thread = threadIdx.x;
            asm volatile("" : "+v"(thread));  // or every address made from it would be held through all tiles, in memory
            wide::tile<PROJ, POW2, VEC>(a, lds_w, thread, ft, Neighbours{vt * TVW, a.N - 1}, left < TVW ? (uint32_t)left : TVW);
        }
    }
}

uint16_t to_bf16(float x) {  // round to nearest even; NaN stays NaN
    uint32_t u;
    std::memcpy(&u, &x, 4);
    if ((u & 0x7F800000u) == 0x7F800000u) return (uint16_t)((u >> 16) | ((u & 0xFFFFu) ? 0x40u : 0u));
    return (uint16_t)((u + 0x7FFFu + ((u >> 16) & 1u)) >> 16);
}

float from_bf16(uint16_t h) {
    const uint32_t u = (uint32_t)h << 16;
    float x;
    std::memcpy(&x, &u, 4);
    return x;
}

}  // namespace

uint32_t dense_wide_row_tile() { return TF; }
uint32_t dense_wide_col_step() { return KB; }

// The three bf16 planes of a coefficient matrix [k][n] in the order the kernel reads them:
// [function tile of 256][stage of 16 coordinates][plane][row][coordinate], zeros beyond k and n.
void build_dense_planes(const float *a, uint32_t k, uint32_t n, uint32_t kpad, uint32_t npad,
                        std::vector<uint16_t> &planes) {
    planes.assign((size_t)3 * kpad * npad, 0);
    const uint32_t stages = npad / KB;
    for (uint32_t j = 0; j < k; ++j)
        for (uint32_t c = 0; c < n; ++c) {
            const float x = a[(size_t)j * n + c];
            const uint16_t h1 = to_bf16(x);
            const float r1 = x - from_bf16(h1);
            const uint16_t h2 = to_bf16(r1);
            const uint16_t h3 = to_bf16(r1 - from_bf16(h2));
            const size_t at = ((size_t)(j / TF) * stages + c / KB) * kStagePlanes + (size_t)(j % TF) * KB + c % KB;
            planes[at] = h1;
            planes[at + TF * KB] = h2;
            planes[at + 2 * TF * KB] = h3;
        }
}

bool dense_wide_supported(const lsh_params *p) {
    return p->m == p->n && p->d_dense_planes != nullptr && p->n % 4 == 0 && (uint64_t)p->k * 4 < (1ull << 32);
}

int launch_dense_wide(const lsh_params *p, bool proj, const float *d_data, uint64_t N, void *d_out, void *stream) {
    if (dense_half_used(p)) return launch_dense_half(p, proj, d_data, N, d_out, stream);
    wide::Args a;
    a.data = d_data;
    a.planes = static_cast<const uint16_t *>(p->d_dense_planes);
    a.off = p->d_off;
    a.N = N;
    a.n = p->n;
    a.npad = (p->n + KB - 1) / KB * KB;
    a.k = p->k;
    a.kpad = (p->k + TF - 1) / TF * TF;
    a.w = p->w;
    a.inv_w = 1.0f / p->w;
    a.out = d_out;
    int exp2 = 0;
    const bool pw = proj || std::frexp(p->w, &exp2) == 0.5f;
    const bool vec = p->k % 4 == 0;
    // one workgroup per CU (144 KB of LDS), a multiple of 8 so that every XCD gets the same number
    uint32_t wgs = (uint32_t)(p->num_cus > 0 ? p->num_cus : 256) / 8 * 8;
    if (wgs < 8) wgs = 8;
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
#define LSH_WIDE_CASE(P_, W_, V_) \
    if (proj == P_ && pw == W_ && vec == V_) { \
        auto fn = &dense_split_wide_kernel<P_, W_, V_>; \
        if (ensure_lds_limit(reinterpret_cast<const void *>(fn), wide::kLdsBytes) != LSH_OK) return LSH_ERR_HIP; \
        hipLaunchKernelGGL(fn, dim3(wgs), dim3(wide::kThreads), wide::kLdsBytes, s, a); \
    }
    LSH_WIDE_CASE(false, true, true) LSH_WIDE_CASE(false, false, true) LSH_WIDE_CASE(true, true, true)
    LSH_WIDE_CASE(false, true, false) LSH_WIDE_CASE(false, false, false) LSH_WIDE_CASE(true, true, false)
#undef LSH_WIDE_CASE
    return hipGetLastError() == hipSuccess ? LSH_OK : LSH_ERR_HIP;
}

}  // namespace lsh
