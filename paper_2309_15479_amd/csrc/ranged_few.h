// What ranged_few_kernel (ranged_kernel.hip) reads of a wave's lists and where its LDS holds an entry's coordinate: compiled
// into the kernel and into the host's walk of the same lists (selfcheck.cpp).
#pragma once
#include <hip/hip_runtime.h>

#include <type_traits>

#include "lsh_internal.h"

namespace lsh {

// LDS holds four whole vectors as slots of 16 bytes, one coordinate of the four each, in ranges of kWindowCoords: one for
// each stage of a tile, up to kFewStages.
constexpr uint32_t kFewStages = 160 * 1024 / (kWindowCoords * 16);
// Quads of entries requested ahead of their use.
constexpr uint32_t kFewAhead = 8;

typedef unsigned short ushortx2 __attribute__((ext_vector_type(2)));

// A pair of entries names slots of the ring of ranges, 1024 x (range modulo 8) + coordinate in the range.  The range meant is the
// one among those readable in the pair's stage, stage .. stage + 6, that has the ring slot: -> 256 x range + coordinate, two
// numbers at a time.  (Padding entries name the stage's own range: LDS holds zeros for stages without a range.)
__host__ __device__ __forceinline__ uint32_t few_slots(uint32_t pair, uint32_t stage) {
    const ushortx2 since = __builtin_bit_cast(ushortx2, pair) - (unsigned short)(stage << 10);
    const ushortx2 far = (since & (unsigned short)0x1C00) >> (unsigned short)2;
    return __builtin_bit_cast(uint32_t, (since & (unsigned short)0xFF) + far + (unsigned short)(stage << 8));
}

// The order in which a wave works through its `quads` quads, kFewAhead of them having been requested: read(q, d) brings the
// coordinates of quad q, requested as number d = q % kFewAhead, multiply(q, d) adds its products, request(q, d) asks for
// quad q in place of the one multiplied last.
template <class Read, class Multiply, class Request>
__host__ __device__ __forceinline__ void few_quads(uint32_t quads, Read read, Multiply multiply, Request request) {
    read(0, 0);
    // No test around a request: the compiler's count of those in flight is then exact (with tests it waited for the newest one,
    // a trip to L2 a quad).  The last group, up to eight quads, has none, and tests for the end of the list instead: behind it
    // there is nothing to read.
    auto eight = [&](auto last_tag, uint32_t q0) __attribute__((always_inline)) {
        constexpr bool last = decltype(last_tag)::value;
#pragma unroll
        for (uint32_t d = 0; d < kFewAhead; ++d) {
            const uint32_t q = q0 + d;
            if (!last || q + 1 < quads) read(q + 1, (d + 1) % kFewAhead);
            if (!last || q < quads) multiply(q, d);
            if constexpr (!last) request(q + kFewAhead, d);
        }
    };
    uint32_t q0 = 0;
    for (; q0 + kFewAhead < quads; q0 += kFewAhead) eight(std::false_type{}, q0);
    eight(std::true_type{}, q0);
}

}  // namespace lsh
