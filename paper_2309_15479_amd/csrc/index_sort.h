// Sorting all tables of an index by buckets (index_sort.hip).
#pragma once
#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>

namespace lsh {

// whether tables of N pairs are sorted by buckets; device memory that takes besides the tables
bool bucket_sort_takes(uint64_t N, uint32_t L);
size_t bucket_sort_scratch(uint64_t N, uint32_t L);
// d_keys [N][L] -> d_out_keys, d_out_ids [L][N]: every column's keys ascending, the rows they came from, rows
// ascending within equal keys.  scratch: 16-byte aligned.  Enqueues the launches and returns.
void launch_bucket_sort(const uint64_t *d_keys, uint64_t N, uint32_t L, void *scratch, uint64_t *d_out_keys,
                        uint32_t *d_out_ids, hipStream_t s);

}  // namespace lsh
