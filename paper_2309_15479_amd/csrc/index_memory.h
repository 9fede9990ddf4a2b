// Device memory of the index: the tables of live indexes and the scratch of builds.
#pragma once
#include <hip/hip_runtime.h>

#include <cstddef>

namespace lsh {

// hipMalloc and hipFree map and unmap memory and wait for the device, and the default
// stream-ordered pool gives its memory back at every synchronisation: on the SIFT shape (384 MB of
// tables, 390 MB of scratch, 2.4 ms of kernels) that is 0.7 ms each time an index is built and destroyed alone, and
// was 1 to 17 ms where a program rebuilds one while the old one stands, by what else it holds.  Blocks are therefore kept and handed out again while any index is alive on their
// device, up to kIdleLimit idle bytes; the destruction of the last one gives all of them back.
// All functions are safe to call from several threads.
constexpr size_t kIdleLimit = size_t(2) << 30;

struct IndexBlock {
    void *ptr = nullptr;
    size_t bytes = 0;
    bool stream_ordered = false;  // from hipMallocAsync: scratch that would not fit the limit
};

// one more / one fewer index on the device; the last leave() frees the idle blocks
void index_memory_enter(int device);
void index_memory_leave(int device);
// a block of at least `bytes` on the current device, for work enqueued on `stream` from here on; scratch: it is
// handed back with index_memory_give_scratch on the same stream.  false: out of memory
bool index_memory_take(int device, size_t bytes, bool scratch, hipStream_t stream, IndexBlock &out);
// work on `stream` enqueued so far may still use the block; does not wait
void index_memory_give_scratch(int device, const IndexBlock &block, hipStream_t stream);
// waits until all work enqueued on the current device is done; false: it could not be waited for
bool index_memory_wait();
// nothing on the device uses the block any more
void index_memory_give(int device, const IndexBlock &block);

}  // namespace lsh
