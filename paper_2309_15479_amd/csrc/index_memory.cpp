// See index_memory.h.
#include "index_memory.h"

#include <cstdint>
#include <mutex>

namespace lsh {
namespace {

struct Idle {
    IndexBlock block;
    hipEvent_t last_use;  // null: nothing uses the block
};

// Fixed arrays: nothing here may throw (the callers are C entries), or be destroyed while an index that a program
// holds to its end still needs it.
constexpr int kDevices = 64;     // on others nothing is kept
constexpr uint32_t kIdle = 256;  // blocks kept at most

struct DeviceMemory {
    uint64_t live = 0;
    size_t idle_bytes = 0;
    size_t scratch_bytes = 0;  // scratch in use: it comes back to the idle blocks
    uint32_t idle_count = 0;
    Idle idle[kIdle] = {};  // oldest first

    Idle remove(uint32_t i) {
        const Idle out = idle[i];
        for (--idle_count; i < idle_count; ++i) idle[i] = idle[i + 1];
        idle_bytes -= out.block.bytes;
        return out;
    }
    // returns the oldest block if there is no room for one more
    Idle add(const Idle &i) {
        const Idle out = idle_count == kIdle ? remove(0) : Idle{};
        idle[idle_count++] = i;
        idle_bytes += i.block.bytes;
        return out;
    }
};

std::mutex mu;
DeviceMemory memory[kDevices];

DeviceMemory *kept(int device) { return device >= 0 && device < kDevices ? &memory[device] : nullptr; }

void release(const Idle &i) {
    if (!i.block.ptr) return;
    (void)hipFree(i.block.ptr);  // waits for the device
    if (i.last_use) (void)hipEventDestroy(i.last_use);
}

// idle blocks, oldest first, until the rest satisfies `enough`
template <typename Enough>
void release_until(DeviceMemory &m, Enough enough) {
    for (;;) {
        Idle i;
        {
            std::lock_guard<std::mutex> lock(mu);
            if (!m.idle_count || enough()) return;
            i = m.remove(0);
        }
        release(i);
    }
}

void forget_scratch(DeviceMemory *m, bool scratch, size_t bytes) {
    if (!m || !scratch) return;
    std::lock_guard<std::mutex> lock(mu);
    m->scratch_bytes -= bytes;
}

}  // namespace

void index_memory_enter(int device) {
    DeviceMemory *m = kept(device);
    if (!m) return;
    std::lock_guard<std::mutex> lock(mu);
    ++m->live;
}

void index_memory_leave(int device) {
    DeviceMemory *m = kept(device);
    if (!m) return;
    {
        std::lock_guard<std::mutex> lock(mu);
        --m->live;
    }
    release_until(*m, [&] { return m->live != 0; });
}

bool index_memory_take(int device, size_t bytes, bool scratch, hipStream_t stream, IndexBlock &out) {
    bytes = (bytes + 65535) / 65536 * 65536;
    DeviceMemory *const m = kept(device);
    Idle found = {};
    hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(stream, &capture) != hipSuccess || capture != hipStreamCaptureStatusNone) {
        // work recorded now runs when its graph does, later and any number of times: it gets no
        // block that others use in between, and what the runtime refuses to a capture is refused
        out.stream_ordered = scratch;
        out.bytes = bytes;
        if ((scratch ? hipMallocAsync(&out.ptr, bytes, stream) : hipMalloc(&out.ptr, bytes)) == hipSuccess) return true;
        (void)hipGetLastError();
        out = IndexBlock();
        return false;
    }
    if (m) {
        std::lock_guard<std::mutex> lock(mu);
        uint32_t best = kIdle;
        for (uint32_t i = 0; i < m->idle_count; ++i) {
            const size_t have = m->idle[i].block.bytes;
            // scratch, back after the build, takes up to twice what is asked for; tables stay as long as their index
            if (have < bytes || have - bytes > (scratch ? bytes : bytes / 8)) continue;
            if (best == kIdle || have < m->idle[best].block.bytes) best = i;
        }
        if (best != kIdle) {
            found = m->remove(best);
            if (scratch) m->scratch_bytes += found.block.bytes;
        } else if (scratch && m->idle_bytes + m->scratch_bytes + bytes > kIdleLimit) {
            out.stream_ordered = true;
        } else if (scratch) {
            m->scratch_bytes += bytes;
        }
    } else {
        out.stream_ordered = scratch;
    }
    if (found.block.ptr) {
        if (found.last_use) {  // the work that used it last, on whatever stream, comes first
            const bool ok = hipStreamWaitEvent(stream, found.last_use, 0) == hipSuccess ||
                            hipEventSynchronize(found.last_use) == hipSuccess;
            (void)hipEventDestroy(found.last_use);
            if (!ok) {
                (void)hipFree(found.block.ptr);
                forget_scratch(m, scratch, found.block.bytes);
                return false;
            }
        }
        out = found.block;
        return true;
    }
    out.bytes = bytes;
    auto allocate = [&] {
        return (out.stream_ordered ? hipMallocAsync(&out.ptr, bytes, stream) : hipMalloc(&out.ptr, bytes)) == hipSuccess;
    };
    if (allocate()) return true;
    (void)hipGetLastError();
    if (m) release_until(*m, [] { return false; });
    if (allocate()) return true;
    (void)hipGetLastError();
    forget_scratch(m, scratch && !out.stream_ordered, bytes);
    out = IndexBlock();
    return false;
}

void index_memory_give_scratch(int device, const IndexBlock &block, hipStream_t stream) {
    if (!block.ptr) return;
    if (block.stream_ordered) {
        (void)hipFreeAsync(block.ptr, stream);
        return;
    }
    DeviceMemory *const m = kept(device);  // not null: scratch of other devices is stream-ordered
    hipEvent_t ev = nullptr;
    if (hipEventCreateWithFlags(&ev, hipEventDisableTiming) != hipSuccess || hipEventRecord(ev, stream) != hipSuccess) {
        if (ev) (void)hipEventDestroy(ev);
        (void)hipGetLastError();
        (void)hipFree(block.ptr);  // waits for the device
        forget_scratch(m, true, block.bytes);
        return;
    }
    Idle out;
    {
        std::lock_guard<std::mutex> lock(mu);
        m->scratch_bytes -= block.bytes;
        out = m->add({block, ev});
    }
    release(out);
}

bool index_memory_wait() {
    // hipFree waits for all work on the device and may be called while a stream captures in relaxed mode, or in
    // another thread; hipDeviceSynchronize would invalidate the capture
    void *token = nullptr;
    const bool ok = hipMalloc(&token, 4) == hipSuccess && hipFree(token) == hipSuccess;
    if (!ok) (void)hipGetLastError();
    return ok;
}

void index_memory_give(int device, const IndexBlock &block) {
    if (!block.ptr) return;
    DeviceMemory *const m = kept(device);
    if (!m || block.bytes > kIdleLimit) {
        (void)hipFree(block.ptr);
        return;
    }
    Idle out;
    {
        std::lock_guard<std::mutex> lock(mu);
        out = m->add({block, nullptr});
    }
    release(out);
    release_until(*m, [&] { return m->idle_bytes + m->scratch_bytes <= kIdleLimit; });
}

}  // namespace lsh
