// See index_memory.h.
#include "index_memory.h"

#include <cstdint>
#include <map>
#include <mutex>
#include <vector>

namespace lsh {
namespace {

struct Idle {
    IndexBlock block;
    hipEvent_t last_use;  // null: nothing uses the block
};

struct DeviceMemory {
    uint64_t live = 0;
    size_t idle_bytes = 0;
    size_t scratch_bytes = 0;  // scratch in use: it comes back to the idle blocks
    std::vector<Idle> idle;  // oldest first
};

std::mutex mu;
std::map<int, DeviceMemory> memory;

void release(const Idle &i) {
    (void)hipFree(i.block.ptr);  // waits for the device
    if (i.last_use) (void)hipEventDestroy(i.last_use);
}

void forget_scratch(int device, bool scratch, size_t bytes) {
    if (!scratch) return;
    std::lock_guard<std::mutex> lock(mu);
    memory[device].scratch_bytes -= bytes;
}

std::vector<Idle> take_all(DeviceMemory &m) {
    std::vector<Idle> all;
    all.swap(m.idle);
    m.idle_bytes = 0;
    return all;
}

}  // namespace

void index_memory_enter(int device) {
    std::lock_guard<std::mutex> lock(mu);
    ++memory[device].live;
}

void index_memory_leave(int device) {
    std::vector<Idle> all;
    {
        std::lock_guard<std::mutex> lock(mu);
        DeviceMemory &m = memory[device];
        if (--m.live == 0) all = take_all(m);
    }
    for (const Idle &i : all) release(i);
}

bool index_memory_take(int device, size_t bytes, bool scratch, hipStream_t stream, IndexBlock &out) {
    bytes = (bytes + 65535) / 65536 * 65536;
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
    {
        std::lock_guard<std::mutex> lock(mu);
        DeviceMemory &m = memory[device];
        size_t best = m.idle.size();
        for (size_t i = 0; i < m.idle.size(); ++i) {
            const size_t have = m.idle[i].block.bytes;
            if (have < bytes || have / 2 > bytes) continue;  // not more than twice what is asked for
            if (best == m.idle.size() || have < m.idle[best].block.bytes) best = i;
        }
        if (best != m.idle.size()) {
            found = m.idle[best];
            m.idle.erase(m.idle.begin() + best);
            m.idle_bytes -= found.block.bytes;
            if (scratch) m.scratch_bytes += found.block.bytes;
        } else if (scratch && m.idle_bytes + m.scratch_bytes + bytes > kIdleLimit) {
            out.stream_ordered = true;
        } else if (scratch) {
            m.scratch_bytes += bytes;
        }
    }
    if (found.block.ptr) {
        if (found.last_use) {  // the work that used it last, on whatever stream, comes first
            const bool ok = hipStreamWaitEvent(stream, found.last_use, 0) == hipSuccess ||
                            hipEventSynchronize(found.last_use) == hipSuccess;
            (void)hipEventDestroy(found.last_use);
            if (!ok) {
                (void)hipFree(found.block.ptr);
                forget_scratch(device, scratch, found.block.bytes);
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
    std::vector<Idle> all;
    {
        std::lock_guard<std::mutex> lock(mu);
        all = take_all(memory[device]);
    }
    for (const Idle &i : all) release(i);
    if (allocate()) return true;
    (void)hipGetLastError();
    forget_scratch(device, scratch && !out.stream_ordered, bytes);
    out = IndexBlock();
    return false;
}

void index_memory_give_scratch(int device, const IndexBlock &block, hipStream_t stream) {
    if (!block.ptr) return;
    if (block.stream_ordered) {
        (void)hipFreeAsync(block.ptr, stream);
        return;
    }
    hipEvent_t ev = nullptr;
    if (hipEventCreateWithFlags(&ev, hipEventDisableTiming) != hipSuccess || hipEventRecord(ev, stream) != hipSuccess) {
        if (ev) (void)hipEventDestroy(ev);
        (void)hipGetLastError();
        (void)hipFree(block.ptr);  // waits for the device
        forget_scratch(device, true, block.bytes);
        return;
    }
    std::lock_guard<std::mutex> lock(mu);
    DeviceMemory &m = memory[device];
    m.scratch_bytes -= block.bytes;
    m.idle.push_back({block, ev});
    m.idle_bytes += block.bytes;
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
    std::vector<Idle> over;
    {
        std::lock_guard<std::mutex> lock(mu);
        DeviceMemory &m = memory[device];
        m.idle.push_back({block, nullptr});
        m.idle_bytes += block.bytes;
        while (!m.idle.empty() && m.idle_bytes + m.scratch_bytes > kIdleLimit) {
            over.push_back(m.idle.front());
            m.idle_bytes -= m.idle.front().block.bytes;
            m.idle.erase(m.idle.begin());
        }
    }
    for (const Idle &i : over) release(i);
}

}  // namespace lsh
