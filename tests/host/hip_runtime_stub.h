// A stand-in for the parts of the HIP runtime that index_memory.cpp calls, for tests of its book-keeping on
// the CPU: pointers are made up, nothing is allocated, and every call is counted.
#pragma once
#include <cstddef>
#include <cstdint>
#include <map>
#include <mutex>

enum hipError_t { hipSuccess = 0, hipErrorOutOfMemory = 2 };
enum hipStreamCaptureStatus { hipStreamCaptureStatusNone = 0, hipStreamCaptureStatusActive = 1 };
typedef struct stub_stream *hipStream_t;
typedef struct stub_event *hipEvent_t;
constexpr unsigned hipEventDisableTiming = 2;

struct Stub {
    std::mutex mu;
    std::map<uintptr_t, size_t> blocks;  // allocated, by address
    std::map<uintptr_t, bool> async;
    uintptr_t next = 1 << 20;
    size_t bytes = 0, most = SIZE_MAX;  // allocated now, and at most
    int mallocs = 0, frees = 0, events = 0, wrong = 0;

    hipError_t take(void **p, size_t n, bool ordered) {
        std::lock_guard<std::mutex> lock(mu);
        if (n > most || bytes > most - n) return hipErrorOutOfMemory;
        *p = reinterpret_cast<void *>(next);
        blocks[next] = n;
        async[next] = ordered;
        next += n + 4096;
        bytes += n;
        ++mallocs;
        return hipSuccess;
    }
    hipError_t give(void *p, bool ordered) {
        std::lock_guard<std::mutex> lock(mu);
        auto it = blocks.find(reinterpret_cast<uintptr_t>(p));
        if (it == blocks.end() || async[it->first] != ordered) {
            ++wrong;
            return hipErrorOutOfMemory;
        }
        bytes -= it->second;
        blocks.erase(it);
        ++frees;
        return hipSuccess;
    }
};
inline Stub stub;

inline hipError_t hipMalloc(void **p, size_t n) { return stub.take(p, n, false); }
inline hipError_t hipFree(void *p) { return stub.give(p, false); }
inline hipError_t hipMallocAsync(void **p, size_t n, hipStream_t) { return stub.take(p, n, true); }
inline hipError_t hipFreeAsync(void *p, hipStream_t) { return stub.give(p, true); }
inline hipError_t hipGetLastError() { return hipSuccess; }
inline hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus *s) { *s = hipStreamCaptureStatusNone; return hipSuccess; }
inline hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
inline hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
inline hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
inline hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) {
    std::lock_guard<std::mutex> lock(stub.mu);
    *e = reinterpret_cast<hipEvent_t>(uintptr_t(0x100) + (uintptr_t)++stub.events);
    return hipSuccess;
}
inline hipError_t hipEventDestroy(hipEvent_t) {
    std::lock_guard<std::mutex> lock(stub.mu);
    --stub.events;
    return hipSuccess;
}
