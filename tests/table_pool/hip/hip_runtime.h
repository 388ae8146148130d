// The few calls of the HIP runtime that table_pool.h makes, on queues whose progress the test decides.
#pragma once
#include <stddef.h>
#include <stdlib.h>
#include <string.h>

#include <map>
#include <memory>
#include <set>

enum hipError_t { hipSuccess, hipErrorOutOfMemory, hipErrorNotReady, hipErrorUnknown };
enum hipMemcpyKind { hipMemcpyHostToDevice };
enum hipStreamCaptureStatus { hipStreamCaptureStatusNone, hipStreamCaptureStatusActive };
constexpr unsigned hipStreamNonBlocking = 1, hipEventDisableTiming = 2;

struct Queue {
    long put = 0, done = 0;   // operations queued and finished
    bool capturing = false;
};
struct Event {
    std::shared_ptr<Queue> queue;
    long at = 0;
};
typedef struct Handle* hipStream_t;   // (a handle: the queue that it names may change)
inline hipStream_t stream(long i) { return reinterpret_cast<hipStream_t>(i); }
typedef Event* hipEvent_t;

inline std::map<hipStream_t, std::shared_ptr<Queue>> g_queue;
inline std::set<void*> g_memory;
inline int g_waits = 0;                   // calls that waited for work
inline void (*g_on_wait)() = nullptr;     // ... tell the test
inline bool g_no_events = false;

inline Queue& queue_of(hipStream_t s) {
    auto& q = g_queue[s];
    if (!q) q = std::make_shared<Queue>();
    return *q;
}
inline void waited() {
    ++g_waits;
    if (g_on_wait) g_on_wait();
}
inline hipError_t hipGetLastError() { return hipSuccess; }
inline hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) {
    *s = stream(1000);
    return hipSuccess;
}
inline hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
inline hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
inline hipError_t hipStreamIsCapturing(hipStream_t s, hipStreamCaptureStatus* st) {
    *st = queue_of(s).capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
    return hipSuccess;
}
inline hipError_t hipMalloc(void** p, size_t bytes) {
    *p = malloc(bytes);
    g_memory.insert(*p);
    return hipSuccess;
}
inline hipError_t hipFree(void* p) {
    waited();
    g_memory.erase(p);
    free(p);
    return hipSuccess;
}
inline hipError_t hipMemcpyAsync(void* d, const void* s, size_t bytes, hipMemcpyKind, hipStream_t) {
    memcpy(d, s, bytes);
    return hipSuccess;
}
inline hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) {
    if (g_no_events) return hipErrorUnknown;
    *e = new Event();
    return hipSuccess;
}
inline hipError_t hipEventDestroy(hipEvent_t e) {
    delete e;
    return hipSuccess;
}
inline hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) {
    queue_of(s);
    e->queue = g_queue[s];
    e->at = e->queue->put;
    return hipSuccess;
}
inline hipError_t hipEventQuery(hipEvent_t e) { return e->queue->done >= e->at ? hipSuccess : hipErrorNotReady; }
inline hipError_t hipEventSynchronize(hipEvent_t e) {
    waited();
    if (e->queue->done < e->at) e->queue->done = e->at;
    return hipSuccess;
}
