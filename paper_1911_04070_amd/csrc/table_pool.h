// Device memory for the small tables of batch graphs on one tree (lengths, row deltas, roots), kept by the tree from one
// graph to the next: a training loop makes and destroys a graph per step, and a hipFree or a copy on the caller's stream
// would wait for the whole step before it.
//
// A block is handed out again when the work that read it is through.  Every call on a batch graph records an event of its
// own behind its last kernel, on its stream, and the block waits for all of them: a stream handle does not say which
// event a later one stands for (hipStreamPerThread is one queue per host thread, and a handle can come back after its stream
// has been destroyed).  A block with more than kTableUses calls, or one used inside a stream capture, which can be
// replayed at any time, is not handed out again but freed with its graph.  At most kTableBlocks blocks a tree are kept;
// they go with it and the graphs on it.
//
// Host code; needs nothing but the HIP runtime's API.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <mutex>
#include <new>
#include <vector>

namespace bpt {

constexpr int kTableBlocks = 8;
constexpr size_t kTableUses = 256;   // (a graph made per step sees a forward and a backward of every layer)

struct TableBlock {
    int32_t* p = nullptr;
    size_t capacity = 0;               // int32s
    bool unknown = false;              // used where no event says when: not handed out again
    std::vector<hipEvent_t> events;    // the first `uses` have been recorded since the block was handed out
    size_t uses = 0;
};

struct TablePool {
    std::mutex m;   // (never held while something is waited for: calls of other threads note their uses under it)
    hipStream_t copies = nullptr;
    std::vector<TableBlock*> free;   // destroyed graphs' blocks, oldest first
    int blocks = 0;                  // these and the ones in use

    TablePool() { free.reserve(kTableBlocks); }
    TablePool(const TablePool&) = delete;
    TablePool& operator=(const TablePool&) = delete;
    ~TablePool() {
        for (TableBlock* b : free) destroy(b);
        if (copies) (void)hipStreamDestroy(copies);
    }

    // A block of the tree's with the values h in it, in place when this returns.  *out may be set on an error as well: the
    // graph's destruction gives it back.
    hipError_t acquire(const std::vector<int32_t>& h, TableBlock** out) {
        TableBlock *b = nullptr, *small = nullptr;
        bool wait = false;
        {
            std::lock_guard<std::mutex> lock(m);
            if (!copies) {
                const hipError_t e = hipStreamCreateWithFlags(&copies, hipStreamNonBlocking);
                if (e != hipSuccess) return e;
            }
            // the first that is large enough and idle; with all blocks there are in use, the oldest, when it is
            for (int pass = 0; pass < 2 && !b; ++pass) {
                if (pass == 1 && blocks < kTableBlocks) break;
                for (size_t i = 0; i < free.size() && !b; ++i)
                    if (free[i]->capacity >= h.size() && (pass == 1 || idle(*free[i], false))) b = take(i);
                wait = b && pass == 1;
            }
            if (!b && blocks >= kTableBlocks && !free.empty()) {   // none is large enough: one makes way
                small = take(0);
                --blocks;
            }
        }
        if (small) destroy(small);
        if (wait && !idle(*b, true)) {   // (an event that cannot be waited for: the block is not used again)
            {
                std::lock_guard<std::mutex> lock(m);
                --blocks;
            }
            destroy(b);
            b = nullptr;
        }
        if (b) {
            b->uses = 0;
        } else {
            b = new TableBlock();
            b->capacity = 1024;
            while (b->capacity < h.size()) b->capacity *= 2;
            const hipError_t e = hipMalloc((void**)&b->p, b->capacity * sizeof(int32_t));
            if (e != hipSuccess) {
                delete b;
                return e;
            }
            std::lock_guard<std::mutex> lock(m);
            ++blocks;
        }
        *out = b;
        const hipError_t e = hipMemcpyAsync(b->p, h.data(), h.size() * sizeof(int32_t), hipMemcpyHostToDevice, copies);
        return e != hipSuccess ? e : hipStreamSynchronize(copies);
    }

    // the graph that held the block is gone
    void release(TableBlock* b) {
        {
            std::lock_guard<std::mutex> lock(m);
            if (!b->unknown && blocks <= kTableBlocks) {
                free.push_back(b);
                return;
            }
            --blocks;
        }
        destroy(b);
    }

    // a call has put its kernels, which read the block, on `st`
    void note(TableBlock& b, hipStream_t st) {
        std::lock_guard<std::mutex> lock(m);
        if (b.unknown) return;
        hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
        const bool known = hipStreamIsCapturing(st, &cap) == hipSuccess && cap == hipStreamCaptureStatusNone && b.uses < kTableUses &&
                           (b.uses < b.events.size() || add_event(b)) && hipEventRecord(b.events[b.uses], st) == hipSuccess;
        if (known) {
            ++b.uses;
        } else {
            (void)hipGetLastError();
            b.unknown = true;
        }
    }

private:
    static bool add_event(TableBlock& b) {
        hipEvent_t ev = nullptr;
        if (hipEventCreateWithFlags(&ev, hipEventDisableTiming) != hipSuccess) return false;
        try {
            b.events.push_back(ev);
        } catch (const std::bad_alloc&) {
            (void)hipEventDestroy(ev);
            return false;
        }
        return true;
    }
    // whether the work that read the block is through (wait: until it is)
    static bool idle(const TableBlock& b, bool wait) {
        for (size_t i = b.uses; i-- > 0;) {   // the last call first: where any is not through, it is the likeliest
            const hipError_t e = wait ? hipEventSynchronize(b.events[i]) : hipEventQuery(b.events[i]);
            if (e != hipSuccess) {
                (void)hipGetLastError();   // (not ready)
                return false;
            }
        }
        return true;
    }
    TableBlock* take(size_t i) {
        TableBlock* b = free[i];
        free.erase(free.begin() + i);
        return b;
    }
    static void destroy(TableBlock* b) {
        for (hipEvent_t ev : b->events) (void)hipEventDestroy(ev);
        (void)hipFree(b->p);   // (waits for the device)
        delete b;
    }
};

}  // namespace bpt
