// Scratch of calls that allocate their own: device memory, pinned host memory and two events, kept between calls.
//
// Allocating and freeing cost such a call 0.15 to 0.4 ms (hipMalloc 25 to 55 us, hipHostMalloc 20, hipFree 30 to 40, hipHostFree 70 to 230 and more where other memory is mapped), as
// much as three to five components of a transition.  Up to four idle pieces are kept, each of at most 64 MiB of device and 1 MiB of pinned memory; larger ones are freed by the call
// that allocated them.  A piece belongs to one call from take() to give(), and give() comes behind a wait for the stream that used it, so
// calls of several threads, streams and devices never share one.  Idle pieces are given back by release(), and where an allocation fails.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include <mutex>
#include <vector>

struct tsvd_scratch {
    int device = -1;
    size_t bytes = 0, pinned_bytes = 0;
    uint8_t *base = nullptr, *pinned = nullptr;
    hipEvent_t event[2] = {nullptr, nullptr};
};

class tsvd_scratch_pool {
    static constexpr size_t MAX_IDLE = 4, MAX_BYTES = (size_t)64 << 20, MAX_PINNED = (size_t)1 << 20;
    std::mutex m;
    std::vector<tsvd_scratch> idle;

    static void free_piece(tsvd_scratch& s) {
        for (hipEvent_t e : s.event)
            if (e) (void)hipEventDestroy(e);
        if (s.pinned) (void)hipHostFree(s.pinned);
        if (s.base) (void)hipFree(s.base);
        s = tsvd_scratch();
    }
    static bool allocate(tsvd_scratch& s) {
        if (hipMalloc(reinterpret_cast<void**>(&s.base), s.bytes) == hipSuccess &&
            hipHostMalloc(reinterpret_cast<void**>(&s.pinned), s.pinned_bytes, hipHostMallocDefault) == hipSuccess &&
            hipEventCreateWithFlags(&s.event[0], hipEventDisableTiming) == hipSuccess && hipEventCreateWithFlags(&s.event[1], hipEventDisableTiming) == hipSuccess)
            return true;
        const tsvd_scratch wanted = s;
        free_piece(s);
        s.device = wanted.device, s.bytes = wanted.bytes, s.pinned_bytes = wanted.pinned_bytes;
        (void)hipGetLastError();
        return false;
    }

public:
    // A piece of at least these sizes on the current device, its memory as the last call left it.
    bool take(size_t bytes, size_t pinned_bytes, tsvd_scratch* s) {
        int device = 0;
        if (hipGetDevice(&device) != hipSuccess) return false;
        {
            std::lock_guard<std::mutex> lock(m);
            size_t best = idle.size();
            for (size_t i = 0; i < idle.size(); ++i)
                if (idle[i].device == device && idle[i].bytes >= bytes && idle[i].pinned_bytes >= pinned_bytes && (best == idle.size() || idle[i].bytes < idle[best].bytes))
                    best = i;
            if (best < idle.size()) {
                *s = idle[best];
                idle.erase(idle.begin() + (ptrdiff_t)best);
                return true;
            }
        }
        // (rounded up, so that calls of nearly the same sizes find each other's)
        s->device = device;
        s->bytes = (bytes + (1 << 20) - 1) >> 20 << 20;
        s->pinned_bytes = (pinned_bytes + (1 << 16) - 1) >> 16 << 16;
        if (allocate(*s)) return true;
        release();
        return allocate(*s);
    }
    // done: nothing enqueued uses the piece any more.
    void give(tsvd_scratch& s, bool done) {
        if (done && s.bytes <= MAX_BYTES && s.pinned_bytes <= MAX_PINNED) {
            std::lock_guard<std::mutex> lock(m);
            if (idle.size() < MAX_IDLE) {
                idle.push_back(s);
                s = tsvd_scratch();
                return;
            }
            // the smallest makes room
            size_t least = 0;
            for (size_t i = 1; i < idle.size(); ++i)
                if (idle[i].bytes < idle[least].bytes) least = i;
            if (idle[least].bytes < s.bytes) std::swap(idle[least], s);
        }
        free_piece(s);
    }
    void release() {
        std::vector<tsvd_scratch> pieces;
        {
            std::lock_guard<std::mutex> lock(m);
            pieces.swap(idle);
        }
        for (tsvd_scratch& s : pieces) free_piece(s);
    }
};
