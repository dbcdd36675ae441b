// Scratch of calls that allocate their own: device memory, pinned host memory and two events, kept between calls.
//
// Allocating and freeing cost such a call 0.15 to 0.4 ms (hipMalloc 25 to 55 us, hipHostMalloc 20, hipFree 30 to 40, hipHostFree 70 to 230 and more where other memory is mapped), as
// much as three to five components of a transition.  Up to four idle pieces of 64 MiB of device memory in all, and 1 MiB of pinned memory each, are kept; where that is not enough for the piece that
// comes back, those that have been idle longest are freed.  A piece belongs to one call from take() to give(), and give() comes behind a wait for the stream that used it, so
// calls of several threads, streams and devices never share one.  Idle pieces are given back by release(), and where the device has no memory left for this library (tsvd_device_malloc);
// other allocators of the process do not know of them.  Nothing here throws.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include <mutex>
#include <new>
#include <utility>

struct tsvd_scratch {
    int device = -1;
    size_t bytes = 0, pinned_bytes = 0;
    uint8_t *base = nullptr, *pinned = nullptr;
    hipEvent_t event[2] = {nullptr, nullptr};
};

class tsvd_scratch_pool {
    static constexpr int MAX_IDLE = 4;
    static constexpr size_t MAX_BYTES = (size_t)64 << 20, MAX_PINNED = (size_t)1 << 20;
    std::mutex m;
    tsvd_scratch idle[MAX_IDLE];                             // the first `count`, longest idle first
    int count = 0;
    size_t idle_bytes = 0;

    static void free_piece(tsvd_scratch& s) {
        for (hipEvent_t e : s.event)
            if (e) (void)hipEventDestroy(e);
        if (s.pinned) (void)hipHostFree(s.pinned);
        if (s.base) (void)hipFree(s.base);
        s = tsvd_scratch();
    }
    static hipError_t allocate(tsvd_scratch& s) {
        hipError_t e = hipMalloc(reinterpret_cast<void**>(&s.base), s.bytes);
        if (e == hipSuccess) e = hipHostMalloc(reinterpret_cast<void**>(&s.pinned), s.pinned_bytes, hipHostMallocDefault);
        for (int k = 0; e == hipSuccess && k < 2; ++k) e = hipEventCreateWithFlags(&s.event[k], hipEventDisableTiming);
        if (e == hipSuccess) return e;
        const tsvd_scratch wanted = s;
        free_piece(s);
        s.device = wanted.device, s.bytes = wanted.bytes, s.pinned_bytes = wanted.pinned_bytes;
        (void)hipGetLastError();
        return e;
    }
    tsvd_scratch remove(int at) {                            // (under the lock)
        const tsvd_scratch s = idle[at];
        for (--count; at < count; ++at) idle[at] = idle[at + 1];
        idle_bytes -= s.bytes;
        return s;
    }

public:
    // A piece of at least these sizes on the current device, its memory as the last call left it.
    bool take(size_t bytes, size_t pinned_bytes, tsvd_scratch* s) {
        int device = 0;
        if (hipGetDevice(&device) != hipSuccess) return false;
        {
            std::lock_guard<std::mutex> lock(m);
            int best = -1;
            for (int i = 0; i < count; ++i)
                if (idle[i].device == device && idle[i].bytes >= bytes && idle[i].pinned_bytes >= pinned_bytes && (best < 0 || idle[i].bytes < idle[best].bytes)) best = i;
            if (best >= 0) {
                *s = remove(best);
                return true;
            }
        }
        // (rounded up, so that calls of nearly the same sizes find each other's)
        s->device = device;
        s->bytes = (bytes + (1 << 20) - 1) >> 20 << 20;
        s->pinned_bytes = (pinned_bytes + (1 << 16) - 1) >> 16 << 16;
        const hipError_t e = allocate(*s);
        if (e != hipErrorOutOfMemory) return e == hipSuccess;
        release();
        return allocate(*s) == hipSuccess;
    }
    // done: nothing enqueued uses the piece any more.
    void give(tsvd_scratch& s, bool done) {
        if (!done || s.bytes > MAX_BYTES || s.pinned_bytes > MAX_PINNED) return free_piece(s);
        tsvd_scratch out[MAX_IDLE];
        int outs = 0;
        {
            std::lock_guard<std::mutex> lock(m);
            while (count == MAX_IDLE || idle_bytes + s.bytes > MAX_BYTES) out[outs++] = remove(0);
            idle[count++] = s;
            idle_bytes += s.bytes;
            s = tsvd_scratch();
        }
        for (int i = 0; i < outs; ++i) free_piece(out[i]);
    }
    void release() {
        tsvd_scratch out[MAX_IDLE];
        int outs = 0;
        {
            std::lock_guard<std::mutex> lock(m);
            while (count > 0) out[outs++] = remove(0);
        }
        for (int i = 0; i < outs; ++i) free_piece(out[i]);
    }
};

// The pool of the process (never destroyed: the runtime may be gone by then, and takes the memory with it).
inline tsvd_scratch_pool& tsvd_idle_scratch() {
    alignas(tsvd_scratch_pool) static unsigned char memory[sizeof(tsvd_scratch_pool)];
    static tsvd_scratch_pool* const pool = new (memory) tsvd_scratch_pool;
    return *pool;
}

// hipMalloc for the library's other memory: idle scratch is no reason to fail.  (Other errors are left alone: under another stream's capture nothing may be freed either.)
inline hipError_t tsvd_device_malloc(void** p, size_t bytes) {
    const hipError_t e = hipMalloc(p, bytes);
    if (e != hipErrorOutOfMemory) return e;
    (void)hipGetLastError();
    tsvd_idle_scratch().release();
    return hipMalloc(p, bytes);
}
