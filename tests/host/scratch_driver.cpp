// Host-only driver for the pool of idle scratch (tsvd_scratch.h), built with -fsanitize=address,undefined by tests/test_host_sanitizers.py: the HIP calls that the pool
// makes are those below, which count, and fail on request.  Exit status 0 = all checks passed and no sanitizer report.
#include <cstdio>
#include <cstdlib>
#include <map>
#include <new>

static bool heap_is_full = false;
void* operator new(size_t n) {
    if (heap_is_full) throw std::bad_alloc();
    return std::malloc(n);
}
void operator delete(void* p) noexcept { std::free(p); }
void operator delete(void* p, size_t) noexcept { std::free(p); }

#include "../../paper_2308_07641_amd/csrc/tsvd_scratch.h"

#define CHECK(c) do { if (!(c)) { std::fprintf(stderr, "check failed at line %d: %s\n", __LINE__, #c); return 1; } } while (0)

// The device: `limit` bytes of memory, and host memory and events without end.  (Sizes in front of what is handed out; no container, the heap may be full.)
static size_t used = 0, limit = (size_t)-1, pinned_used = 0;
static int events = 0, device_now = 0, mallocs = 0, frees = 0;
static hipError_t refuse = hipSuccess;
static void* handed_out(size_t n, size_t* sum) {
    size_t* p = static_cast<size_t*>(std::malloc(2 * sizeof(size_t)));       // (the memory itself is never touched)
    p[0] = n;
    *sum += n;
    return p;
}
static hipError_t take_back(void* p, size_t* sum) {
    *sum -= static_cast<size_t*>(p)[0];
    std::free(p);
    return hipSuccess;
}
extern "C" {
hipError_t hipMalloc(void** p, size_t n) {
    ++mallocs;
    if (refuse != hipSuccess) return refuse;
    if (used + n > limit) return hipErrorOutOfMemory;
    *p = handed_out(n, &used);
    return hipSuccess;
}
hipError_t hipFree(void* p) {
    ++frees;
    return refuse != hipSuccess ? refuse : take_back(p, &used);
}
hipError_t hipHostMalloc(void** p, size_t n, unsigned) {
    *p = handed_out(n, &pinned_used);
    return hipSuccess;
}
hipError_t hipHostFree(void* p) { return take_back(p, &pinned_used); }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) {
    *e = reinterpret_cast<hipEvent_t>((size_t)++events);
    return hipSuccess;
}
hipError_t hipEventDestroy(hipEvent_t) {
    --events;
    return hipSuccess;
}
hipError_t hipGetDevice(int* d) {
    *d = device_now;
    return hipSuccess;
}
hipError_t hipGetLastError() { return hipSuccess; }
}

static const size_t MiB = (size_t)1 << 20;

static int keeps_and_gives_back() {
    tsvd_scratch_pool pool;
    tsvd_scratch s[6];
    CHECK(pool.take(3 * MiB - 5, 1000, &s[0]) && s[0].bytes == 3 * MiB && s[0].pinned_bytes == 65536 && s[0].device == 0);
    uint8_t* const at = s[0].base;
    pool.give(s[0], true);
    CHECK(s[0].base == nullptr && used == 3 * MiB);
    CHECK(pool.take(2 * MiB, 65536, &s[0]) && s[0].base == at);              // a smaller call finds it
    CHECK(pool.take(2 * MiB, 65536, &s[1]) && s[1].base != at);              // and it is nobody else's meanwhile
    pool.give(s[1], true);
    pool.give(s[0], true);
    CHECK(pool.take(1 * MiB, 1, &s[0]) && s[0].bytes == 2 * MiB);            // the smallest that fits
    device_now = 1;
    CHECK(pool.take(1 * MiB, 1, &s[1]) && s[1].device == 1 && s[1].bytes == 1 * MiB);        // and of this device only
    device_now = 0;
    pool.give(s[0], false);                                                  // (work of it may be running: not for others)
    CHECK(used == 4 * MiB);
    pool.give(s[1], true);
    for (int i = 0; i < 6; ++i) CHECK(pool.take(4 * MiB, 1, &s[i]));
    for (int i = 0; i < 6; ++i) pool.give(s[i], true);
    CHECK(used == 16 * MiB && events == 8);                                  // four at most
    CHECK(pool.take(65 * MiB, 1, &s[0]));
    pool.give(s[0], true);
    CHECK(used == 16 * MiB);                                                 // none above 64 MiB
    for (int i = 0; i < 3; ++i) CHECK(pool.take((size_t)(20 + 10 * i) * MiB, 1, &s[i]));
    for (int i = 0; i < 3; ++i) pool.give(s[i], true);
    CHECK(used == 40 * MiB);                                                 // nor more than that in all: the last one
    CHECK(pool.take(30 * MiB, 1, &s[0]) && s[0].bytes == 40 * MiB);
    pool.give(s[0], true);
    CHECK(pool.take(MiB, 2 * MiB, &s[0]));
    pool.give(s[0], true);
    CHECK(pinned_used <= 4 * MiB);
    pool.release();
    CHECK(used == 0 && pinned_used == 0 && events == 0);
    return 0;
}

// C entries reach the pool: it may not throw, nor lose memory, where the heap has none.
static int works_without_heap() {
    heap_is_full = true;
    tsvd_scratch s[5];
    tsvd_scratch_pool pool;
    for (auto& p : s)
        if (!pool.take(MiB, 1, &p)) return 1;
    for (auto& p : s) pool.give(p, true);
    pool.release();
    heap_is_full = false;
    CHECK(used == 0 && pinned_used == 0 && events == 0);
    return 0;
}

// Idle scratch is no reason for an allocation of the library to fail; other errors than a full device are handed on, and nothing is freed for them.
static int is_no_reason_to_fail() {
    tsvd_scratch_pool& pool = tsvd_idle_scratch();
    tsvd_scratch s;
    void* p = nullptr;
    limit = 100 * MiB;
    CHECK(pool.take(60 * MiB, 1, &s));
    pool.give(s, true);
    CHECK(used == 60 * MiB);
    CHECK(tsvd_device_malloc(&p, 70 * MiB) == hipSuccess && used == 70 * MiB);
    CHECK(hipFree(p) == hipSuccess);
    CHECK(pool.take(60 * MiB, 1, &s));
    pool.give(s, true);
    tsvd_scratch t;
    CHECK(pool.take(80 * MiB, 1, &t) && used == 80 * MiB);                   // nor for one of its own
    pool.give(t, true);
    CHECK(used == 0);
    CHECK(pool.take(60 * MiB, 1, &s));
    pool.give(s, true);
    CHECK(tsvd_device_malloc(&p, 101 * MiB) == hipErrorOutOfMemory && used == 0);
    CHECK(pool.take(60 * MiB, 1, &s));
    pool.give(s, true);
    refuse = hipErrorStreamCaptureUnsupported;
    frees = mallocs = 0;
    CHECK(tsvd_device_malloc(&p, MiB) == refuse && mallocs == 1 && frees == 0);
    CHECK(!pool.take(80 * MiB, 1, &t) && mallocs == 2 && frees == 0);
    refuse = hipSuccess;
    limit = (size_t)-1;
    pool.release();
    CHECK(used == 0 && pinned_used == 0 && events == 0);
    return 0;
}

int main() {
    if (keeps_and_gives_back() || works_without_heap() || is_no_reason_to_fail()) return 1;
    std::printf("scratch driver: ok\n");
    return 0;
}
