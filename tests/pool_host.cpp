// The memory pool on a host without a GPU: the driver's allocation calls and
// the clock are stood in for here, so that ages and failures can be set.
#include <cassert>
#include <cstdio>
#include <cstdlib>
#include <ctime>
#include <set>

#include "../paper_2508_04917_amd/csrc/pool.hip"

static std::set<void *> live;  // what the driver has handed out
static long now_s = 1000;
static bool fail_malloc = false;

extern "C" int clock_gettime(clockid_t, struct timespec *t) noexcept {
    t->tv_sec = now_s;
    t->tv_nsec = 0;
    return 0;
}

hipError_t hipMalloc(void **p, size_t) {
    if (fail_malloc) return hipErrorOutOfMemory;
    *p = std::malloc(1);
    live.insert(*p);
    return hipSuccess;
}
hipError_t hipFree(void *p) {
    assert(live.erase(p) == 1);
    return hipSuccess;
}
hipError_t hipGetDevice(int *d) {
    *d = 0;
    return hipSuccess;
}
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipDeviceSynchronize() { return hipSuccess; }
hipError_t hipMemGetInfo(size_t *f, size_t *t) {
    *f = *t = size_t(16) << 30;  // the pool's bound is 1 GiB
    return hipSuccess;
}
const char *hipGetErrorString(hipError_t) { return ""; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipHostFree(void *) { return hipSuccess; }
int dd_ctx::fail(int code, const char *, ...) {
    err = "failed";
    return code;
}

static const size_t MB = size_t(1) << 20;

static void *get(size_t b) {
    void *p = nullptr;
    assert(ddilu::pool_alloc(&p, b) == hipSuccess);
    return p;
}

#define CHECK(c)                                             \
    do {                                                     \
        if (!(c)) {                                          \
            std::printf("line %d: %s\n", __LINE__, #c);      \
            return 1;                                        \
        }                                                    \
    } while (0)

int main() {
    // blocks kept, reused, and given back by age at the next allocation
    void *a = get(8 * MB), *b = get(64 * MB);
    ddilu::pool_free(a);
    now_s += 40;
    ddilu::pool_free(b);
    CHECK(live.size() == 2);
    now_s += 40;  // a is 80 s old, b 40 s
    void *c = get(1);
    CHECK(live.count(a) == 0 && live.count(b) == 1 && live.size() == 2);
    // a block that is asked for is used whatever its age; others of that age go
    void *d = get(300 * MB);
    ddilu::pool_free(d);
    now_s += 61;
    CHECK(get(64 * MB) == b);
    CHECK(live.count(d) == 0 && live.size() == 2);
    // and at the next release
    void *e = get(16 * MB);
    ddilu::pool_free(e);
    now_s += 61;
    ddilu::pool_free(c);
    CHECK(live.count(e) == 0 && live.size() == 2);
    // everything goes on request
    ddilu::pool_free(b);
    ddilu::pool_trim(-1);
    CHECK(live.empty());
    // a failing allocation empties the pool
    a = get(8 * MB);
    ddilu::pool_free(a);
    fail_malloc = true;
    CHECK(ddilu::pool_alloc(&c, 64 * MB) == hipErrorOutOfMemory && live.empty());
    // memory that a call can do without leaves no error message behind
    dd_ctx h;
    CHECK(h.try_alloc(&c, 64 * MB) == hipErrorOutOfMemory && h.err.empty());
    CHECK(h.alloc_bytes(&c, 64 * MB) == DD_ENOMEM && !h.err.empty());
    return 0;
}
