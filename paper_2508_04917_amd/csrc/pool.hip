// Device memory of the handles.  hipMalloc and hipFree of a handle's buffers
// (4 GB for 128^3 3x3 blocks) cost more than the setup kernels: freed pages
// are cleared by the driver before they can be handed out again, 130 ms per
// setup in a program that builds and destroys one system after another.  A
// destroyed handle's buffers therefore stay with the library for the next
// handle, up to a bound (kShare of the device's memory).  What goes back to the
// driver: over the bound the longest unused; what has lain unused for
// kIdle, whenever the library allocates or frees device memory (there
// is no thread that looks while it is not called); everything when an
// allocation of the library's fails and on dd_destroy(NULL), which a program
// calls that wants the memory for others.
//
// A block enters the pool only after the device has been idle since its last
// possible use (dd_ctx::reclaim and the destructor synchronise the device, as
// hipFree does), so it may be handed to any stream and thread.  One mutex
// guards the table; no lock is held across a driver call that can wait for
// work.
#include <algorithm>
#include <chrono>
#include <map>
#include <mutex>
#include <unordered_map>

#include "internal.h"

namespace ddilu {

namespace {

using Clock = std::chrono::steady_clock;
constexpr size_t kShare = 16;  // at most 1/kShare of a device's memory is kept
constexpr std::chrono::seconds kIdle{60};

struct Block {
    void *p;
    Clock::time_point since;
};

struct Device {
    std::multimap<size_t, Block> free;
    size_t held = 0, bound = 0;
    Clock::time_point look = Clock::time_point::max();  // no block is older than kIdle before
};

struct Pool {
    std::mutex mu;
    std::map<int, Device> dev;
    std::unordered_map<void *, std::pair<size_t, int>> size;  // every block the pool handed out or holds
};

Pool &pool() {
    static Pool *p = new Pool;  // never destroyed: handles may outlive static objects
    return *p;
}

size_t rounded(size_t b) {
    const size_t unit = b >= (size_t(1) << 21) ? size_t(1) << 21 : 4096;
    return (b + unit - 1) / unit * unit;
}

void take_out(Pool &P, Device &D, std::multimap<size_t, Block>::iterator it, std::vector<void *> &out) {
    D.held -= it->first;
    out.push_back(it->second.p);
    P.size.erase(it->second.p);
    D.free.erase(it);
}

void take_expired(Pool &P, Device &D, std::vector<void *> &out) {
    const Clock::time_point now = Clock::now();
    if (now <= D.look) return;  // every call of the library passes here many times
    D.look = Clock::time_point::max();
    for (auto it = D.free.begin(); it != D.free.end();) {
        const auto next = std::next(it);
        if (now - it->second.since > kIdle)
            take_out(P, D, it, out);
        else
            D.look = std::min(D.look, it->second.since + kIdle);
        it = next;
    }
}

void give_back(const std::vector<void *> &v) {
    for (void *q : v) (void)hipFree(q);
}

}  // namespace

hipError_t pool_alloc(void **out, size_t bytes) {
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    const size_t need = rounded(bytes);
    std::vector<void *> old;
    void *found = nullptr;
    Pool &P = pool();
    {
        std::lock_guard<std::mutex> lock(P.mu);
        Device &D = P.dev[dev];
        auto it = D.free.lower_bound(need);
        if (it != D.free.end() && it->first - need <= need / 4) {  // a quarter more than asked at most
            found = it->second.p;
            D.held -= it->first;
            D.free.erase(it);
        }
        take_expired(P, D, old);
    }
    give_back(old);
    if (found) {
        *out = found;
        return hipSuccess;
    }
    e = hipMalloc(out, need);
    if (e != hipSuccess) {
        (void)hipGetLastError();
        pool_trim(dev);
        e = hipMalloc(out, need);
        if (e != hipSuccess) {
            (void)hipGetLastError();
            return e;
        }
    }
    std::lock_guard<std::mutex> lock(P.mu);
    P.size[*out] = {need, dev};
    return hipSuccess;
}

void pool_free(void *q) {
    if (!q) return;
    std::vector<void *> out;
    Pool &P = pool();
    {
        std::lock_guard<std::mutex> lock(P.mu);
        const auto s = P.size.find(q);
        if (s == P.size.end()) return;
        Device &D = P.dev[s->second.second];
        if (!D.bound) {
            size_t avail = 0, total = 0;
            if (hipMemGetInfo(&avail, &total) != hipSuccess) total = 0;
            D.bound = std::max<size_t>(total / kShare, 1);
        }
        const Clock::time_point now = Clock::now();
        D.free.insert({s->second.first, Block{q, now}});
        D.held += s->second.first;
        D.look = std::min(D.look, now + kIdle);
        take_expired(P, D, out);
        // over the bound the longest unused go: the largest first would give
        // back what was just freed whenever the pool is full of smaller blocks
        while (D.held > D.bound && !D.free.empty())
            take_out(P, D,
                     std::min_element(D.free.begin(), D.free.end(),
                                      [](const auto &a, const auto &b) { return a.second.since < b.second.since; }),
                     out);
    }
    give_back(out);
}

void pool_trim(int device) {
    std::vector<void *> out;
    Pool &P = pool();
    {
        std::lock_guard<std::mutex> lock(P.mu);
        for (auto &d : P.dev) {
            if (device >= 0 && d.first != device) continue;
            while (!d.second.free.empty()) take_out(P, d.second, d.second.free.begin(), out);
        }
    }
    give_back(out);
}

}  // namespace ddilu

void dd_ctx::retire(void *q) {
    if (!q) return;
    auto it = std::find(allocs.begin(), allocs.end(), q);
    if (it == allocs.end()) return;
    allocs.erase(it);
    retired.push_back(q);
}

// Work that may still read the retired buffers, on any stream of the handle's
// device, ends first.
void dd_ctx::reclaim() {
    if (retired.empty()) return;
    int dev = device;
    if (hipGetDevice(&dev) != hipSuccess) return;
    const bool other = device >= 0 && device != dev;
    if (other && hipSetDevice(device) != hipSuccess) return;
    const hipError_t e = hipDeviceSynchronize();
    if (other) (void)hipSetDevice(dev);
    if (e != hipSuccess) return;  // kept for the destructor
    for (void *q : retired) ddilu::pool_free(q);
    retired.clear();
}

hipError_t dd_ctx::try_alloc(void **p, size_t bytes) {
    if (device < 0) (void)hipGetDevice(&device);
    hipError_t e = ddilu::pool_alloc(p, bytes);
    if (e != hipSuccess && !retired.empty()) {
        reclaim();
        e = ddilu::pool_alloc(p, bytes);
    }
    if (e == hipSuccess) allocs.push_back(*p);
    return e;
}

int dd_ctx::alloc_bytes(void **p, size_t bytes) {
    const hipError_t e = try_alloc(p, bytes);
    if (e != hipSuccess) return fail(DD_ENOMEM, "hipMalloc of %zu bytes failed: %s", bytes, hipGetErrorString(e));
    return DD_OK;
}

dd_ctx::~dd_ctx() {
    for (hipEvent_t e : events) (void)hipEventDestroy(e);
    for (hipEvent_t e : tsolve)
        if (e) (void)hipEventDestroy(e);
    retired.insert(retired.end(), allocs.begin(), allocs.end());
    allocs.clear();
    reclaim();
    for (void *q : retired) (void)hipFree(q);  // the device is in error: leave nothing in the pool
    if (ks_host) (void)hipHostFree(ks_host);
}
