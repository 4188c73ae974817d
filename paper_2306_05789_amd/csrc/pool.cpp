// Device scratch reused across assemblies, products and solves.
//
// An assembly's ACA batches need several GB of scratch (the factor columns
// of every block up to its rank cap, and the per-step partial sums) for a
// few hundred milliseconds.  Allocating and freeing that on every assembly
// costs host time, and hipFree waits for the whole device, so an assembly
// freeing its scratch on one thread stalls until the concurrent assembly on
// another stream has drained too.  Scratch that has been given back after its
// stream drained (DevBuf::settled) is kept here per device and handed out
// again; a buffer released without that guarantee (an exception unwinding
// past queued work) is freed with hipFree instead.  The working vectors of a
// product or a solve (3 to 15 buffers a call) come from here too: allocated and
// freed on each call they cost a 16-column product of the 29^3 operator 330 of
// its 1050 us and the 13-column mixed one of 37x22x31 350 of 740.
#include <algorithm>
#include <atomic>
#include <chrono>
#include <map>

#include "rte_internal.h"

namespace rte {

namespace {

struct Idle {
    int device;
    void *p;
    size_t cap;
    uint64_t stamp;
};

struct Pool {
    std::mutex mu;
    std::vector<Idle> idle;
    std::map<int, size_t> bytes;   // idle bytes per device
    std::map<int, size_t> total;   // memory of each device (asked once: a query costs more than a product's launches)
    uint64_t clock = 0;
};

Pool &pool() {
    static Pool *p = new Pool();   // lives until the process ends (buffers stay with the device)
    return *p;
}

thread_local double t_alloc_ms = 0.0;

struct Clock {
    std::chrono::steady_clock::time_point t0 = std::chrono::steady_clock::now();
    ~Clock() {
        t_alloc_ms += std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - t0).count();
    }
};

// Every device allocation of the library goes through these two.  Checking aid:
// RTE_MEMORY_CAP in the environment is the number of bytes that they may hold together;
// an allocation beyond it fails as on a full device.
std::atomic<size_t> g_held{0};

hipError_t device_malloc(void **p, size_t bytes) {
    const size_t held = g_held.fetch_add(bytes) + bytes;
    hipError_t e = hipSuccess;
    if (const char *cap = std::getenv("RTE_MEMORY_CAP"))
        if (held > std::strtoull(cap, nullptr, 10)) e = hipErrorOutOfMemory;
    if (e == hipSuccess) e = hipMalloc(p, bytes);
    if (e != hipSuccess) g_held.fetch_sub(bytes);
    return e;
}

void device_free(void *p, size_t bytes) {
    (void)hipFree(p);
    g_held.fetch_sub(bytes);
}

constexpr size_t kGranule = (size_t)2 << 20, kPage = 4096;
constexpr size_t kIdleMost = 4096;   // buffers (a search of the idle ones stays short)

// keep at most an eighth of the device memory and kIdleMost buffers idle, dropping the least recently given back first
void cap_idle_locked(Pool &P, int dev) {
    size_t &total = P.total[dev];
    if (total == 0) {
        size_t fb = 0;
        if (hipMemGetInfo(&fb, &total) != hipSuccess) {
            (void)hipGetLastError();
            total = 0;
            return;
        }
    }
    while (P.bytes[dev] > total / 8 || P.idle.size() > kIdleMost) {
        if (P.bytes[dev] == 0) return;   // what is idle is another device's
        auto it = std::min_element(P.idle.begin(), P.idle.end(), [&](const Idle &a, const Idle &b) {
            return (a.device == dev ? a.stamp : UINT64_MAX) < (b.device == dev ? b.stamp : UINT64_MAX);
        });
        device_free(it->p, it->cap);
        P.bytes[dev] -= it->cap;
        P.idle.erase(it);
    }
}

}  // namespace

double &alloc_ms_this_thread() { return t_alloc_ms; }

size_t device_bytes_held() { return g_held.load(); }

void *pool_take(size_t bytes, size_t *cap, bool exact) {
    Clock c;
    int dev = 0;
    HIP_CHECK(hipGetDevice(&dev));
    const size_t unit = exact ? kPage : kGranule;
    const size_t want = (bytes + unit - 1) / unit * unit, most = exact ? want : 2 * want;
    Pool &P = pool();
    {
        std::lock_guard<std::mutex> g(P.mu);
        // best fit among the idle buffers of this device that are at most twice as large (exact: no larger)
        auto best = P.idle.end();
        for (auto it = P.idle.begin(); it != P.idle.end(); ++it)
            if (it->device == dev && it->cap >= want && it->cap <= most &&
                (best == P.idle.end() || it->cap < best->cap))
                best = it;
        if (best != P.idle.end()) {
            void *p = best->p;
            *cap = best->cap;
            P.bytes[dev] -= best->cap;
            P.idle.erase(best);
            return p;
        }
    }
    void *p = nullptr;
    hipError_t e = device_malloc(&p, want);
    if (e == hipErrorOutOfMemory) {
        (void)hipGetLastError();
        pool_trim();
        e = device_malloc(&p, want);
    }
    if (e != hipSuccess)
        throw Error(e == hipErrorOutOfMemory ? RTE_E_OUT_OF_MEMORY : RTE_E_DEVICE,
                    std::string("hipMalloc (scratch): ") + hipGetErrorString(e));
    *cap = want;
    return p;
}

void pool_give(void *p, size_t cap) {
    Clock c;
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) {
        (void)hipGetLastError();
        device_free(p, cap);
        return;
    }
    Pool &P = pool();
    std::lock_guard<std::mutex> g(P.mu);
    P.idle.push_back({dev, p, cap, ++P.clock});
    P.bytes[dev] += cap;
    cap_idle_locked(P, dev);
}

size_t pool_idle_bytes() {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) {
        (void)hipGetLastError();
        return 0;
    }
    Pool &P = pool();
    std::lock_guard<std::mutex> g(P.mu);
    return P.bytes[dev];
}

void pool_trim() {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) {
        (void)hipGetLastError();
        return;
    }
    Pool &P = pool();
    std::lock_guard<std::mutex> g(P.mu);
    for (auto it = P.idle.begin(); it != P.idle.end();) {
        if (it->device == dev) {
            device_free(it->p, it->cap);
            P.bytes[dev] -= it->cap;
            it = P.idle.erase(it);
        } else {
            ++it;
        }
    }
}

void DevBuf::alloc(size_t b) {
    release();
    if (b) {
        Clock c;
        hipError_t e = device_malloc(&p, b);
        if (e == hipErrorOutOfMemory) {   // idle scratch may be what is missing
            (void)hipGetLastError();
            pool_trim();
            e = device_malloc(&p, b);
        }
        if (e != hipSuccess) {
            p = nullptr;
            throw Error(e == hipErrorOutOfMemory ? RTE_E_OUT_OF_MEMORY : RTE_E_DEVICE,
                        std::string("hipMalloc: ") + hipGetErrorString(e));
        }
    }
    bytes = b;
}

void DevBuf::release() noexcept {
    if (p) {
        bool kept = false;
        if (pooled && settled) {
            try {
                pool_give(p, cap);
                kept = true;
            } catch (...) {
            }
        }
        if (!kept) {
            Clock c;
            device_free(p, pooled ? cap : bytes);
        }
    }
    p = nullptr;
    bytes = cap = 0;
    pooled = settled = false;
}

DevBuf DevBuf::scratch(size_t b, bool exact) {
    DevBuf d;
    if (b) {
        d.p = pool_take(b, &d.cap, exact);
        d.pooled = true;
    }
    d.bytes = b;
    return d;
}

}  // namespace rte
