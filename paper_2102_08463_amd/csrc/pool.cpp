// Device memory of plans and batches.
//
// Freeing a block unmaps it: destroying a plan of 380 MB (3D, 4e6 points) took
// 4.5 ms and making one 0.9 ms, several times the work of a differentiable
// transform, which makes a plan per call.  Freed blocks are therefore kept
// for the next plan: at most kKeepBytes per device (oldest returned first),
// none longer than kKeepSeconds at the next allocation or free, all of them
// when an allocation fails or mnufft_release_memory asks.  A block enters the pool only when the device no longer
// uses it (its owner has waited), so any stream and thread may take it.
#include "host_common.h"

#include <algorithm>
#include <chrono>
#include <mutex>
#include <unordered_map>

namespace mn {
namespace host {
namespace {

constexpr size_t kKeepBytes = (size_t)1 << 30;
constexpr double kKeepSeconds = 10.0;

using Clock = std::chrono::steady_clock;

struct Block {
    void *ptr;
    size_t bytes;
    int dev;
    Clock::time_point since;
};

struct Pool {
    std::mutex m;
    std::unordered_map<void *, Block> live;
    std::vector<Block> idle;  // oldest first

    static bool past(const Block &b, Clock::time_point now)
    {
        return std::chrono::duration<double>(now - b.since).count() > kKeepSeconds;
    }

    // Returns blocks past their time, when there are any.
    void age()
    {
        if (!idle.empty() && past(idle.front(), Clock::now())) trim(-1, SIZE_MAX);
    }

    // Returns idle blocks of dev (all devices if negative) to the system:
    // those past their time, then the oldest until `keep` bytes remain.
    void trim(int dev, size_t keep)
    {
        const Clock::time_point now = Clock::now();
        size_t held = 0;
        for (const Block &b : idle)
            if (dev < 0 || b.dev == dev) held += b.bytes;
        size_t n = 0;
        for (const Block &b : idle) {
            const bool mine = dev < 0 || b.dev == dev;
            if (past(b, now) || (mine && held > keep)) {
                if (mine) held -= b.bytes;
                (void)hipFree(b.ptr);
            } else {
                idle[n++] = b;
            }
        }
        idle.resize(n);
    }
};

// (never destroyed: the HIP runtime may be gone when statics are)
Pool &pool()
{
    static Pool *p = new Pool();
    return *p;
}

// Eight sizes per octave, so that blocks fit plans of about the same size.
size_t size_class(size_t bytes)
{
    if (bytes > kKeepBytes / 2) return bytes;
    size_t top = 1;
    while (top * 2 <= bytes) top *= 2;
    const size_t step = std::max<size_t>(512, top / 8);
    return (bytes + step - 1) / step * step;
}

}  // namespace

hipError_t pool_alloc(void **ptr, size_t bytes)
{
    *ptr = nullptr;
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    size_t size = size_class(bytes);
    try {
        Pool &p = pool();
        std::lock_guard<std::mutex> lock(p.m);
        for (size_t i = 0; i < p.idle.size(); ++i) {
            const Block b = p.idle[i];
            if (b.dev != dev || b.bytes != size) continue;
            p.live.emplace(b.ptr, b);
            p.idle.erase(p.idle.begin() + i);
            *ptr = b.ptr;
            p.age();
            return hipSuccess;
        }
        p.age();
        e = hipMalloc(ptr, size);
        if (e == hipErrorOutOfMemory && !p.idle.empty()) {
            (void)hipGetLastError();
            p.trim(-1, 0);
            e = hipMalloc(ptr, size);
        }
        if (e == hipErrorOutOfMemory && size > bytes) {  // without the class's rest
            (void)hipGetLastError();
            size = bytes;
            e = hipMalloc(ptr, size);
        }
        if (e != hipSuccess) {
            *ptr = nullptr;
            (void)hipGetLastError();
            return e;
        }
        try {
            p.live.emplace(*ptr, Block{*ptr, size, dev, Clock::now()});
        } catch (...) {
            (void)hipFree(*ptr);
            *ptr = nullptr;
            return hipErrorOutOfMemory;
        }
        return hipSuccess;
    } catch (...) {
        return hipErrorOutOfMemory;
    }
}

void pool_free(void *ptr, bool idle)
{
    if (!ptr) return;
    try {
        Pool &p = pool();
        std::lock_guard<std::mutex> lock(p.m);
        auto it = p.live.find(ptr);
        if (it == p.live.end()) return;
        Block b = it->second;
        p.live.erase(it);
        if (!idle || b.bytes > kKeepBytes / 2) {
            (void)hipFree(ptr);
            return;
        }
        b.since = Clock::now();
        try {
            p.idle.push_back(b);
        } catch (...) {
            (void)hipFree(ptr);
            return;
        }
        p.trim(b.dev, kKeepBytes);
    } catch (...) {
    }
}

}  // namespace host
}  // namespace mn

extern "C" int mnufft_release_memory(void)
{
    try {
        mn::host::Pool &p = mn::host::pool();
        std::lock_guard<std::mutex> lock(p.m);
        p.trim(-1, 0);
    } catch (...) {
        return MNUFFT_ERR_HIP;
    }
    return MNUFFT_OK;
}
