// Device memory of the library's objects, kept for reuse when an object goes.
//
// hipMalloc and hipFree of an instance's tables cost more than making them:
// 250 MB at n = m = 5000 take 0.4 to 6 ms a pair (the driver maps and unmaps
// the pages) against 0.2 ms of kernels.  A freed block waits in a cache for
// the next object that asks for about its size.
//
//  - A block enters the cache only when its device has finished all work (the
//    wait hipFree makes too), so any stream and thread may take it next.
//  - The cache holds at most PMP_DEVICE_CACHE_MB (default 1024) per device;
//    past that the block freed longest ago goes back to the driver, as does
//    every block that nobody has asked for in kMaxIdle.  When the driver is
//    out of memory everything cached goes back and the allocation is tried
//    again.
//  - While the calling entry point's stream is being captured the cache is
//    left alone: the driver is asked, as without one, and decides.
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <chrono>
#include <cstdlib>
#include <list>
#include <mutex>
#include <unordered_map>

namespace pmp {

class DevicePool {
public:
    static DevicePool &get()
    {
        static DevicePool *p = new DevicePool;  // never destroyed: outlives the runtime
        return *p;
    }

    // Within a CallScope of a stream under capture, blocks come from and go to
    // the driver directly.
    struct CallScope {
        explicit CallScope(hipStream_t s) : before(direct())
        {
            hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
            if (hipStreamIsCapturing(s, &st) != hipSuccess) {
                (void)hipGetLastError();  // (the legacy stream beside a capture)
                st = hipStreamCaptureStatusActive;
            }
            direct() = st != hipStreamCaptureStatusNone;
        }
        ~CallScope() { direct() = before; }
        CallScope(const CallScope &) = delete;
        CallScope &operator=(const CallScope &) = delete;
        const bool before;
    };

    // Several frees with one wait for the device: the scope's first free
    // waits, the others belong to the same object.
    struct FreeScope {
        FreeScope() : before(waited()) { waited() = -1; }
        ~FreeScope() { waited() = before; }
        FreeScope(const FreeScope &) = delete;
        FreeScope &operator=(const FreeScope &) = delete;
        const int before;
    };

    hipError_t alloc(void **out, size_t bytes)
    {
        *out = nullptr;
        bytes = (bytes + 511) & ~size_t(511);
        int dev = 0;
        hipError_t e = hipGetDevice(&dev);
        if (e != hipSuccess)
            return e;
        if (!direct()) {
            std::lock_guard<std::mutex> lock(mu_);
            auto best = cached_.end();
            for (auto it = cached_.begin(); it != cached_.end(); ++it)
                if (it->dev == dev && it->bytes >= bytes && it->bytes <= bytes + bytes / 4 + 4096 &&
                    (best == cached_.end() || it->bytes < best->bytes))
                    best = it;
            if (best != cached_.end()) {
                *out = best->p;
                live_[best->p] = {best->bytes, dev};
                held_[dev] -= best->bytes;
                cached_.erase(best);
                return hipSuccess;
            }
        }
        e = hipMalloc(out, bytes);
        if (e == hipErrorOutOfMemory && !direct() && give_back(dev)) {
            (void)hipGetLastError();
            e = hipMalloc(out, bytes);
        }
        if (e != hipSuccess) {
            *out = nullptr;
            return e;
        }
        std::lock_guard<std::mutex> lock(mu_);
        live_[*out] = {bytes, dev};
        return hipSuccess;
    }

    void free(void *p)
    {
        if (!p)
            return;
        Live b{0, 0};
        {
            std::lock_guard<std::mutex> lock(mu_);
            const auto it = live_.find(p);
            if (it != live_.end()) {
                b = it->second;
                live_.erase(it);
            }
        }
        if (b.bytes == 0 || b.bytes > limit_ || direct() || !wait_for(b.dev)) {
            (void)hipFree(p);
            return;
        }
        std::list<Block> out;
        {
            std::lock_guard<std::mutex> lock(mu_);
            const Clock::time_point now = Clock::now();
            cached_.push_back({p, b.bytes, b.dev, now});  // (oldest first)
            held_[b.dev] += b.bytes;
            for (auto it = cached_.begin(); it != cached_.end();) {
                const auto next = std::next(it);
                if (now - it->since > kMaxIdle || (it->dev == b.dev && held_[b.dev] > limit_)) {
                    held_[it->dev] -= it->bytes;
                    out.splice(out.end(), cached_, it);
                }
                it = next;
            }
        }
        for (const Block &o : out)
            (void)hipFree(o.p);
    }

private:
    using Clock = std::chrono::steady_clock;
    static constexpr std::chrono::seconds kMaxIdle{10};
    struct Live {
        size_t bytes;
        int dev;
    };
    struct Block {
        void *p;
        size_t bytes;
        int dev;
        Clock::time_point since;
    };

    DevicePool()
    {
        const char *v = std::getenv("PMP_DEVICE_CACHE_MB");
        limit_ = (size_t)(v && *v ? std::max(0L, std::atol(v)) : 1024L) << 20;
    }

    static bool &direct()
    {
        static thread_local bool d = false;
        return d;
    }
    // -2: outside a FreeScope; -1: in one, no wait yet; else the device the
    // scope has waited for
    static int &waited()
    {
        static thread_local int w = -2;
        return w;
    }

    // All work of device dev done (false: the wait is not possible now)
    static bool wait_for(int dev)
    {
        if (waited() == dev)
            return true;
        int cur = dev;
        if (hipGetDevice(&cur) != hipSuccess || (cur != dev && hipSetDevice(dev) != hipSuccess))
            return false;
        const bool ok = hipDeviceSynchronize() == hipSuccess;
        if (!ok)
            (void)hipGetLastError();
        if (cur != dev)
            (void)hipSetDevice(cur);
        if (ok && waited() == -1)
            waited() = dev;
        return ok;
    }

    // Every cached block of a device to the driver; false if there was none.
    bool give_back(int dev)
    {
        std::list<Block> out;
        {
            std::lock_guard<std::mutex> lock(mu_);
            for (auto it = cached_.begin(); it != cached_.end();) {
                const auto next = std::next(it);
                if (it->dev == dev)
                    out.splice(out.end(), cached_, it);
                it = next;
            }
            held_[dev] = 0;
        }
        for (const Block &o : out)
            (void)hipFree(o.p);
        return !out.empty();
    }

    std::mutex mu_;
    size_t limit_ = 0;
    std::list<Block> cached_;                // oldest first
    std::unordered_map<int, size_t> held_;   // cached bytes by device
    std::unordered_map<void *, Live> live_;  // blocks in use
};

}  // namespace pmp
