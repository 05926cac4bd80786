// Device memory of the library's objects, kept for reuse when an object goes.
//
// hipMalloc and hipFree of an instance's tables cost more than making them:
// 250 MB at n = m = 5000 take 0.4 to 6 ms a pair (the driver maps and unmaps
// the pages) against 0.2 ms of kernels.  A freed block waits in a cache for
// the next object that asks for about its size.
//
//  - A block enters the cache only when nothing that uses it is left on the
//    device, which its object's StreamUse says without asking the device: the
//    library has waited for everything it enqueued for the object.  Any stream
//    and thread may take it next.  The blocks of an object whose work may
//    still run go to hipFree, which waits.  (A wait for the whole device here
//    instead would not be allowed while any stream of the process is being
//    captured, by whatever thread, and would spoil that capture.)
//  - The cache holds at most PMP_DEVICE_CACHE_MB (default 1024, 0: nothing)
//    per device; past that the block freed longest ago goes back to the driver.
//    A block that nobody has asked for in kMaxIdle goes back at the next
//    allocation or free of the library (there is no thread that would do it in
//    between), everything goes back at trim() (pmp_device_cache_trim) and when
//    the driver is out of memory, whereupon the allocation is tried again.
//  - While the stream of the calling entry point is being captured (every
//    entry point that takes a stream opens a CallScope) the cache is left
//    alone: the driver is asked, as without one, and decides.
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <chrono>
#include <cstdlib>
#include <list>
#include <map>
#include <mutex>
#include <unordered_map>
#include <utility>

namespace pmp {

// What the library has enqueued for an object and not waited for: nothing, work
// on one stream, or work that a wait for one stream does not cover (several
// streams, a captured graph, the per-thread default stream).  Streams are told
// apart by their handles.
class StreamUse {
public:
    // Work was enqueued on s, or recorded into a graph that s is captured into
    // and that may be launched on any stream at any time.
    void enqueued(hipStream_t s, bool captured)
    {
        std::lock_guard<std::mutex> lock(mu_);
        ++marks_;
        if (captured || s == hipStreamPerThread || (state_ != kIdle && stream_ != s))
            state_ = kMany;
        else if (state_ == kIdle)
            state_ = kOne;
        stream_ = s;
    }
    // Taken before a wait; waited(s, it) afterwards clears the work on s unless
    // more was enqueued meanwhile (an instance is used by several runs' calls).
    uint64_t marks() const
    {
        std::lock_guard<std::mutex> lock(mu_);
        return marks_;
    }
    void waited(hipStream_t s, uint64_t marks)
    {
        std::lock_guard<std::mutex> lock(mu_);
        if (state_ == kOne && stream_ == s && marks_ == marks)
            state_ = kIdle;
    }
    bool idle() const
    {
        std::lock_guard<std::mutex> lock(mu_);
        return state_ == kIdle;
    }

private:
    enum State { kIdle, kOne, kMany };
    mutable std::mutex mu_;
    State state_ = kIdle;
    hipStream_t stream_ = nullptr;
    uint64_t marks_ = 0;
};

// An entry point's stream: within the scope of one that is being captured into
// a graph, blocks come from and go to the driver directly.
class CallScope {
public:
    explicit CallScope(hipStream_t s) : captured(stream_captured(s)), before_(direct())
    {
        direct() = captured;
    }
    ~CallScope() { direct() = before_; }
    CallScope(const CallScope &) = delete;
    CallScope &operator=(const CallScope &) = delete;
    const bool captured;

    static bool &direct()
    {
        static thread_local bool d = false;
        return d;
    }

private:
    static bool stream_captured(hipStream_t s)
    {
        hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
        if (hipStreamIsCapturing(s, &st) != hipSuccess) {
            (void)hipGetLastError();  // (the legacy stream beside a capture)
            return true;
        }
        return st != hipStreamCaptureStatusNone;
    }
    const bool before_;
};

// One entry point's use of its objects on its stream: unless it says that it
// has waited for the stream, what it enqueued counts as left when it returns.
class StreamCall : public CallScope {
public:
    // (null pointers are skipped)
    explicit StreamCall(hipStream_t s, StreamUse *a, StreamUse *b = nullptr,
                        StreamUse *c = nullptr)
        : CallScope(s), s_(s),
          uses_{{a, a ? a->marks() : 0}, {b, b ? b->marks() : 0}, {c, c ? c->marks() : 0}}
    {
    }
    void waited()
    {
        left_ = false;
        for (const Use &u : uses_)
            if (u.use)
                u.use->waited(s_, u.marks);
    }
    // (work enqueued after a wait within the call)
    void more() { left_ = true; }
    ~StreamCall()
    {
        if (!left_)
            return;
        for (const Use &u : uses_)
            if (u.use)
                u.use->enqueued(s_, captured);
    }

private:
    struct Use {
        StreamUse *use;
        uint64_t marks;
    };
    const hipStream_t s_;
    bool left_ = true;
    const Use uses_[3];
};

class DevicePool {
public:
    static DevicePool &get()
    {
        static DevicePool *p = new DevicePool;  // never destroyed: outlives the runtime
        return *p;
    }

    // Within a FreeScope(true) freed blocks have no work left on the device
    // and are kept; elsewhere they go to the driver.
    struct FreeScope {
        explicit FreeScope(bool idle) : before(keep()) { keep() = idle; }
        ~FreeScope() { keep() = before; }
        FreeScope(const FreeScope &) = delete;
        FreeScope &operator=(const FreeScope &) = delete;
        const bool before;
    };

    hipError_t alloc(void **out, size_t bytes)
    {
        *out = nullptr;
        bytes = (bytes + 511) & ~size_t(511);
        int dev = 0;
        hipError_t e = hipGetDevice(&dev);
        if (e != hipSuccess)
            return e;
        std::list<Block> idle;
        if (!CallScope::direct()) {
            std::lock_guard<std::mutex> lock(mu_);
            const auto fit = by_size_.lower_bound({dev, bytes});  // the smallest that holds it
            if (fit != by_size_.end() && fit->first.first == dev &&
                fit->first.second <= bytes + bytes / 4 + 4096) {
                std::list<Block> taken;
                *out = fit->second->p;
                live_[*out] = {fit->second->bytes, dev};
                drop(fit->second, taken);
            }
            expire(Clock::now(), idle);
        }
        to_driver(idle);
        if (*out)
            return hipSuccess;
        e = hipMalloc(out, bytes);
        if (e == hipErrorOutOfMemory && !CallScope::direct() && trim(dev)) {
            (void)hipGetLastError();
            e = hipMalloc(out, bytes);
        }
        if (e != hipSuccess) {
            (void)hipGetLastError();  // (reported here, not by the next launch)
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
        if (b.bytes == 0 || b.bytes > limit_ || CallScope::direct() || !keep()) {
            (void)hipFree(p);
            return;
        }
        std::list<Block> out;
        {
            std::lock_guard<std::mutex> lock(mu_);
            const Clock::time_point now = Clock::now();
            const auto at = cached_.insert(cached_.end(), {p, b.bytes, b.dev, now, {}});
            at->place = by_size_.insert({{b.dev, b.bytes}, at});
            held_[b.dev] += b.bytes;
            expire(now, out);
            for (auto it = cached_.begin(); held_[b.dev] > limit_;) {
                const auto next = std::next(it);
                if (it->dev == b.dev)
                    drop(it, out);
                it = next;
            }
        }
        to_driver(out);
    }

    // Every cached block of a device (dev < 0: of all) to the driver; false if
    // there was none.
    bool trim(int dev = -1)
    {
        std::list<Block> out;
        {
            std::lock_guard<std::mutex> lock(mu_);
            for (auto it = cached_.begin(); it != cached_.end();) {
                const auto next = std::next(it);
                if (dev < 0 || it->dev == dev)
                    drop(it, out);
                it = next;
            }
        }
        to_driver(out);
        return !out.empty();
    }

private:
    using Clock = std::chrono::steady_clock;
    static constexpr std::chrono::seconds kMaxIdle{10};
    struct Live {
        size_t bytes;
        int dev;
    };
    struct Block;
    using BySize = std::multimap<std::pair<int, size_t>, std::list<Block>::iterator>;
    struct Block {
        void *p;
        size_t bytes;
        int dev;
        Clock::time_point since;
        BySize::iterator place;
    };

    DevicePool()
    {
        const char *v = std::getenv("PMP_DEVICE_CACHE_MB");
        limit_ = (size_t)(v && *v ? std::max(0L, std::atol(v)) : 1024L) << 20;
    }

    static bool &keep()
    {
        static thread_local bool k = false;
        return k;
    }

    // A cached block to `out` (with mu_ held; to_driver gives it back after).
    void drop(std::list<Block>::iterator it, std::list<Block> &out)
    {
        held_[it->dev] -= it->bytes;
        by_size_.erase(it->place);
        out.splice(out.end(), cached_, it);
    }
    void expire(Clock::time_point now, std::list<Block> &out)
    {
        while (!cached_.empty() && now - cached_.front().since > kMaxIdle)
            drop(cached_.begin(), out);
    }
    static void to_driver(const std::list<Block> &blocks)
    {
        for (const Block &b : blocks)
            (void)hipFree(b.p);
    }

    std::mutex mu_;
    size_t limit_ = 0;
    std::list<Block> cached_;                // oldest first
    BySize by_size_;                         // the same by device and size
    std::unordered_map<int, size_t> held_;   // cached bytes by device
    std::unordered_map<void *, Live> live_;  // blocks in use
};

}  // namespace pmp
