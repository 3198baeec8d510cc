// pic_readback.hip -- exports of libpic: device arrays to host arrays of doubles.
//
// What bounds an export is the host: it converts to FP64 and writes an array whose pages are new, at a few
// GB/s per thread, where the copy engine delivers about 50.  So chunks are copied into a ring of pinned
// buffers (a copy into pageable memory is staged through the runtime's own buffers, one piece at a time),
// and up to kThreads threads convert each chunk while the next ones are in flight.  The fields of the
// 1024^2 disk (25 MB of floats) take 1.6 ms, those of the 256^3 sphere (407 MB) 16; a pageable
// copy of each array and one converting thread took 4.5 and 147 ms.
#include "pic_readback.h"

#include <algorithm>
#include <atomic>
#include <condition_variable>
#include <cstdlib>
#include <mutex>
#include <thread>

namespace pic {

namespace {

constexpr size_t kSlotBytes = 8u << 20;  // one chunk of all sources of a job
constexpr int kSlots = 3;
constexpr int kThreads = 8;
// Bytes copied that are worth a thread of their own.  A thread takes some 50 us to start: with one per MB, the
// fields of a 333^2 disk (2.6 MB) took 335 us when read again and again, 261 without threads or ring,
// 226 with one per 4 MB (25 MB: 1.6 ms either way).
constexpr size_t kPerThread = 4u << 20;
constexpr size_t kMaxIdle = 2;           // rings kept for the next exports
constexpr size_t kSmall = 3u << 19;      // exports up to this size go through pageable memory of their own:
                                         // a first pinned ring takes longer to allocate than they take, and
                                         // 1.2 MB take 160 us so and 171 through the ring, 1.6 MB 196 and 188
constexpr size_t kMaxSources = 16;
constexpr size_t kPad = 64;              // sources start on cache lines of their slot

struct Ring {
    char* p = nullptr;
    bool pinned = false;
};

std::mutex g_mu;
std::vector<Ring> g_idle;
long g_users = 0;

void free_ring(Ring r)
{
    if (r.pinned) (void)hipHostFree(r.p);
    else std::free(r.p);
}

// an idle ring, or a new one (pageable where no pinned memory is to be had: slower, not wrong)
Ring take_ring()
{
    {
        std::lock_guard<std::mutex> lock(g_mu);
        if (!g_idle.empty()) {
            const Ring r = g_idle.back();
            g_idle.pop_back();
            return r;
        }
    }
    Ring r;
    // an allocation is no part of a capture that another thread may have open
    hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
    (void)hipThreadExchangeStreamCaptureMode(&mode);
    void* p = nullptr;
    if (hipHostMalloc(&p, kSlotBytes * kSlots, hipHostMallocPortable) == hipSuccess) {
        r.p = static_cast<char*>(p);
        r.pinned = true;
    } else {
        (void)hipGetLastError();
        r.p = static_cast<char*>(std::malloc(kSlotBytes * kSlots));
    }
    (void)hipThreadExchangeStreamCaptureMode(&mode);
    return r;
}

void give_ring(Ring r)
{
    {
        std::lock_guard<std::mutex> lock(g_mu);
        if (g_users > 0 && g_idle.size() < kMaxIdle) {
            g_idle.push_back(r);
            return;
        }
    }
    free_ring(r);
}

// Runs f(part, parts) on every part at once: the caller's thread and a few workers, which live for one
// export.  Workers that cannot be started are done without.
class Parallel {
public:
    explicit Parallel(int parts)
    {
        for (int k = 1; k < parts; ++k) {
            try {
                workers_.emplace_back([this, k] { work(k); });
            } catch (...) {
                break;
            }
        }
        parts_ = 1 + (int)workers_.size();
    }
    ~Parallel()
    {
        {
            std::lock_guard<std::mutex> lock(mu_);
            stop_ = true;
        }
        go_.notify_all();
        for (auto& w : workers_) w.join();
    }
    void run(const std::function<void(int, int)>& f)
    {
        {
            std::lock_guard<std::mutex> lock(mu_);
            f_ = &f;
            left_ = parts_ - 1;
            ++round_;
        }
        go_.notify_all();
        f(0, parts_);
        std::unique_lock<std::mutex> lock(mu_);
        done_.wait(lock, [this] { return left_ == 0; });
    }

private:
    void work(int k)
    {
        long seen = 0;
        for (;;) {
            const std::function<void(int, int)>* f;
            {
                std::unique_lock<std::mutex> lock(mu_);
                go_.wait(lock, [&] { return stop_ || round_ != seen; });
                if (stop_) return;
                seen = round_;
                f = f_;
            }
            (*f)(k, parts_);
            std::lock_guard<std::mutex> lock(mu_);
            if (--left_ == 0) done_.notify_one();
        }
    }
    std::vector<std::thread> workers_;
    std::mutex mu_;
    std::condition_variable go_, done_;
    const std::function<void(int, int)>* f_ = nullptr;
    int parts_ = 1, left_ = 0;
    long round_ = 0;
    bool stop_ = false;
};

struct Chunk {
    const ReadbackJob* job;
    size_t first, count;
};

}  // namespace

void readback_retain()
{
    std::lock_guard<std::mutex> lock(g_mu);
    ++g_users;
}

void readback_release()
{
    std::vector<Ring> old;
    {
        std::lock_guard<std::mutex> lock(g_mu);
        if (--g_users > 0) return;
        old.swap(g_idle);
    }
    for (const Ring& r : old) free_ring(r);
}

static size_t padded(size_t bytes) { return (bytes + kPad - 1) / kPad * kPad; }

// everything copied, then one wait, then put by this thread
static hipError_t readback_small(const std::vector<ReadbackJob>& jobs, size_t bytes, hipStream_t st)
{
    char* const buf = static_cast<char*>(std::malloc(bytes));
    if (!buf) return hipErrorOutOfMemory;
    hipError_t e = hipSuccess;
    char* p = buf;
    for (const auto& j : jobs)
        for (const auto& x : j.src) {
            if (e == hipSuccess && j.n > 0) e = hipMemcpyAsync(p, x.dev, x.elem * j.n, hipMemcpyDeviceToHost, st);
            p += padded(x.elem * j.n);
        }
    const hipError_t w = hipStreamSynchronize(st);
    if (e == hipSuccess) e = w;
    p = buf;
    for (const auto& j : jobs) {
        const char* arrays[kMaxSources];
        for (size_t k = 0; k < j.src.size(); ++k) {
            arrays[k] = p;
            p += padded(j.src[k].elem * j.n);
        }
        if (e == hipSuccess && j.n > 0) j.put(arrays, 0, j.n);
    }
    std::free(buf);
    return e;
}

hipError_t readback(const std::vector<ReadbackJob>& jobs, hipStream_t st)
{
    size_t bytes = 0;
    for (const auto& j : jobs) {
        if (j.src.size() > kMaxSources) return hipErrorInvalidValue;
        for (const auto& x : j.src) bytes += padded(x.elem * j.n);
    }
    if (bytes == 0) return hipSuccess;
    if (bytes <= kSmall) return readback_small(jobs, bytes, st);
    std::vector<Chunk> chunks;
    for (const auto& j : jobs) {
        size_t per = 0;
        for (const auto& x : j.src) per += x.elem;
        if (per == 0 || j.n == 0) continue;
        const size_t most = (kSlotBytes - kPad * j.src.size()) / per;
        for (size_t a = 0; a < j.n; a += most) chunks.push_back({&j, a, std::min(most, j.n - a)});
    }
    const Ring ring = take_ring();
    if (!ring.p) return hipErrorOutOfMemory;
    hipError_t e = hipSuccess;
    hipEvent_t ev[kSlots] = {};
    // where the chunk's sources lie in its slot, `skip` elements in
    auto at = [&](const Chunk& c, int slot, size_t skip, const char** arrays) {
        const char* p = ring.p + kSlotBytes * (size_t)slot;
        for (size_t k = 0; k < c.job->src.size(); ++k) {
            arrays[k] = p + skip * c.job->src[k].elem;
            p += padded(c.count * c.job->src[k].elem);
        }
    };
    auto copy = [&](size_t i) {
        const Chunk& c = chunks[i];
        const int slot = (int)(i % kSlots);
        const char* arrays[kMaxSources];
        at(c, slot, 0, arrays);
        hipError_t r = hipSuccess;
        for (size_t k = 0; k < c.job->src.size() && r == hipSuccess; ++k) {
            const auto& x = c.job->src[k];
            r = hipMemcpyAsync(const_cast<char*>(arrays[k]), static_cast<const char*>(x.dev) + c.first * x.elem,
                               c.count * x.elem, hipMemcpyDeviceToHost, st);
        }
        return r == hipSuccess ? hipEventRecord(ev[slot], st) : r;
    };
    try {
        for (int k = 0; k < kSlots && e == hipSuccess; ++k) e = hipEventCreateWithFlags(&ev[k], hipEventDisableTiming);
        const int want = (int)std::min<size_t>(kThreads, 1 + bytes / kPerThread);
        Parallel pool(std::max(1, std::min(want, (int)std::thread::hardware_concurrency())));
        size_t next = 0;
        for (size_t i = 0; i < chunks.size() && e == hipSuccess; ++i) {
            // the slots of every chunk before i are free again
            for (; next < chunks.size() && next < i + kSlots && e == hipSuccess; ++next) e = copy(next);
            if (e == hipSuccess) e = hipEventSynchronize(ev[i % kSlots]);
            if (e != hipSuccess) break;
            const Chunk& c = chunks[i];
            pool.run([&](int part, int parts) {
                const size_t a = c.count * (size_t)part / (size_t)parts, b = c.count * (size_t)(part + 1) / (size_t)parts;
                if (a == b) return;
                const char* arrays[kMaxSources];
                at(c, (int)(i % kSlots), a, arrays);
                c.job->put(arrays, c.first + a, b - a);
            });
        }
    } catch (...) {
        e = hipErrorOutOfMemory;
    }
    // after an error copies may still be on their way into the ring
    if (e != hipSuccess) (void)hipStreamSynchronize(st);
    for (auto x : ev)
        if (x) (void)hipEventDestroy(x);
    give_ring(ring);
    return e;
}

}  // namespace pic
