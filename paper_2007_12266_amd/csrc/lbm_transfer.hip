// Host <-> device copies of large caller buffers (images, neighbour tables, fields, states).
//
// The caller's host memory is pageable. A copy from pageable memory is staged by the runtime
// through pinned memory with one host thread, which caps it well below what the link carries.
// Here the staging is explicit: two pinned buffers of kChunk bytes, filled (or drained) by up
// to kThreads host threads while the DMA of the other buffer runs. The buffers are allocated
// once per process (pinned with hipHostMalloc) and shared under a mutex, so concurrent callers
// take turns; copies below kDirect bytes go straight to hipMemcpyAsync.
//
// Small results (a field of a small domain, the sums of a reduction) need no device buffer at
// all: their kernels write into pinned host memory (PinnedOut), the host waits for the stream and
// copies them out. A device-to-host copy of pageable memory costs 40 us and more before its first
// byte (a field of 20 thousand voxels took 95 us, now 25; one of 512 thousand 259, now 158; a
// reduction 60, now 45).
#include <algorithm>
#include <condition_variable>
#include <cstring>
#include <mutex>
#include <system_error>
#include <thread>
#include <vector>

#include "lbm_internal.h"

namespace lbm {
namespace {

constexpr size_t kChunk = 32u << 20;
constexpr size_t kDirect = 4u << 20;
constexpr unsigned kThreads = 8;

struct Staging {
    std::mutex mu;
    void* buf[2] = {nullptr, nullptr};
};

Staging& staging() {
    static Staging st;
    return st;
}

// The buffers of PinnedOut, kPinnedBytes each: at most kPinnedBuffers exist, made as they are first
// needed and kept for the process, each taken by one caller at a time. Further callers go through
// their device buffers instead of pinning and releasing 8 MiB in every call (8 to 16 threads that
// step, reduce and read a 32^3 bead pack take the same either way, within the 10% that runs differ).
constexpr int kPinnedBuffers = 4;
struct PinnedPool {
    std::mutex mu;
    void* idle[kPinnedBuffers];
    int n_idle = 0;
    int n_made = 0;
};

PinnedPool& pinned_pool() {
    static PinnedPool p;
    return p;
}

hipError_t ensure_buffers(Staging& st) {
    for (void*& b : st.buf)
        if (!b) {
            const hipError_t e = hipHostMalloc(&b, kChunk, hipHostMallocPortable);
            if (e != hipSuccess) {
                b = nullptr;
                return e;
            }
        }
    return hipSuccess;
}

// memcpy on up to kThreads threads, each a contiguous slice.
void copy_threads(void* dst, const void* src, size_t n) {
    const unsigned hw = std::max(1u, std::min(kThreads, std::thread::hardware_concurrency()));
    if (n < (1u << 20) || hw == 1) {
        std::memcpy(dst, src, n);
        return;
    }
    const size_t slice = (n + hw - 1) / hw;
    std::vector<std::thread> pool;
    for (unsigned t = 0; t < hw; ++t) {
        const size_t b = t * slice;
        if (b >= n) break;
        const size_t len = std::min(slice, n - b);
        try {
            pool.emplace_back([=] { std::memcpy((char*)dst + b, (const char*)src + b, len); });
        } catch (const std::system_error&) {
            std::memcpy((char*)dst + b, (const char*)src + b, len);   // no thread: copy here
        }
    }
    for (std::thread& th : pool) th.join();
}

// Two events per call (created on the current device, like the stream's work).
struct Events {
    hipEvent_t ev[2] = {nullptr, nullptr};
    hipError_t err = hipSuccess;
    Events() {
        for (hipEvent_t& e : ev)
            if (err == hipSuccess) err = hipEventCreateWithFlags(&e, hipEventDisableTiming);
    }
    ~Events() {
        for (hipEvent_t e : ev)
            if (e) (void)hipEventDestroy(e);
    }
};

// An error return leaves no DMA running on a staging buffer that the next caller would reuse.
hipError_t drained(hipError_t e, hipStream_t s) {
    (void)hipStreamSynchronize(s);
    return e;
}

}  // namespace

PinnedOut::PinnedOut(size_t bytes) {
    if (bytes > kPinnedBytes) return;
    PinnedPool& p = pinned_pool();
    {
        std::lock_guard<std::mutex> lock(p.mu);
        if (p.n_idle > 0) {
            ptr_ = p.idle[--p.n_idle];
            return;
        }
        if (p.n_made == kPinnedBuffers) return;
        ++p.n_made;
    }
    if (hipHostMalloc(&ptr_, kPinnedBytes, hipHostMallocPortable) != hipSuccess) {
        (void)hipGetLastError();
        ptr_ = nullptr;
        std::lock_guard<std::mutex> lock(p.mu);
        --p.n_made;
    }
}

PinnedOut::~PinnedOut() {
    if (!ptr_) return;
    PinnedPool& p = pinned_pool();
    std::lock_guard<std::mutex> lock(p.mu);
    p.idle[p.n_idle++] = ptr_;
}

// The copying threads are started before the wait for the stream, so that starting them (about
// 15 us each) runs beside the kernel; one for each 512 KiB, as eight took longer to start than a
// small result takes to copy (us a field of 1.4 MB through a device buffer 108, with eight threads
// from 1 MiB 119, now 67; 2.1 MB 151 / 130 / 86; 3.0 MB 195 / 133 / 112; 4.1 MB 259 / 160 / 158).
hipError_t PinnedOut::take(void* dst, size_t bytes, hipStream_t s) {
    const unsigned hw = std::max(1u, std::min(kThreads, std::thread::hardware_concurrency()));
    const size_t parts = std::max<size_t>(1, std::min<size_t>(hw, bytes >> 19));
    const size_t slice = (bytes + parts - 1) / parts;
    auto part = [&](size_t k) {
        const size_t b = k * slice;
        if (b < bytes) std::memcpy((char*)dst + b, (const char*)ptr_ + b, std::min(slice, bytes - b));
    };
    std::mutex mu;
    std::condition_variable cv;
    int go = 0;   // 1: the result is there, -1: there is none
    std::vector<std::thread> threads;
    size_t started = 1;
    try {
        threads.reserve(parts - 1);
        for (; started < parts; ++started)
            threads.emplace_back([&, k = started] {
                std::unique_lock<std::mutex> lock(mu);
                cv.wait(lock, [&] { return go != 0; });
                lock.unlock();
                if (go > 0) part(k);
            });
    } catch (const std::exception&) {
        // No thread, or no memory for one: this one copies the rest.
    }
    const hipError_t e = hipStreamSynchronize(s);
    {
        std::lock_guard<std::mutex> lock(mu);
        go = e == hipSuccess ? 1 : -1;
    }
    cv.notify_all();
    if (e == hipSuccess) {
        part(0);
        for (size_t k = started; k < parts; ++k) part(k);
    }
    for (std::thread& t : threads) t.join();
    return e;
}

hipError_t copy_to_device(void* dst, const void* src, size_t bytes, hipStream_t s) {
    if (bytes == 0) return hipSuccess;
    if (bytes < kDirect) {
        const hipError_t e = hipMemcpyAsync(dst, src, bytes, hipMemcpyHostToDevice, s);
        return e != hipSuccess ? e : hipStreamSynchronize(s);
    }
    Staging& st = staging();
    std::lock_guard<std::mutex> lock(st.mu);
    if (hipError_t e = ensure_buffers(st)) return e;
    Events evs;
    if (evs.err != hipSuccess) return evs.err;
    bool pending[2] = {false, false};
    size_t off = 0;
    for (int k = 0; off < bytes; ++k) {
        const int b = k & 1;
        const size_t len = std::min(kChunk, bytes - off);
        if (pending[b])   // the DMA that last read this buffer has finished
            if (hipError_t e = hipEventSynchronize(evs.ev[b])) return drained(e, s);
        copy_threads(st.buf[b], (const char*)src + off, len);
        if (hipError_t e = hipMemcpyAsync((char*)dst + off, st.buf[b], len,
                                          hipMemcpyHostToDevice, s))
            return drained(e, s);
        if (hipError_t e = hipEventRecord(evs.ev[b], s)) return drained(e, s);
        pending[b] = true;
        off += len;
    }
    return hipStreamSynchronize(s);
}

hipError_t copy_to_host(void* dst, const void* src, size_t bytes, hipStream_t s) {
    if (bytes == 0) return hipSuccess;
    if (bytes < kDirect) {
        const hipError_t e = hipMemcpyAsync(dst, src, bytes, hipMemcpyDeviceToHost, s);
        return e != hipSuccess ? e : hipStreamSynchronize(s);
    }
    Staging& st = staging();
    std::lock_guard<std::mutex> lock(st.mu);
    if (hipError_t e = ensure_buffers(st)) return e;
    Events evs;
    if (evs.err != hipSuccess) return evs.err;
    const size_t nchunks = (bytes + kChunk - 1) / kChunk;
    // Chunk k is copied into buffer k % 2 while the host drains chunk k - 1; the host drained
    // chunk k - 2 (same buffer) before chunk k was queued.
    for (size_t k = 0; k <= nchunks; ++k) {
        if (k < nchunks) {
            const size_t off = k * kChunk, len = std::min(kChunk, bytes - off);
            if (hipError_t e = hipMemcpyAsync(st.buf[k & 1], (const char*)src + off, len,
                                              hipMemcpyDeviceToHost, s))
                return drained(e, s);
            if (hipError_t e = hipEventRecord(evs.ev[k & 1], s)) return drained(e, s);
        }
        if (k > 0) {
            const size_t j = k - 1, off = j * kChunk, len = std::min(kChunk, bytes - off);
            if (hipError_t e = hipEventSynchronize(evs.ev[j & 1])) return drained(e, s);
            copy_threads((char*)dst + off, st.buf[j & 1], len);
        }
    }
    return hipStreamSynchronize(s);
}

}  // namespace lbm
