// host_read.hpp -- reads of device memory into the caller's host arrays.
// Part of the lbm.hip translation unit.
//
// The caller's arrays are ordinary (pageable) memory, usually fresh, so that
// a read also takes their page faults.  The HIP runtime stages such copies
// through its own pinned chunks and copies out of them on the calling thread:
// 10.7 GB/s into fresh memory (537 MB of a 256^3 grid's fields: 50 ms), where
// the link moves 57 GB/s.  Here the data comes through pinned memory: small
// reads through 512 KB, in one go, with one synchronisation for all arrays;
// large ones through a ring of 2 MB chunks, the copies into it
// overlapping the copies out of it on up to 8 threads (43 to 51 GB/s into
// fresh memory).  Arrays that are pinned already are copied to directly (8 MB
// of fields 192 us, through the ring 510).  Between the two the runtime's own way is the faster: the
// threads take 60 to 100 us to start and the memory is mapped already (kLargeRead).
// Pinning takes 0.1 ms for the small memory and over a
// millisecond for a ring, so a read borrows what it needs and gives it back:
// what is idle (at most two rings and four small pieces) serves the next
// reads of any handle, and is freed with the last handle.
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cstring>
#include <memory>
#include <mutex>
#include <thread>
#include <vector>

namespace lbm {

struct HostSegment {
    void *dst;         // host; nullptr: not wanted
    const void *src;   // device
    size_t bytes;
};

// Memory that the runtime copies to as fast as the link moves: the caller's
// own pinned memory, or any other that is not ordinary host memory.
inline bool known_to_runtime(const void *p) {
    hipPointerAttribute_t a;
    if (hipPointerGetAttributes(&a, p) == hipSuccess) return a.type != hipMemoryTypeUnregistered;
    (void)hipGetLastError();
    return false;
}

// While it lives, allocations and frees of this thread do not disturb a stream
// capture that is under way, here or in another thread.
class CaptureGuard {
public:
    CaptureGuard() : relaxed_(hipThreadExchangeStreamCaptureMode(&mode_) == hipSuccess) {}
    CaptureGuard(const CaptureGuard &) = delete;
    CaptureGuard &operator=(const CaptureGuard &) = delete;
    ~CaptureGuard() {
        if (relaxed_) (void)hipThreadExchangeStreamCaptureMode(&mode_);
    }

private:
    hipStreamCaptureMode mode_ = hipStreamCaptureModeRelaxed;
    bool relaxed_;
};

// Pinned memory, or nullptr.
inline void *pinned_alloc(size_t bytes) {
    CaptureGuard guard;
    void *p = nullptr;
    if (hipHostMalloc(&p, bytes, hipHostMallocPortable) != hipSuccess) {
        p = nullptr;
        (void)hipGetLastError();
    }
    return p;
}
inline void pinned_free(void *p) {
    CaptureGuard guard;
    (void)hipHostFree(p);
}

// A ring of pinned chunks and an event per chunk, of the device it was made on.
struct HostRing {
    static constexpr size_t kChunk = size_t(2) << 20;
    static constexpr int kSlots = 8;
    int device = -1;
    char *mem = nullptr;
    hipEvent_t event[kSlots] = {};

    HostRing() = default;
    HostRing(const HostRing &) = delete;
    HostRing &operator=(const HostRing &) = delete;
    ~HostRing() {
        if (mem) pinned_free(mem);
        for (hipEvent_t e : event)
            if (e) (void)hipEventDestroy(e);
    }
    bool open(int dev) {
        device = dev;
        mem = static_cast<char *>(pinned_alloc(kChunk * kSlots));
        bool ok = mem != nullptr;
        for (int k = 0; k < kSlots && ok; ++k)
            ok = hipEventCreateWithFlags(&event[k], hipEventDisableTiming) == hipSuccess;
        if (!ok) (void)hipGetLastError();
        return ok;
    }
};

// Pinned memory of a small read: one copy and one memcpy.  (The fields of a 422 x
// 33 grid, 446 KB, cost 100 us more in 7 pieces through the ring: an event and
// a wait each.)
constexpr size_t kSmallRead = size_t(512) << 10;
// Reads of at least this take the ring.  (us for density and velocity, by the
// runtime / through the ring: 1 MB 78 / 112, 2 MB 137 / 189, 4 MB 253 / 358,
// 6 MB 385 / 398, 8 MB 480 / 437, 24 MB 1434 / 770.)  So do all parts of a long
// array, which is fresh memory where the allocator maps it for itself (32 MB):
// there the runtime's thread also takes its page faults.
constexpr size_t kLargeRead = size_t(7) << 20;
constexpr size_t kLongArray = size_t(32) << 20;
struct PinnedFree {
    void operator()(char *p) const { pinned_free(p); }
};
using SmallPinned = std::unique_ptr<char, PinnedFree>;

// The idle pinned memory of the process.
class HostRingPool {
public:
    static HostRingPool &get() {
        static HostRingPool *pool = new HostRingPool();   // never destroyed: it may outlive the HIP runtime
        return *pool;
    }
    void enter() {
        std::lock_guard<std::mutex> lock(mu_);
        ++users_;
    }
    void leave() {
        std::unique_ptr<HostRing> rings[kIdle];
        SmallPinned small[kIdleSmall];
        std::lock_guard<std::mutex> lock(mu_);
        if (--users_ > 0) return;
        for (int k = 0; k < kIdle; ++k) rings[k] = std::move(idle_[k]);
        for (int k = 0; k < kIdleSmall; ++k) small[k] = std::move(small_[k]);
    }
    // create: allocate when none is idle (else nullptr)
    SmallPinned borrow_small(bool create) {
        {
            std::lock_guard<std::mutex> lock(mu_);
            for (auto &s : small_)
                if (s) return std::move(s);
        }
        return SmallPinned(create ? static_cast<char *>(pinned_alloc(kSmallRead)) : nullptr);
    }
    void give_back(SmallPinned s) {
        std::lock_guard<std::mutex> lock(mu_);
        for (auto &slot : small_)
            if (!slot) {
                slot = std::move(s);
                return;
            }
    }
    std::unique_ptr<HostRing> borrow(int device) {
        {
            std::lock_guard<std::mutex> lock(mu_);
            for (auto &r : idle_)
                if (r && r->device == device) return std::move(r);
        }
        std::unique_ptr<HostRing> r(new (std::nothrow) HostRing());
        if (r && !r->open(device)) r.reset();
        return r;
    }
    void give_back(std::unique_ptr<HostRing> r) {
        std::lock_guard<std::mutex> lock(mu_);
        for (auto &slot : idle_)
            if (!slot) {
                slot = std::move(r);
                return;
            }
    }   // no room: freed with r

private:
    static constexpr int kIdle = 2, kIdleSmall = 4;
    std::mutex mu_;
    int users_ = 0;
    std::unique_ptr<HostRing> idle_[kIdle];
    SmallPinned small_[kIdleSmall];
};

class HostReader {
public:
    static constexpr int kThreads = 8;

    HostReader() { HostRingPool::get().enter(); }
    HostReader(const HostReader &) = delete;
    HostReader &operator=(const HostReader &) = delete;
    ~HostReader() { HostRingPool::get().leave(); }

    // Copies the segments after the work enqueued on `st` and waits for them.
    // may_allocate false: by the runtime's own staging where no pinned memory is
    // idle.  whole: bytes of the array that the segments are a part of.
    template <int N>
    hipError_t read(hipStream_t st, const HostSegment (&seg)[N], bool may_allocate = true, size_t whole = 0) {
        size_t total = 0;
        for (const HostSegment &s : seg)
            if (s.dst) total += (s.bytes + 15) / 16 * 16;
        // (under 64 KB the copy out takes less than the question)
        bool direct = total > (size_t(64) << 10);
        for (const HostSegment &s : seg) direct = direct && (!s.dst || known_to_runtime(s.dst));
        if (direct) return read_plain(st, seg, N);
        int device = -1;
        if (total <= kSmallRead) {
            if (SmallPinned mem = HostRingPool::get().borrow_small(may_allocate)) {
                const hipError_t e = read_small(st, mem.get(), seg, N);
                HostRingPool::get().give_back(std::move(mem));
                return e;
            }
        } else if ((total >= kLargeRead || whole >= kLongArray) && may_allocate && hipGetDevice(&device) == hipSuccess) {
            if (std::unique_ptr<HostRing> ring = HostRingPool::get().borrow(device)) {
                const hipError_t e = read_large(st, *ring, seg, N, total);
                HostRingPool::get().give_back(std::move(ring));
                return e;
            }
        }
        return read_plain(st, seg, N);
    }

private:
    struct Piece {
        char *dst;
        const char *src;
        size_t bytes;
    };

    hipError_t read_plain(hipStream_t st, const HostSegment *seg, int n) {
        for (int k = 0; k < n; ++k) {
            if (!seg[k].dst) continue;
            const hipError_t e = hipMemcpyAsync(seg[k].dst, seg[k].src, seg[k].bytes, hipMemcpyDeviceToHost, st);
            if (e != hipSuccess) return e;
        }
        return hipStreamSynchronize(st);
    }

    hipError_t read_small(hipStream_t st, char *mem, const HostSegment *seg, int n) {
        size_t at = 0;
        for (int k = 0; k < n; ++k) {
            if (!seg[k].dst) continue;
            const hipError_t e = hipMemcpyAsync(mem + at, seg[k].src, seg[k].bytes, hipMemcpyDeviceToHost, st);
            if (e != hipSuccess) {
                (void)hipStreamSynchronize(st);   // nothing writes the memory any more
                return e;
            }
            at += (seg[k].bytes + 15) / 16 * 16;
        }
        const hipError_t e = hipStreamSynchronize(st);
        if (e != hipSuccess) return e;
        at = 0;
        for (int k = 0; k < n; ++k) {
            if (!seg[k].dst) continue;
            std::memcpy(seg[k].dst, mem + at, seg[k].bytes);
            at += (seg[k].bytes + 15) / 16 * 16;
        }
        return hipSuccess;
    }

    hipError_t read_large(hipStream_t st, HostRing &ring, const HostSegment *seg, int nseg, size_t total) {
        constexpr size_t kChunk = HostRing::kChunk;
        constexpr int kSlots = HostRing::kSlots;
        std::vector<Piece> piece;
        std::unique_ptr<std::atomic<bool>[]> done;   // piece copied out, its slot free
        // whole chunks for long reads, shorter pieces so that every thread gets some
        const size_t len = std::min(kChunk, std::max(size_t(256) << 10, (total / (2 * kThreads) + 4095) / 4096 * 4096));
        std::vector<std::thread> crew;
        std::atomic<int> arrived{0};
        std::atomic<bool> stop{false};
        int n = 0, workers = 0;
        auto work = [&](int w) {
            for (int k = w; k < n; k += workers) {
                while (arrived.load(std::memory_order_acquire) <= k) {
                    if (stop.load(std::memory_order_relaxed)) return;
                    std::this_thread::yield();
                }
                std::memcpy(piece[k].dst, ring.mem + (size_t)(k % kSlots) * kChunk, piece[k].bytes);
                done[k].store(true, std::memory_order_release);
            }
        };
        try {
            for (int s = 0; s < nseg; ++s)
                for (size_t at = 0; seg[s].dst && at < seg[s].bytes; at += len)
                    piece.push_back({static_cast<char *>(seg[s].dst) + at, static_cast<const char *>(seg[s].src) + at,
                                     std::min(len, seg[s].bytes - at)});
            n = (int)piece.size();
            done.reset(new std::atomic<bool>[n]);
            for (int k = 0; k < n; ++k) done[k].store(false, std::memory_order_relaxed);
            const unsigned cpus = std::thread::hardware_concurrency();
            const int most = (int)std::min<size_t>(kThreads, std::max<size_t>(1, total / (size_t(512) << 10)));
            workers = std::min({most, n, cpus ? (int)cpus : 1});
        } catch (...) {
            return hipErrorOutOfMemory;
        }
        // The crew comes when the first piece has: until then the stream may still
        // be at work on what was enqueued before the read, for any time, and a
        // crew would spin on it (a read behind 0.29 s of steps kept 9 cores busy
        // all that time).  A crew that cannot be had in full is a smaller one;
        // the calling thread copies out itself when there is none.
        const int wanted = workers;
        std::atomic<int> hired{-1};
        auto start = [&](int w) {
            int c;
            while ((c = hired.load(std::memory_order_acquire)) < 0) std::this_thread::yield();
            if (w < c) work(w);
        };
        auto hire = [&]() {
            try {
                crew.reserve(wanted);
                for (int w = 0; w < wanted; ++w) crew.emplace_back(start, w);
            } catch (...) {
            }
            workers = (int)crew.size();
            hired.store(workers, std::memory_order_release);
        };

        hipError_t e = hipSuccess;
        int issued = 0, here = 0;
        while (here < n && e == hipSuccess) {
            if (issued < n && (issued < kSlots || done[issued - kSlots].load(std::memory_order_acquire))) {
                const int slot = issued % kSlots;
                e = hipMemcpyAsync(ring.mem + (size_t)slot * kChunk, piece[issued].src, piece[issued].bytes,
                                   hipMemcpyDeviceToHost, st);
                if (e == hipSuccess) e = hipEventRecord(ring.event[slot], st);
                ++issued;
            } else if (here < issued) {
                e = hipEventSynchronize(ring.event[here % kSlots]);
                if (e != hipSuccess) break;
                if (here == 0) hire();
                arrived.store(here + 1, std::memory_order_release);
                if (workers == 0) {
                    std::memcpy(piece[here].dst, ring.mem + (size_t)(here % kSlots) * kChunk, piece[here].bytes);
                    done[here].store(true, std::memory_order_relaxed);
                }
                ++here;
            } else {
                std::this_thread::yield();
            }
        }
        if (e != hipSuccess) stop.store(true, std::memory_order_relaxed);
        for (std::thread &t : crew) t.join();
        if (e != hipSuccess) (void)hipStreamSynchronize(st);   // the ring is not written any more
        return e;
    }
};

}  // namespace lbm
