// pond_readback.h -- device-to-host copies of fields into a caller's pageable arrays
// (host code of the C-ABI layer).
#pragma once

#include <hip/hip_runtime.h>
#include <sched.h>

#include <algorithm>
#include <atomic>
#include <cstring>
#include <mutex>
#include <thread>

#include "pond_internal.h"

namespace pond {

// ---------------------------------------------------------------------------
// Read-back of fields into the caller's arrays.  A copy into pageable memory runs at 7-10
// GB/s: the runtime takes the pages of a fresh array, faulted in one by one, through its own
// staging on one thread.  Here the DMA goes into pinned pieces, and a few threads move them
// to the caller's memory, faulting its pages side by side: 2048^2 (201 MB) 6.0 ms instead of
// 20.9, 1024 x 512 (25 MB) 0.8 instead of 1.5, or 1.5 instead of 3.6 into pages new to the process.
// Where all fields fit a piece the kernel that forms them writes them there (hipHostMalloc'ed
// memory is the device's too): 1000 nodes take 34 us, by five copies 134.  A copy into the
// piece takes 41, but the first one above 16 KiB starts a copy engine, 6 ms that a process of
// such lattices does not pay otherwise.  Parts of more fields that fit a piece take one copy.
// Between the sizes the runtime's own copies stay: there the gain is at most 0.3 ms, and
// helpers that meet another pool's spinning threads wait milliseconds for a core (512^2 right
// after a conversion on all 16 cores: 0.8 ms by the runtime, 1.2 with one helper, 2.1 with
// three, 3.8 with five).
//
// The pinned pieces are one allocation of at most kStageBytes for the process, made by the
// first read-back, freed with the last handle.  A read-back that finds it in use (another
// thread's), or cannot have it, copies straight into the caller's memory.
// ---------------------------------------------------------------------------
constexpr size_t kPieceBytes = 2u << 20;
constexpr int kPieces = 8;
constexpr size_t kStageBytes = kPieces * kPieceBytes;

struct Stage {
    std::mutex in_use, count;
    char *buf = nullptr; // guarded by in_use
    int handles = 0;     // guarded by count
    void enter()
    {
        std::lock_guard<std::mutex> l(count);
        ++handles;
    }
    void leave()
    {
        std::lock_guard<std::mutex> l(count);
        if (--handles > 0) return;
        // no handle is left to read back; a handle made meanwhile waits for `count`
        std::lock_guard<std::mutex> u(in_use);
        if (buf) (void)hipHostFree(buf);
        buf = nullptr;
    }
};
inline Stage g_stage;

struct ReadBack {
    static constexpr int kMost = 8;
    struct Part {
        char *dst;
        const char *src;
        size_t bytes;
    } part[kMost];
    int parts = 0;
    size_t total = 0;
    void add(const Part &p)
    {
        part[parts++] = p;
        total += p.bytes;
    }
    void add(double *dst, const double *src, size_t count)
    {
        add(Part{(char *)dst, (const char *)src, count * sizeof(double)});
    }
    hipError_t direct(hipStream_t st) const
    {
        for (int i = 0; i < parts; ++i) {
            const hipError_t e = hipMemcpyAsync(part[i].dst, part[i].src, part[i].bytes, hipMemcpyDeviceToHost, st);
            if (e != hipSuccess) return e;
        }
        return hipStreamSynchronize(st);
    }
    // one piece holds everything
    hipError_t single(hipStream_t st, char *buf) const
    {
        size_t at = 0;
        for (int i = 0; i < parts; at += part[i++].bytes) {
            // (parts that follow each other in device memory go in one copy)
            size_t n = part[i].bytes;
            const char *src = part[i].src;
            const size_t first = at;
            while (i + 1 < parts && part[i + 1].src == src + n) {
                at += part[i].bytes;
                n += part[++i].bytes;
            }
            const hipError_t e = hipMemcpyAsync(buf + first, src, n, hipMemcpyDeviceToHost, st);
            if (e != hipSuccess) return e;
        }
        const hipError_t e = hipStreamSynchronize(st);
        if (e != hipSuccess) return e;
        at = 0;
        for (int i = 0; i < parts; at += part[i++].bytes) std::memcpy(part[i].dst, buf + at, part[i].bytes);
        return hipSuccess;
    }
    // pieces in turn, each by the thread that is free, which has one slot of the staging
    hipError_t pieces(hipStream_t st, char *buf) const
    {
        size_t first[kMost + 1] = {0};
        for (int i = 0; i < parts; ++i) first[i + 1] = first[i] + (part[i].bytes + kPieceBytes - 1) / kPieceBytes;
        const size_t n = first[parts];
        std::atomic<size_t> next{0};
        std::atomic<int> failed{(int)hipSuccess};
        const StreamDevice on(st);
        hipError_t e = on.status;
        // the fields are written before a helper reads them: the caller's stream may be the
        // per-thread one, which is another stream in each thread
        if (e == hipSuccess) e = hipStreamSynchronize(st);
        if (e != hipSuccess) return e;
        // a helper for every four pieces, on at most half of the host's cores: 1024 x 512 0.76 ms
        // with three (0.93 with one, 0.80 with seven), 2048^2 5.6 with seven (6.7 with three);
        // as many of them as events can be had
        const int most = std::min(kPieces, std::max(1, (int)std::thread::hardware_concurrency() / 2)) - 1;
        const int threads = 1 + (int)std::min<size_t>(most, total / (4 * kPieceBytes));
        hipEvent_t done[kPieces];
        int slots = 0;
        while (slots < threads && hipEventCreateWithFlags(&done[slots], hipEventDisableTiming) == hipSuccess) ++slots;
        if (slots < threads) (void)hipGetLastError();
        if (slots == 0) return direct(st);
        auto work = [&](int slot) {
            char *mine = buf + slot * kPieceBytes;
            hipError_t r = hipSuccess;
            for (size_t k; r == hipSuccess && (k = next.fetch_add(1)) < n;) {
                int i = 0;
                while (k >= first[i + 1]) ++i;
                const size_t off = (k - first[i]) * kPieceBytes, bytes = std::min(kPieceBytes, part[i].bytes - off);
                r = hipMemcpyAsync(mine, part[i].src + off, bytes, hipMemcpyDeviceToHost, st);
                if (r == hipSuccess) r = hipEventRecord(done[slot], st);
                if (r == hipSuccess) r = hipEventSynchronize(done[slot]);
                if (r == hipSuccess) std::memcpy(part[i].dst + off, mine, bytes);
            }
            if (r == hipSuccess) return;
            (void)hipStreamSynchronize(st); // no copy into the staging outlives the call
            failed = (int)r;
        };
        std::thread helper[kPieces];
        try {
            for (int t = 1; t < slots; ++t)
                helper[t] = std::thread([&, t] {
                    if (hipSetDevice(on.device) == hipSuccess) work(t);
                });
        } catch (...) { // fewer helpers: the pieces are taken by those there are
        }
        work(0);
        for (auto &t : helper)
            if (t.joinable()) t.join();
        for (int t = 0; t < slots; ++t) (void)hipEventDestroy(done[t]);
        return (hipError_t)failed.load();
    }
    static hipMemoryType memory_of(const void *p)
    {
        hipPointerAttribute_t a;
        if (hipPointerGetAttributes(&a, p) == hipSuccess) return a.type;
        (void)hipGetLastError();
        return hipMemoryTypeUnregistered;
    }
    // cores that the calling thread, and so its helpers, may run on
    static int cores()
    {
        cpu_set_t set;
        if (sched_getaffinity(0, sizeof set, &set) == 0) return CPU_COUNT(&set);
        return std::max(1, (int)std::thread::hardware_concurrency());
    }
    // Reads back the added parts of the `whole` doubles that `write` (an address, to which it
    // enqueues the kernel that forms them) leaves at `dev`; ends with the copies done, the
    // stream's earlier work included.
    template <typename Write> hipError_t run(hipStream_t st, double *dev, size_t whole, Write write) const
    {
        hipError_t e;
        std::unique_lock<std::mutex> l(g_stage.in_use, std::defer_lock);
        // an array on the device is none that the host may write (0.3 us a query)
        bool host = true;
        for (int i = 0; i < parts && total <= kPieceBytes; ++i)
            host = host && memory_of(part[i].dst) != hipMemoryTypeDevice;
        if (whole * sizeof(double) <= kPieceBytes && host && staging(l)) {
            if ((e = write((double *)g_stage.buf)) != hipSuccess || (e = hipStreamSynchronize(st)) != hipSuccess) return e;
            for (int i = 0; i < parts; ++i)
                std::memcpy(part[i].dst, g_stage.buf + (part[i].src - (const char *)dev), part[i].bytes);
            return hipSuccess;
        }
        if ((e = write(dev)) != hipSuccess) return e;
        if (!host || (total > kPieceBytes && total <= kStageBytes)) return direct(st);
        if (total > kStageBytes) {
            // page-locked arrays take the DMA themselves (2048^2: 4.0 ms, 5.4 through the pieces)
            ReadBack locked, paged;
            for (int i = 0; i < parts; ++i)
                (memory_of(part[i].dst) != hipMemoryTypeUnregistered ? locked : paged).add(part[i]);
            if (locked.parts && (e = locked.direct(st)) != hipSuccess) return e;
            // on one core helpers only take turns (1024^2 4.9 ms, 4.75 by the runtime; on two
            // 2.9 against 4.76)
            if (paged.total <= kStageBytes || cores() == 1 || !staging(l)) return paged.direct(st);
            return paged.pieces(st, g_stage.buf);
        }
        return staging(l) ? single(st, g_stage.buf) : direct(st);
    }

private:
    // takes the staging, unless another read-back has it or there is none to be had
    static bool staging(std::unique_lock<std::mutex> &l)
    {
        if (!l.owns_lock() && !l.try_lock()) return false;
        if (g_stage.buf) return true;
        void *p = nullptr;
        if (hipHostMalloc(&p, kStageBytes, hipHostMallocPortable) == hipSuccess) g_stage.buf = (char *)p;
        else (void)hipGetLastError();
        return g_stage.buf != nullptr;
    }
};

} // namespace pond
