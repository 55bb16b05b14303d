// lhmm_stage.h -- read-backs to the caller's memory through pinned memory
// that an engine keeps (not part of the public ABI).
//
// A copy to pageable memory goes through the runtime's own staging: 26 us for
// 36 KB, 82 us for 171 KB, each with its own wait.  Asynchronous copies to
// pinned memory and one wait take 10 and 16 us, of which 10 are the wait.
// What exceeds half of the stage goes in pieces: one is on its way while the
// host takes the other.
#ifndef LHMM_STAGE_H
#define LHMM_STAGE_H

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>
#include <mutex>

struct HostStage {
    static constexpr size_t HALF = 512 * 1024;
    struct Part {
        const void* src;  // device
        size_t bytes;     // of whole elements of at most 16 bytes
    };

    // fill(offset, bytes, pinned) enqueues the bytes [offset, offset + bytes)
    // of `total` on the stream, take(offset, bytes, pinned) receives them;
    // offsets are multiples of 16.  The work on the stream before it has ended
    // when it returns, also where there is nothing to read.  Runs with the
    // engine's device current, whatever the caller's: the events belong to it,
    // and so do a null stream and what fill launches.
    template <class Fill, class Take>
    hipError_t run(hipStream_t st, size_t total, Fill fill, Take take) {
        const OnDevice here(device);
        if (here.error != hipSuccess) return here.error;
        if (total == 0) return hipStreamSynchronize(st);
        std::lock_guard<std::mutex> lock(busy);  // threads that read one engine take turns
        hipError_t e = grow(total);
        for (size_t o = 0; e == hipSuccess && o < total + HALF; o += HALF) {
            if (o < total) {
                e = fill(o, std::min(HALF, total - o), half(o));
                if (e == hipSuccess) e = hipEventRecord(done[o / HALF % 2], st);
            }
            if (e == hipSuccess && o > 0) {  // the piece before
                const size_t q = o - HALF;
                e = hipEventSynchronize(done[q / HALF % 2]);
                if (e == hipSuccess) take(q, std::min(HALF, total - q), half(q));
            }
        }
        if (e != hipSuccess) (void)hipStreamSynchronize(st);  // nothing of this call writes to the stage any more
        return e;
    }

    // Copies of n parts: take(part, offset in the part, bytes, pinned).
    template <class Take>
    hipError_t read(hipStream_t st, const Part* parts, int n, Take take) {
        size_t total = 0;
        for (int k = 0; k < n; ++k) total += round16(parts[k].bytes);
        // the pieces of the parts in [o, o + len): f(part, offset in the part, bytes, offset from o)
        auto pieces = [&](size_t o, size_t len, auto f) {
            size_t base = 0;
            for (int k = 0; k < n; ++k) {
                const size_t lo = std::max(o, base), hi = std::min(o + len, base + parts[k].bytes);
                if (lo < hi) f(k, lo - base, hi - lo, lo - o);
                base += round16(parts[k].bytes);
            }
        };
        return run(
            st, total,
            [&](size_t o, size_t len, char* pinned) {
                hipError_t e = hipSuccess;
                pieces(o, len, [&](int k, size_t at, size_t bytes, size_t to) {
                    if (e == hipSuccess)
                        e = hipMemcpyAsync(pinned + to, (const char*)parts[k].src + at, bytes, hipMemcpyDeviceToHost, st);
                });
                return e;
            },
            [&](size_t o, size_t len, const char* pinned) {
                pieces(o, len, [&](int k, size_t at, size_t bytes, size_t from) { take(k, at, bytes, pinned + from); });
            });
    }

    // Plain copies; parts whose destination is null are left out.
    template <int N>
    hipError_t copy(hipStream_t st, const Part (&parts)[N], void* const (&dst)[N]) {
        Part p[N];
        char* d[N];
        int n = 0;
        for (int k = 0; k < N; ++k)
            if (dst[k]) {
                p[n] = parts[k];
                d[n++] = (char*)dst[k];
            }
        return read(st, p, n, [&](int k, size_t at, size_t bytes, const char* x) { std::memcpy(d[k] + at, x, bytes); });
    }

    void release() {
        if (host) (void)hipHostFree(host);
        for (hipEvent_t& d : done) {
            if (d) (void)hipEventDestroy(d);
            d = nullptr;
        }
        host = nullptr;
        cap = 0;
    }

    // Called once by an engine's create, with its device current.  Pinned memory
    // for read-backs of `total` bytes (0: with the first one, where the
    // allocation would be most of a short create); run() grows it where needed.
    hipError_t reserve(size_t total) {
        const hipError_t e = hipGetDevice(&device);
        return e == hipSuccess ? grow(total) : e;
    }

private:
    // makes a device current, and the caller's again at the end
    struct OnDevice {
        hipError_t error;
        int before = -1;
        explicit OnDevice(int device) {
            error = hipGetDevice(&before);
            if (error != hipSuccess || before == device) {
                before = -1;
            } else {
                error = hipSetDevice(device);
            }
        }
        ~OnDevice() {
            if (before >= 0) (void)hipSetDevice(before);
        }
        OnDevice(const OnDevice&) = delete;
        OnDevice& operator=(const OnDevice&) = delete;
    };

    hipError_t grow(size_t total) {
        const size_t need = std::min(round16(total), 2 * HALF);
        for (hipEvent_t& d : done) {
            const hipError_t e = d ? hipSuccess : hipEventCreateWithFlags(&d, hipEventDisableTiming);
            if (e != hipSuccess) return e;
        }
        if (need <= cap) return hipSuccess;
        if (host) (void)hipHostFree(host);
        host = nullptr;
        cap = 0;
        const hipError_t e = hipHostMalloc((void**)&host, need);
        if (e == hipSuccess) cap = need;
        return e;
    }

    static size_t round16(size_t b) { return (b + 15) / 16 * 16; }
    char* half(size_t o) const { return host + o / HALF % 2 * HALF; }
    std::mutex busy;
    int device = 0;
    char* host = nullptr;
    size_t cap = 0;
    hipEvent_t done[2] = {};
};

#endif
