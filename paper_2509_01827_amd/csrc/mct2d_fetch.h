// Device-to-host copies of query results.  A copy into pageable memory runs at 8
// to 12 GB/s and takes some 20 us even for a control block; through two small
// pinned buffers, one filling while the other is copied out, it runs at the
// link's rate, and one launch fetches a field's components together with the
// control block: one synchronisation per query.  Before -> after: 400 x 400
// displacements (2.6 MB) 286 -> 104 us, a batch specimen's (0.6 MB) 120 -> 43.
#pragma once

#include <hip/hip_runtime.h>
#include <sys/mman.h>

#include <algorithm>
#include <cstdint>
#include <cstring>
#include <memory>
#include <new>
#include <utility>

namespace mct {

// Pieces of device memory and where in pinned host memory they go (64-byte
// aligned), copied by one launch (mct2d_fetch.hip).
struct FetchPieces {
    static constexpr int kMax = 4;
    int n = 0;
    const void *src[kMax];
    void *dst[kMax];
    size_t bytes[kMax];
};
hipError_t launch_fetch(const FetchPieces &f, hipStream_t s);

class Fetch {
  public:
    struct Part {
        const void *src;  // device memory
        size_t bytes;
    };

    Fetch() = default;
    ~Fetch() { release(); }
    // (moved with its model: the buffers have one owner)
    Fetch(Fetch &&o) noexcept { *this = std::move(o); }
    Fetch &operator=(Fetch &&o) noexcept {
        std::swap(buf_, o.buf_);
        std::swap(half_, o.half_);
        std::swap(ev_, o.ev_);
        return *this;
    }

    // Buffers for results of up to `bytes` (kept; at most two of kHalf).  Without
    // them (no pinned memory to be had) run() copies into pageable memory.
    void reserve(size_t bytes) {
        const size_t want = std::min(kHalf, (bytes + 4095) & ~(size_t)4095);
        if (want <= half_) return;
        release();
        if (hipHostMalloc(reinterpret_cast<void **>(&buf_), 2 * want, hipHostMallocDefault) != hipSuccess) {
            (void)hipGetLastError();
            buf_ = nullptr;
            return;
        }
        half_ = want;
        for (hipEvent_t &e : ev_)
            if (hipEventCreateWithFlags(&e, hipEventDisableTiming) != hipSuccess) {
                (void)hipGetLastError();
                e = nullptr;
                release();
                return;
            }
    }

    void release() {
        for (hipEvent_t &e : ev_) {
            if (e) (void)hipEventDestroy(e);
            e = nullptr;
        }
        if (buf_) (void)hipHostFree(buf_);
        buf_ = nullptr;
        half_ = 0;
    }

    // Copies the parts behind the work already in the stream and hands every
    // piece over in order: take(part, offset in it, data, bytes); pieces start at
    // multiples of 64 bytes of their part.  out: where the caller puts them (its
    // pages are made present while the device is busy).
    template <class Take>
    hipError_t run(hipStream_t stream, const Part *parts, int n, void *out, size_t out_bytes, Take &&take) {
        if (!buf_) {
            for (int i = 0; i < n; ++i) {
                const std::unique_ptr<char[]> tmp(new (std::nothrow) char[parts[i].bytes]);
                if (!tmp) return hipErrorOutOfMemory;
                hipError_t e = hipMemcpyAsync(tmp.get(), parts[i].src, parts[i].bytes, hipMemcpyDeviceToHost, stream);
                if (e == hipSuccess) e = hipStreamSynchronize(stream);
                if (e != hipSuccess) return e;
                take(i, (size_t)0, tmp.get(), parts[i].bytes);
            }
            return hipSuccess;
        }
        struct Piece {
            int part;
            size_t off, bytes, at;
        };
        Piece in[2][FetchPieces::kMax];
        int count[2] = {0, 0};
        int part = 0;
        size_t off = 0;
        auto fill = [&](int b) {
            count[b] = 0;
            size_t at = 0;
            FetchPieces f;
            while (part < n && at < half_ && f.n < FetchPieces::kMax) {
                const size_t len = std::min(parts[part].bytes - off, half_ - at);
                if (len > 0) {
                    f.src[f.n] = static_cast<const char *>(parts[part].src) + off;
                    f.dst[f.n] = buf_ + b * half_ + at;
                    f.bytes[f.n++] = len;
                    in[b][count[b]++] = {part, off, len, at};
                }
                off += len;
                at = (at + len + 63) & ~(size_t)63;
                if (off == parts[part].bytes) {
                    ++part;
                    off = 0;
                }
            }
            if (f.n == 0) return hipSuccess;
            const hipError_t e = launch_fetch(f, stream);
            return e != hipSuccess ? e : hipEventRecord(ev_[b], stream);
        };
        hipError_t e = fill(0);
        if (e == hipSuccess) e = fill(1);
        if (e == hipSuccess) populate(out, out_bytes);
        for (int b = 0; e == hipSuccess && count[b] > 0; b ^= 1) {
            if ((e = hipEventSynchronize(ev_[b])) != hipSuccess) break;
            for (int i = 0; i < count[b]; ++i) {
                const Piece &p = in[b][i];
                take(p.part, p.off, buf_ + b * half_ + p.at, p.bytes);
            }
            e = fill(b);
        }
        if (e != hipSuccess) (void)hipStreamSynchronize(stream);  // no copy into the buffers is left under way
        return e;
    }

  private:
    // Fresh memory takes a page fault per 4 KB when it is first written, 400 us
    // for 2.6 MB; one request for the whole range while the device still works
    // costs a quarter and is mostly hidden.  (A hint: failure changes nothing.)
    static void populate(void *out, size_t bytes) {
        const size_t page = 4096, a = (reinterpret_cast<size_t>(out) + page - 1) & ~(page - 1);
        const size_t b = (reinterpret_cast<size_t>(out) + bytes) & ~(page - 1);
        if (bytes >= 128 * 1024 && b > a) (void)madvise(reinterpret_cast<void *>(a), b - a, 23 /* MADV_POPULATE_WRITE */);
    }

    static constexpr size_t kHalf = 1 << 20;
    char *buf_ = nullptr;
    size_t half_ = 0;
    hipEvent_t ev_[2] = {nullptr, nullptr};
};

}  // namespace mct
