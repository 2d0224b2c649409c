// Copies pieces of device memory into pinned host memory (gfx950): one launch
// for the control block and the components of a field, in place of a copy
// command each (some 10 us apiece).  Bound by the host link: every wavefront
// stores whole 512-byte runs.
#include "mct2d_fetch.h"

namespace mct {
namespace {

constexpr int kThreads = 256;

__global__ __launch_bounds__(kThreads) void k_fetch(FetchPieces f) {
    const size_t t = (size_t)blockIdx.x * kThreads + threadIdx.x, nt = (size_t)gridDim.x * kThreads;
    for (int i = 0; i < f.n; ++i) {
        const size_t n = f.bytes[i];
        // (the destination is 64-byte aligned; a source of another alignment is
        // read in bytes)
        const size_t words = (reinterpret_cast<size_t>(f.src[i]) & 7) == 0 ? n / 8 : 0;
        const uint64_t *const s = static_cast<const uint64_t *>(f.src[i]);
        uint64_t *const d = static_cast<uint64_t *>(f.dst[i]);
        for (size_t q = t; q < words; q += nt) d[q] = s[q];
        const uint8_t *const sb = static_cast<const uint8_t *>(f.src[i]);
        uint8_t *const db = static_cast<uint8_t *>(f.dst[i]);
        for (size_t q = 8 * words + 4 * t; q < n; q += 4 * nt) {
            if (q + 4 <= n) {
                const uint32_t v = (uint32_t)sb[q] | (uint32_t)sb[q + 1] << 8 | (uint32_t)sb[q + 2] << 16 |
                                   (uint32_t)sb[q + 3] << 24;
                *reinterpret_cast<uint32_t *>(db + q) = v;
            } else {
                for (size_t b = q; b < n; ++b) db[b] = sb[b];
            }
        }
    }
}

}  // namespace

hipError_t launch_fetch(const FetchPieces &f, hipStream_t s) {
    size_t total = 0;
    for (int i = 0; i < f.n; ++i) total += f.bytes[i];
    const size_t blocks = (total / 8 + kThreads - 1) / kThreads;
    (void)hipGetLastError();
    k_fetch<<<(unsigned)std::min<size_t>(std::max<size_t>(blocks, 1), 512), kThreads, 0, s>>>(f);
    return hipGetLastError();
}

}  // namespace mct
