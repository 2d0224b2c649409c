// Values handed between the workgroups of a running launch (the resident
// steps): tagged words in device memory.
//
// A word is 64 bits: a 21-bit tag (the epoch of the step that wrote it) and
// 43 bits of a value.  Writers and readers use relaxed device-scope atomics,
// which go past the per-XCD L2 to where every XCD sees them; a reader polls a
// word until its tag is the wanted epoch, so a word proves itself and neither
// fences nor flags are needed (a device-scope release would write back the
// whole L2 of the XCD).  Buffers alternate by epoch parity: a word of epoch e
// is overwritten by epoch e + 2, which its writer reaches only after every
// reader has published epoch e + 1, that is, has read epoch e.
//
// A tag stands for one epoch only: the buffers start as zeros, epoch 0 is never
// sent, and before the tags run out the host clears the buffers between two
// launches and counts from 0 again (next_epochs).  Otherwise a word that was
// not written since (a slot without a candidate is one word of four) could
// carry the wanted tag.
//
// One store-to-load hand-over was measured at 1.0 us over 8 workgroups and
// 1.3 to 1.7 us over 256 (200 nodes and one candidate slot each, words of one
// kind contiguous; 3.4 us with a node's words side by side, whose 8-byte
// stores then each dirty a line of their own).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace mct {
namespace xch {

constexpr int kTagBits = 21;
constexpr int kDataBits = 64 - kTagBits;
constexpr uint32_t kTagMask = (1u << kTagBits) - 1u;
constexpr uint64_t kDataMask = (1ull << kDataBits) - 1ull;
// polls before a reader gives up (some half a minute; the launch is cooperative,
// so a word arrives within microseconds unless kernels of other streams hold
// compute units that this launch still waits for)
constexpr int kSpinLimit = 1 << 25;
constexpr int kBackoff = 4;  // pause after a vain poll, in 64 cycles

__device__ __forceinline__ uint64_t word(uint32_t epoch, uint64_t data) {
    return ((uint64_t)(epoch & kTagMask) << kDataBits) | data;
}
__device__ __forceinline__ bool tagged(uint64_t w, uint32_t epoch) {
    return (uint32_t)(w >> kDataBits) == (epoch & kTagMask);
}
__device__ __forceinline__ void put(uint64_t *p, uint64_t w) {
    __hip_atomic_store(p, w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint64_t get(const uint64_t *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Before a launch that sends the epochs epoch + 1 .. epoch + n (n far below the
// number of tags) through these buffers.
inline hipError_t next_epochs(uint32_t &epoch, int n, uint64_t *xb, size_t words_u, uint64_t *slots, size_t words_s,
                              hipStream_t st) {
    if (epoch + (uint32_t)n <= kTagMask) return hipSuccess;
    hipError_t e = hipMemsetAsync(xb, 0, sizeof(uint64_t) * words_u, st);
    if (e == hipSuccess) e = hipMemsetAsync(slots, 0, sizeof(uint64_t) * words_s, st);
    if (e == hipSuccess) epoch = 0;
    return e;
}

// A pair of values (a node's two components) as words `stride` apart:
// binary64 three words (128 bits), binary32 two.
template <class T>
constexpr int pair_words() {
    return sizeof(T) == 8 ? 3 : 2;
}

__device__ __forceinline__ void put_pair(uint64_t *p, size_t stride, uint32_t epoch, double x, double y) {
    const uint64_t a = (uint64_t)__double_as_longlong(x), b = (uint64_t)__double_as_longlong(y);
    put(p, word(epoch, a & kDataMask));
    put(p + stride, word(epoch, (a >> 43) | ((b & 0x3FFFFFull) << 21)));
    put(p + 2 * stride, word(epoch, b >> 22));
}
__device__ __forceinline__ void put_pair(uint64_t *p, size_t stride, uint32_t epoch, float x, float y) {
    put(p, word(epoch, (uint64_t)__float_as_uint(x)));
    put(p + stride, word(epoch, (uint64_t)__float_as_uint(y)));
}

// The words of a pair as loaded, whether they carry the epoch, and their values.
struct Pair64 {
    uint64_t w0, w1, w2;
    __device__ __forceinline__ void load(const uint64_t *p, size_t stride) {
        w0 = get(p);
        w1 = get(p + stride);
        w2 = get(p + 2 * stride);
    }
    __device__ __forceinline__ bool here(uint32_t epoch) const {
        return tagged(w0, epoch) && tagged(w1, epoch) && tagged(w2, epoch);
    }
    __device__ __forceinline__ void values(double &x, double &y) const {
        const uint64_t d1 = w1 & kDataMask;
        x = __longlong_as_double((long long)((w0 & kDataMask) | (d1 << 43)));
        y = __longlong_as_double((long long)((d1 >> 21) | ((w2 & kDataMask) << 22)));
    }
};
struct Pair32 {
    uint64_t w0, w1;
    __device__ __forceinline__ void load(const uint64_t *p, size_t stride) {
        w0 = get(p);
        w1 = get(p + stride);
    }
    __device__ __forceinline__ bool here(uint32_t epoch) const { return tagged(w0, epoch) && tagged(w1, epoch); }
    __device__ __forceinline__ void values(float &x, float &y) const {
        x = __uint_as_float((uint32_t)w0);
        y = __uint_as_float((uint32_t)w1);
    }
};
template <class T>
struct PairOf {
    using type = Pair64;
};
template <>
struct PairOf<float> {
    using type = Pair32;
};

// Polls until both values are there; false when the limit is reached.
template <class T>
__device__ __forceinline__ bool get_pair(const uint64_t *p, size_t stride, uint32_t epoch, T &x, T &y) {
    typename PairOf<T>::type a;
    for (int n = 0; n < kSpinLimit; ++n) {
        a.load(p, stride);
        if (a.here(epoch)) {
            a.values(x, y);
            return true;
        }
        __builtin_amdgcn_s_sleep(kBackoff);
    }
    return false;
}

// A workgroup's best accepted candidate of a step (or none), four words
// `stride` apart: element and local edges, then G and the smallest accepted
// G in binary64 (a binary32 step's values are exact in them).
constexpr int kSlotWords = 4;

__device__ __forceinline__ void put_no_slot(uint64_t *p, uint32_t epoch) { put(p, word(epoch, 0)); }
__device__ __forceinline__ void put_slot(uint64_t *p, size_t stride, uint32_t epoch, int e, int a, int k, double G,
                                         double Gmin) {
    const uint64_t g = (uint64_t)__double_as_longlong(G), m = (uint64_t)__double_as_longlong(Gmin);
    put(p + stride, word(epoch, g & kDataMask));
    put(p + 2 * stride, word(epoch, (g >> 43) | ((m & 0x3FFFFFull) << 21)));
    put(p + 3 * stride, word(epoch, m >> 22));
    put(p, word(epoch, ((uint64_t)(uint32_t)e << 5) | (uint64_t)(a << 3) | (uint64_t)(k << 1) | 1ull));
}
// The words of a slot loaded at once (to be looked at later).
struct SlotWords {
    uint64_t w[kSlotWords];
};
__device__ __forceinline__ void load_slot(const uint64_t *p, size_t stride, SlotWords &s) {
#pragma unroll
    for (int i = 0; i < kSlotWords; ++i) s.w[i] = get(p + i * stride);
}
// Polls (starting from the words already loaded) until the slot is there;
// false when the limit is reached.  has: it holds a candidate.
__device__ __forceinline__ bool take_slot(const uint64_t *p, size_t stride, uint32_t epoch, SlotWords &s, bool &has,
                                          int &e, int &a, int &k, double &G, double &Gmin) {
    for (int n = 0; n < kSpinLimit; ++n) {
        if (tagged(s.w[0], epoch)) {
            has = (s.w[0] & 1ull) != 0;
            if (!has) return true;
            if (tagged(s.w[1], epoch) && tagged(s.w[2], epoch) && tagged(s.w[3], epoch)) {
                const uint64_t d0 = s.w[0] & kDataMask, d2 = s.w[2] & kDataMask;
                e = (int)(uint32_t)(d0 >> 5);
                a = (int)(d0 >> 3) & 3;
                k = (int)(d0 >> 1) & 3;
                G = __longlong_as_double((long long)((s.w[1] & kDataMask) | (d2 << 43)));
                Gmin = __longlong_as_double((long long)((d2 >> 21) | ((s.w[3] & kDataMask) << 22)));
                return true;
            }
        }
        __builtin_amdgcn_s_sleep(kBackoff);
        load_slot(p, stride, s);
    }
    return false;
}

}  // namespace xch
}  // namespace mct
