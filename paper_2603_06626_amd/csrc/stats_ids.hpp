// The cached ids of one token in registers, for the routing statistics.
#pragma once
#include "common.hpp"

namespace grouter {

// N >= k ids of a token, N = 4 or 8.  They are fetched with loads of 8 bytes (uint8) or 16 (int32) that need no more than the
// elements' own alignment and take in ids of the tokens behind; at the end of the array the window begins earlier and the ids
// are moved to their places when they are used.  So a fetch is always the same few instructions, without a branch, and several
// can be on their way at a time (one load per id, each under a condition, had the compiler wait for all of them at once).
template <class IdxT, int N>
struct IdWindow;

template <int N>
struct IdWindow<uint8_t, N> {
    static constexpr int kWindow = 8;   // elements that have to exist
    uint32_t w[2];
    int shift;
    // the window that begins at element `at` of base, of which `last` is the last that may begin one (below 0 where fewer than a
    // window's elements are left behind base: it then begins before base)
    __device__ __forceinline__ void fetch(const uint8_t* __restrict__ base, int at, int last) {
        const int from = min(at, last);
        shift = at - from;
        __builtin_memcpy(w, base + from, 8);
    }
    __device__ __forceinline__ void settle() {
        const uint64_t v = (((uint64_t)w[1] << 32) | w[0]) >> (8 * min(shift, 7));
        w[0] = (uint32_t)v;
        w[1] = (uint32_t)(v >> 32);
    }
    __device__ __forceinline__ uint32_t id(int j) const { return (w[j >> 2] >> (8 * (j & 3))) & 0xffu; }
};

template <int N>
struct IdWindow<int32_t, N> {
    static constexpr int kWindow = N;
    typedef uint32_t Quad __attribute__((ext_vector_type(4), aligned(4)));
    Quad q[N / 4];
    int shift;
    __device__ __forceinline__ void fetch(const int32_t* __restrict__ base, int at, int last) {
        const int from = min(at, last);
        shift = at - from;
#pragma unroll
        for (int i = 0; i < N / 4; ++i) q[i] = *reinterpret_cast<const Quad*>(base + from + 4 * i);
    }
    __device__ __forceinline__ void settle() {
        if (__any(shift > 0)) {
#pragma unroll
            for (int by = N / 2; by > 0; by >>= 1)
#pragma unroll
                for (int j = 0; j + by < N; ++j) q[j / 4][j % 4] = (shift & by) ? q[(j + by) / 4][(j + by) % 4] : q[j / 4][j % 4];
        }
    }
    __device__ __forceinline__ uint32_t id(int j) const { return q[j / 4][j % 4]; }
};

}  // namespace grouter
