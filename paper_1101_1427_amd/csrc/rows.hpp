// 16-site pieces of lattice rows of any even edge: loads that stay inside
// the replica, and the end of a row that is not a multiple of 16 sites.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "intrin.hpp"

namespace smc {

// Sixteen bytes at p (any alignment).
__device__ __forceinline__ uint4 load16_any(const int8_t *p) {
    uint4 v;
    __builtin_memcpy(&v, p, 16);
    return v;
}

// The 128 bits of v moved down (towards byte 0) or up by n bytes, 0 <= n <= 16.
__device__ __forceinline__ uint4 bytes_down(const uint4 &v, uint32_t n) {
    const unsigned __int128 w = ((unsigned __int128)(((uint64_t)v.w << 32) | v.z) << 64) | (((uint64_t)v.y << 32) | v.x);
    const unsigned __int128 s = n >= 16 ? 0 : w >> (8 * n);
    return make_uint4((uint32_t)s, (uint32_t)(s >> 32), (uint32_t)(s >> 64), (uint32_t)(s >> 96));
}
__device__ __forceinline__ uint4 bytes_up(const uint4 &v, uint32_t n) {
    const unsigned __int128 w = ((unsigned __int128)(((uint64_t)v.w << 32) | v.z) << 64) | (((uint64_t)v.y << 32) | v.x);
    const unsigned __int128 s = n >= 16 ? 0 : w << (8 * n);
    return make_uint4((uint32_t)s, (uint32_t)(s >> 32), (uint32_t)(s >> 64), (uint32_t)(s >> 96));
}

// The bytes i .. i + 15 of an array of N >= 16; those outside [0, N) come
// back as zeros and are not read.
__device__ __forceinline__ uint4 load16(const int8_t *p, int64_t i, int64_t N) {
    if (__builtin_expect(i >= 0 && i <= N - 16, 1)) return load16_any(p + i);
    if (i < 0) return bytes_up(load16_any(p), (uint32_t)min(-i, (int64_t)16));
    return bytes_down(load16_any(p + (N - 16)), (uint32_t)min(i - (N - 16), (int64_t)16));
}

// Sixteen bytes from site i of an array of N: where i .. i + 15 runs over an
// end of the array the loaded bytes are moved into place by into_place, so that
// several loads can be issued before the first is waited for.
template <typename I>
__device__ __forceinline__ uint4 load_inside(const int8_t *p, I i, I N) {
    return load16_any(p + max((I)0, min(i, N - 16)));
}
template <typename I>
__device__ __forceinline__ void into_place(uint4 &v, I i, I N) {
    if (i < 0) v = bytes_up(v, (uint32_t)min(-i, (I)16));
    if (i > N - 16) v = bytes_down(v, (uint32_t)min(i - (N - 16), (I)16));
}

// The end of a row in a piece of which `left` sites (even, > 0) remain in
// the row; left >= 16: a whole piece.
struct RowEnd {
    uint4 m2;      // 2 in every byte of the row
    uint4 first;   // 0xFF in the byte just past the row's end (none in a whole piece)
    bool partial;

    __device__ __forceinline__ explicit RowEnd(int left) {
        partial = left < 16;
        const uint4 two = make_uint4(0x02020202u, 0x02020202u, 0x02020202u, 0x02020202u);
        if (!partial) {
            m2 = two;
            first = make_uint4(0u, 0u, 0u, 0u);
        } else {
            m2 = bytes_down(two, (uint32_t)(16 - left));
            first = bytes_up(make_uint4(0xFFu, 0u, 0u, 0u), (uint32_t)left);
        }
    }

    // Byte k of the result is site k + 1 of the row, xr being the site after
    // the last one of the piece (periodic).
    __device__ __forceinline__ uint4 shifted_down(const uint4 &v, uint32_t xr) const {
        const uint32_t rep = xr * 0x01010101u;
        auto put = [&](uint32_t w, uint32_t m) { return (w & ~m) | (rep & m); };
        const uint4 w = make_uint4(put(v.x, first.x), put(v.y, first.y), put(v.z, first.z), put(v.w, first.w));
        return make_uint4(alignbyte(w.y, w.x, 1), alignbyte(w.z, w.y, 1), alignbyte(w.w, w.z, 1),
                          (w.w >> 8) | (xr << 24));
    }
};

}  // namespace smc
