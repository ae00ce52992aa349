// Half a byte per site, eight sites per word: the layout of the kernels that keep
// or copy whole replicas (small3d.hip, bins2d.hip).
//
// Pair h of a replica is the sites (2h, 2h + 1), one of either colour; half-byte h of
// array C_c is its colour-c site: the spin in bit 0 (1: -1) and, for EA, the bonds to
// x + 1, y + 1 and z + 1 in bits 1, 2 and 3 (1: -1).  Word g of C_c then holds the eight
// sites whose heads are Philox block g.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "segment3d.hpp"

namespace smc {
namespace halves {

__device__ __forceinline__ uint32_t pick(uint32_t m, uint32_t one, uint32_t zero) { return (one & m) | (zero & ~m); }

// Bits 0 of eight half-bytes: (a ^ b) & 1, (a ^ b ^ c) & 1.
__device__ __forceinline__ uint32_t x2(uint32_t a, uint32_t b) {
    return __builtin_amdgcn_bitop3_b32(a, b, 0x11111111u, 0x28);
}
__device__ __forceinline__ uint32_t x3(uint32_t a, uint32_t b, uint32_t c) { return x2(a ^ b, c); }

// Eight bytes (each below 16) to half-bytes and back.
__device__ __forceinline__ uint32_t of_bytes(const uint2 &b) {
    return perm(b.y | (b.y >> 4), b.x | (b.x >> 4), 0x06040200u);
}
__device__ __forceinline__ uint2 to_bytes(uint32_t w) {
    const uint32_t e = w & 0x0F0F0F0Fu, o = (w >> 4) & 0x0F0F0F0Fu;
    return make_uint2(perm(o, e, 0x05010400u), perm(o, e, 0x07030602u));
}
// Eight 0/1 bytes to bits 0 of half-bytes.
__device__ __forceinline__ uint32_t flags_of(uint32_t F0, uint32_t F1) {
    return perm(F1, F0, 0x06040200u) | (perm(F1, F0, 0x07050301u) << 4);
}

// Four +-1 bytes as the bits of one place in four half-bytes held in bytes.
__device__ __forceinline__ uint32_t place(uint32_t v, int shift) {
    return shift ? (v << (shift - 1)) & (0x01010101u << shift) : (v >> 1) & 0x01010101u;
}
// Sixteen sites as bytes of half-bytes (spins s, n bond arrays j): the even and the odd
// ones of the pairs as words.
template <int NB>
__device__ __forceinline__ uint2 words_of(const uint4 &s, const uint4 (&j)[NB], int n) {
    uint4 w = make_uint4(place(s.x, 0), place(s.y, 0), place(s.z, 0), place(s.w, 0));
#pragma unroll
    for (int mu = 0; mu < NB; ++mu)
        if (mu < n)
            w = make_uint4(w.x | place(j[mu].x, mu + 1), w.y | place(j[mu].y, mu + 1), w.z | place(j[mu].z, mu + 1),
                           w.w | place(j[mu].w, mu + 1));
    return make_uint2(of_bytes(seg3d::half_of(w, 0x06040200u)), of_bytes(seg3d::half_of(w, 0x07050301u)));
}
// The spins of eight pairs as sixteen +-1 bytes.
__device__ __forceinline__ uint4 spins_of(uint32_t even, uint32_t odd) {
    const uint2 e = to_bytes(even), o = to_bytes(odd);
    auto out = [](uint32_t od, uint32_t ev, uint32_t sel) { return bytes_pm1(perm(od, ev, sel) & 0x01010101u); };
    return make_uint4(out(o.x, e.x, 0x05010400u), out(o.x, e.x, 0x07030602u), out(o.y, e.y, 0x05010400u),
                      out(o.y, e.y, 0x07030602u));
}

}  // namespace halves
}  // namespace smc
