// Half-sweeps of uniform 3D Ising / +-J EA batches on a packed copy of the
// lattice (Eq. 2 on the simple cubic lattice): half a byte per site.
//
// Byte h of a replica is the pair of sites (2h, 2h + 1): the even site in the
// low four bits, the odd one in the high four, each with its spin in bit 0 and
// (EA) its bonds to x + 1, y + 1 and z + 1 in bits 1, 2 and 3 (1: -1).  A call
// packs its lattices once, runs all its half-sweeps in place on the copy and
// unpacks the spins.  A half-sweep then reads no couplings and moves a byte per
// update instead of five, its operands need no splitting into even and odd
// sites, and the bond of a neighbour pair comes with the spins.
//
// A thread owns pieces of eight pairs, bytes 8 g .. 8 g + 7: their colour-c sites
// are the in-colour indices of Philox block g.  The y and z neighbours of a
// pair lie L / 2 and L^2 / 2 bytes away, in the same half of the byte.
//
// Edges that are multiples of 16 (k_pairs3d_half): a piece lies in one row, and
// a workgroup takes rows of one parity, so which half of its bytes it
// updates is fixed at compile time; a thread walks a few planes in z and keeps
// its column in registers.  Other edges (k_pairs3d_half_ragged): a piece may
// hold the end of one row and the start of the next (at most two rows, the
// edge being at least 16); byte masks merge what differs between them.
//
// Bound: VALU, about 19 lane-operations per update (the kernel on the caller's
// bytes needs 30 to 37), and launches where the batch is small.
// Per sweep, against the kernels on bytes: EA 256^3 24.0 -> 18.0 us, EA 384^3
// 70 -> 47, EA 512^3 143 -> 98, Ising 256^3 22.0 -> 17.7, four of 100^3 18.4 -> 13.9,
// 64 EA of 18^3 13.0 -> 8.8.
#include "pairs3d.hpp"

#include <stdlib.h>

#include <type_traits>

#include "rows.hpp"
#include "segment3d.hpp"

namespace smc {
namespace {

using namespace seg3d;

constexpr int kThreads = 256;

struct KArgs {
    Pairs3dArgs b;
    Tally tally;
    int64_t stride;  // bytes per replica
    int groups;      // workgroups per replica
    uint32_t one2;   // 0x00010001, opaque to the compiler
};

__host__ __device__ inline int64_t stride_of(int L) {
    const int64_t half = (int64_t)L * L * L / 2;
    return (half + 15) / 16 * 16;
}

// Bits 0 of four bytes: (a ^ b) & 1, (a ^ b ^ c) & 1.
__device__ __forceinline__ uint32_t x2(uint32_t a, uint32_t b) {
    return __builtin_amdgcn_bitop3_b32(a, b, 0x01010101u, 0x28);
}
__device__ __forceinline__ uint32_t x3(uint32_t a, uint32_t b, uint32_t c) { return x2(a ^ b, c); }

// Unsatisfied bonds of four own sites: o own, u and v the sites at x + 1 and
// x - 1, yp .. zm the other neighbours, each with its site in the low half of
// the bytes (the high halves may hold anything).
template <bool EA>
__device__ __forceinline__ uint32_t unsatisfied(uint32_t o, uint32_t u, uint32_t v, uint32_t yp, uint32_t ym,
                                                uint32_t zp, uint32_t zm) {
    if constexpr (EA)
        return x3(o, u, o >> 1) + x3(o, v, v >> 1) + x3(o, yp, o >> 2) + x3(o, ym, ym >> 2) + x3(o, zp, o >> 3) +
               x3(o, zm, zm >> 3);
    else
        return x2(o, u) + x2(o, v) + x2(o, yp) + x2(o, ym) + x2(o, zp) + x2(o, zm);
}

// The decisions of a piece from its counts (o.n0, o.n1): flip flags in o.F0, o.F1.
__device__ __forceinline__ void decide(RowOut &o, uint32_t g, uint32_t c, uint32_t r, const ThrRow &th, const Lut3 &K,
                                       const KArgs &a) {
    const uint4 w = philox4x32_10(make_uint4(g, a.b.t, r, 2 * kTagHead + c), a.b.key);
    uint32_t eq = 0xFFFFFFFFu;
    o.F0 = decide4(o.n0, w.x, w.y, K, a.one2, eq);
    o.F1 = decide4(o.n1, w.z, w.w, K, a.one2, eq);
    if (__builtin_expect(__any(has_tie(eq)), 0)) exact_decisions(o, w, th, K, 8u * g, c, a.b.t, r, a.b.key, has_tie(eq));
}

__device__ __forceinline__ void tally_flips(const RowOut &o, uint32_t &cnt, uint32_t &nsum) {
    cnt = __builtin_amdgcn_sad_u8(o.F0, 0u, __builtin_amdgcn_sad_u8(o.F1, 0u, cnt));
    nsum = __builtin_amdgcn_sad_u8(o.n0 & bytes_ff(o.F0), 0u, __builtin_amdgcn_sad_u8(o.n1 & bytes_ff(o.F1), 0u, nsum));
}

// Delta E of a flip with n unsatisfied bonds is 4 (3 - n).
__device__ __forceinline__ void put_tally(const KArgs &a, int64_t group, int r, uint32_t cnt, uint32_t nsum, int *red) {
    if (!tally_wanted(a.tally)) return;
    int d = 3 * (int)cnt - (int)nsum;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) d += __shfl_xor(d, o, 64);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = d;
    __syncthreads();
    if (threadIdx.x == 0) tally_put(a.tally, group, r, 4ll * (red[0] + red[1] + red[2] + red[3]));
}

__device__ __forceinline__ uint2 ld8(const uint8_t *p, uint32_t i) {
    return *(const uint2 *)__builtin_assume_aligned(p + i, 8);
}
__device__ __forceinline__ uint2 shift4(const uint2 &v) { return make_uint2(v.x >> 4, v.y >> 4); }

// One piece of row (y, z), own sites in half A of its bytes: p its bytes, zm and
// zp those of the planes beside it; returns its new bytes.
template <bool EA, int A>
__device__ __forceinline__ uint2 piece(const uint8_t *S, const uint2 &p, const uint2 &zm, const uint2 &zp, uint32_t at,
                                       uint32_t y_up, uint32_t y_down, uint32_t beside, uint32_t g, uint32_t c,
                                       uint32_t r, const ThrRow &th, const Lut3 &K, const KArgs &a, uint32_t &cnt,
                                       uint32_t &nsum) {
    const uint2 yp = ld8(S, at + y_up), ym = ld8(S, at + y_down);
    const uint32_t ext = S[beside];  // the pair after the piece (own sites odd) or before it (even)
    // the pairs at distance one in x: their even sites at x + 1, or odd ones at x - 1
    uint2 side;
    if constexpr (A)
        side = make_uint2(alignbyte(p.y, p.x, 1), alignbyte(ext, p.y, 1));
    else
        side = shift4(make_uint2((p.x << 8) | ext, alignbyte(p.y, p.x, 3)));
    const uint2 q = shift4(p);
    const uint2 o = A ? q : p, partner = A ? p : q, u = A ? side : partner, v = A ? partner : side;
    auto half = [](const uint2 &n) { return A ? shift4(n) : n; };
    const uint2 yph = half(yp), ymh = half(ym), zph = half(zp), zmh = half(zm);
    RowOut out;
    out.n0 = unsatisfied<EA>(o.x, u.x, v.x, yph.x, ymh.x, zph.x, zmh.x);
    out.n1 = unsatisfied<EA>(o.y, u.y, v.y, yph.y, ymh.y, zph.y, zmh.y);
    decide(out, g, c, r, th, K, a);
    tally_flips(out, cnt, nsum);
    return make_uint2(p.x ^ (out.F0 << (4 * A)), p.y ^ (out.F1 << (4 * A)));
}

// Edges that are multiples of 16.  The first half of a replica's workgroups
// takes the columns whose first row has y + z even, the second half the others;
// Z planes per thread.
template <bool EA, int Z>
__global__ __launch_bounds__(kThreads) void k_pairs3d_half(KArgs a, int c) {
    __shared__ int red[kThreads / 64];
    const uint32_t L = (uint32_t)a.b.L, K8 = L / 16, Lh = L / 2, P = L * Lh;  // pieces and bytes per row, bytes per plane
    const int r = (int)(blockIdx.x / (uint32_t)a.groups);
    const uint32_t group = blockIdx.x - (uint32_t)r * (uint32_t)a.groups, half = (uint32_t)a.groups / 2;
    const uint32_t par = group >= half ? 1u : 0u;
    const uint32_t idx = (group - par * half) * kThreads + threadIdx.x;
    const int row = a.b.row_of_rep ? a.b.row_of_rep[r] : r;
    uint32_t cnt = 0, nsum = 0;
    if (row >= 0 && idx < K8 * Lh * (L / Z)) {
        uint8_t *S = a.b.packed + (int64_t)r * a.stride;
        const uint32_t k = idx % K8, yz = idx / K8, zq = yz / Lh, z0 = zq * Z;
        const uint32_t y = 2 * (yz - zq * Lh) + ((z0 + par) & 1u);
        const uint32_t rr = (uint32_t)r >> a.b.rng_shift;
        const ThrRow th = a.b.thr[row];
        const Lut3 K = lut_of(th);
        uint32_t at = z0 * P + y * Lh + 8 * k;  // byte of the piece
        const uint32_t y_up = y == L - 1 ? 0u - (P - Lh) : Lh, y_down = y == 0 ? P - Lh : 0u - Lh;
        const uint32_t next = k == K8 - 1 ? 8u - Lh : 8u, prev = k == 0 ? Lh - 1u : 0u - 1u;  // relative to the piece
        uint2 below = ld8(S, z0 == 0 ? at + P * (L - 1) : at - P), here = ld8(S, at);
        auto run = [&](auto first) {
            constexpr int A0 = decltype(first)::value;  // half of the own sites in plane z0
#pragma unroll
            for (int j = 0; j < Z; ++j) {
                const uint32_t up = z0 + j == L - 1 ? at - P * (L - 1) : at + P;
                const uint2 above = ld8(S, up);
                constexpr int kOdd = 1;
                uint2 now;
                const uint32_t g = at >> 3;
                if ((A0 + j) & 1)
                    now = piece<EA, kOdd>(S, here, below, above, at, y_up, y_down, at + next, g, (uint32_t)c, rr, th, K,
                                          a, cnt, nsum);
                else
                    now = piece<EA, 0>(S, here, below, above, at, y_up, y_down, at + prev, g, (uint32_t)c, rr, th, K, a,
                                       cnt, nsum);
                if ((now.x ^ here.x) | (now.y ^ here.y)) *(uint2 *)__builtin_assume_aligned(S + at, 8) = now;
                // (only the other colour's halves are read from the plane below)
                below = here;
                here = above;
                at = up;
            }
        };
        if ((par ^ (uint32_t)c) & 1u)
            run(std::integral_constant<int, 1>{});
        else
            run(std::integral_constant<int, 0>{});
    }
    put_tally(a, blockIdx.x, r, cnt, nsum, red);
}

__device__ __forceinline__ uint2 ld8_any(const uint8_t *p, int64_t i) {
    uint2 v;
    __builtin_memcpy(&v, p + i, 8);
    return v;
}
__device__ __forceinline__ uint2 pick(const uint2 &m, const uint2 &one, const uint2 &zero) {
    return make_uint2((one.x & m.x) | (zero.x & ~m.x), (one.y & m.y) | (zero.y & ~m.y));
}
__device__ __forceinline__ uint2 to_u2(uint64_t v) { return make_uint2((uint32_t)v, (uint32_t)(v >> 32)); }

// Any even edge from 16; a piece of row 1 (pairs below `b`) and row 2 (the others).
template <bool EA>
__global__ __launch_bounds__(kThreads) void k_pairs3d_half_ragged(KArgs a, int c) {
    __shared__ int red[kThreads / 64];
    const int L = a.b.L, Lh = L / 2, P = L * Lh, H = P * L;  // bytes per row, plane and replica
    const int r = (int)(blockIdx.x / (uint32_t)a.groups);
    const int g = (int)(blockIdx.x - (uint32_t)r * (uint32_t)a.groups) * kThreads + (int)threadIdx.x;
    const int row = a.b.row_of_rep ? a.b.row_of_rep[r] : r;
    uint32_t cnt = 0, nsum = 0;
    const int h0 = 8 * g;
    if (row >= 0 && h0 < H) {
        uint8_t *S = a.b.packed + (int64_t)r * a.stride;
        const int n = min(8, H - h0);  // pairs of the piece (4 or 8)
        const int q = (int)((uint32_t)h0 / (uint32_t)Lh), left = Lh - (h0 - q * Lh), b = min(left, 8);
        const bool border = left < n;  // the piece holds pairs of two rows
        const int z1 = (int)((uint32_t)q / (uint32_t)L), y1 = q - z1 * L;
        int y2 = y1, z2 = z1;
        if (left < 8) {
            y2 = y1 == L - 1 ? 0 : y1 + 1;
            z2 = y1 == L - 1 ? z1 + 1 : z1;
        }
        auto off = [&](int k, int y, int z) -> int {
            if (k == 0) return y == L - 1 ? Lh - P : Lh;
            if (k == 1) return y == 0 ? P - Lh : -Lh;
            if (k == 2) return z == L - 1 ? P - H : P;
            return z == 0 ? H - P : -P;
        };
        // loads of the ordinary case (eight bytes may run past the replica's
        // ends into its neighbours or the pads; what is not used is masked)
        int d1[4];
        uint2 nb[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            d1[k] = off(k, y1, z1);
            nb[k] = ld8_any(S, max(h0 + d1[k], -8));
        }
        const uint2 p = ld8(S, (uint32_t)h0);
        uint32_t before = S[left == Lh ? h0 + Lh - 1 : h0 - 1];       // first pair's row neighbour
        uint32_t after = S[left == 8 ? h0 + 8 - Lh : h0 + 8];           // last pair's
        const uint64_t second = b >= 8 ? 0ull : ~0ull << (8 * b);
        uint64_t up = (((uint64_t)p.y << 32) | p.x) << 8 | before;
        uint64_t down = ((((uint64_t)p.y << 32) | p.x) >> 8) | ((uint64_t)after << 56);
        if (left < 8) {
            // ends of the two rows: periodic neighbours
            const uint64_t m1 = 0xFFull << (8 * (left - 1));
            down = (down & ~m1) | ((uint64_t)S[h0 + left - Lh] << (8 * (left - 1)));
            if (border) {
                const uint64_t m2 = 0xFFull << (8 * left);
                up = (up & ~m2) | ((uint64_t)S[h0 + left + Lh - 1] << (8 * left));
                const uint2 m = to_u2(second);
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const int d2 = off(k, y2, z2);
                    if (d2 != d1[k]) nb[k] = pick(m, ld8_any(S, max(h0 + d2, -8)), nb[k]);
                }
            }
        }
        const bool A1 = (((y1 + z1) & 1) ^ c) != 0, A2 = (((y2 + z2) & 1) ^ c) != 0;
        const uint2 odd = to_u2((A1 ? ~second : 0ull) | (A2 ? second : 0ull));
        const uint2 ps = shift4(p), o = pick(odd, ps, p), partner = pick(odd, p, ps);
        const uint2 side = pick(odd, to_u2(down), shift4(to_u2(up)));
        const uint2 u = pick(odd, side, partner), v = pick(odd, partner, side);
        uint2 mine[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) mine[k] = pick(odd, shift4(nb[k]), nb[k]);
        const uint32_t rr = (uint32_t)r >> a.b.rng_shift;
        const ThrRow th = a.b.thr[row];
        const Lut3 K = lut_of(th);
        RowOut out;
        out.n0 = unsatisfied<EA>(o.x, u.x, v.x, mine[0].x, mine[1].x, mine[2].x, mine[3].x);
        out.n1 = unsatisfied<EA>(o.y, u.y, v.y, mine[0].y, mine[1].y, mine[2].y, mine[3].y);
        decide(out, (uint32_t)g, (uint32_t)c, rr, th, K, a);
        if (n < 8) out.F1 = 0u;
        tally_flips(out, cnt, nsum);
        if (out.F0 | out.F1) {
            const uint2 f = pick(odd, make_uint2(out.F0 << 4, out.F1 << 4), make_uint2(out.F0, out.F1));
            *(uint2 *)__builtin_assume_aligned(S + h0, 8) = make_uint2(p.x ^ f.x, p.y ^ f.y);
        }
    }
    put_tally(a, blockIdx.x, r, cnt, nsum, red);
}

// Row-major +-1 bytes (and bonds) to packed pairs, and the spins back.
template <bool EA>
__global__ __launch_bounds__(kThreads) void k_pairs3d_pack(const int8_t *spins, const int8_t *coup, KArgs a) {
    const int64_t N = (int64_t)a.b.L * a.b.L * a.b.L;
    const int r = (int)(blockIdx.x / (uint32_t)a.groups);
    const int64_t i = 16 * ((int64_t)(blockIdx.x - (uint32_t)r * (uint32_t)a.groups) * kThreads + threadIdx.x);
    if (i >= N) return;
    uint4 s = load_inside<int64_t>(spins + (int64_t)r * N, i, N), j[3];
    const int8_t *J = nullptr;
    if constexpr (EA) {
        J = coup + (int64_t)(r / a.b.rep_per_sample) * 3 * N;
#pragma unroll
        for (int mu = 0; mu < 3; ++mu) j[mu] = load_inside<int64_t>(J + mu * N, i, N);
    }
    if (__builtin_expect(i > N - 16, 0)) {
        into_place<int64_t>(s, i, N);
        if constexpr (EA)
#pragma unroll
            for (int mu = 0; mu < 3; ++mu) into_place<int64_t>(j[mu], i, N);
    }
    auto word = [](uint32_t v, uint32_t x, uint32_t y, uint32_t z) -> uint32_t {
        uint32_t w = (v >> 1) & 0x01010101u;
        if constexpr (EA) w |= (x & 0x02020202u) | ((y << 1) & 0x04040404u) | ((z << 2) & 0x08080808u);
        return w;
    };
    const uint4 w = make_uint4(word(s.x, j[0].x, j[1].x, j[2].x), word(s.y, j[0].y, j[1].y, j[2].y),
                               word(s.z, j[0].z, j[1].z, j[2].z), word(s.w, j[0].w, j[1].w, j[2].w));
    const uint2 e = half_of(w, 0x06040200u), o = half_of(w, 0x07050301u);
    *(uint2 *)__builtin_assume_aligned(a.b.packed + (int64_t)r * a.stride + i / 2, 8) =
        make_uint2(e.x | (o.x << 4), e.y | (o.y << 4));
}

__global__ __launch_bounds__(kThreads) void k_pairs3d_unpack(int8_t *spins, KArgs a) {
    const int64_t N = (int64_t)a.b.L * a.b.L * a.b.L;
    const int r = (int)(blockIdx.x / (uint32_t)a.groups);
    const int64_t i = 16 * ((int64_t)(blockIdx.x - (uint32_t)r * (uint32_t)a.groups) * kThreads + threadIdx.x);
    if (i >= N) return;
    const uint2 e = *(const uint2 *)__builtin_assume_aligned(a.b.packed + (int64_t)r * a.stride + i / 2, 8);
    const uint2 o = shift4(e);
    auto word = [](uint32_t od, uint32_t ev, uint32_t sel) { return bytes_pm1(perm(od, ev, sel) & 0x01010101u); };
    const uint4 w = make_uint4(word(o.x, e.x, 0x05010400u), word(o.x, e.x, 0x07030602u), word(o.y, e.y, 0x05010400u),
                               word(o.y, e.y, 0x07030602u));
    int8_t *out = spins + (int64_t)r * N + i;
    if (i <= N - 16)
        __builtin_memcpy(out, &w, 16);
    else  // N is a multiple of 8
        __builtin_memcpy(out, &w, 8);
}

KArgs kargs(const Pairs3dArgs &b, int groups) {
    KArgs a;
    a.b = b;
    a.tally = Tally{};
    a.stride = stride_of(b.L);
    a.groups = groups;
    a.one2 = 0x00010001u;
    return a;
}

int piece_groups(int L) {
    const int64_t pieces = ((int64_t)L * L * L + 15) / 16;
    return (int)((pieces + kThreads - 1) / kThreads);
}

}  // namespace

bool pairs3d_supported(int dim, int L) { return dim == 3 && L >= 16 && L <= 1024 && L % 2 == 0; }

size_t pairs3d_bytes(int L, int n_rep) { return (size_t)n_rep * (size_t)stride_of(L) + 2 * pairs3d_pad(); }

int pairs3d_planes(int L, int n_rep) {
    if (L % 16) return 1;
    if (const char *e = getenv("SPINMC_PAIRS3D_PLANES")) {
        const int z = atoi(e);
        if (z == 1 || z == 2 || z == 4) return z;
    }
    const int64_t sites = (int64_t)n_rep * L * L * L;
    return sites >= (int64_t)1 << 23 ? 4 : sites >= (int64_t)1 << 21 ? 2 : 1;
}

int pairs3d_groups(int L, int planes) {
    if (L % 16) return piece_groups(L);
    const int64_t threads = (int64_t)(L / 16) * (L / 2) * (L / planes);  // per parity
    return 2 * (int)((threads + kThreads - 1) / kThreads);
}

hipError_t launch_pairs3d_pack(const int8_t *spins, const int8_t *coup, const Pairs3dArgs &b, hipStream_t s) {
    if (!pairs3d_supported(3, b.L) || b.n_rep < 1 || b.rep_per_sample < 1) return hipErrorInvalidValue;
    const KArgs a = kargs(b, piece_groups(b.L));
    const int64_t blocks = (int64_t)a.groups * b.n_rep;
    if (const char *why = launch_config_error((uint64_t)blocks, kThreads, 0))
        return reject_launch("k_pairs3d_pack", (uint64_t)blocks, kThreads, 0, why);
    if (coup)
        SMC_LAUNCH(k_pairs3d_pack<true>, dim3((unsigned)blocks), dim3(kThreads), 0, s, spins, coup, a);
    else
        SMC_LAUNCH(k_pairs3d_pack<false>, dim3((unsigned)blocks), dim3(kThreads), 0, s, spins, coup, a);
    return hipGetLastError();
}

hipError_t launch_pairs3d_unpack(int8_t *spins, const Pairs3dArgs &b, hipStream_t s) {
    const KArgs a = kargs(b, piece_groups(b.L));
    const int64_t blocks = (int64_t)a.groups * b.n_rep;
    SMC_LAUNCH(k_pairs3d_unpack, dim3((unsigned)blocks), dim3(kThreads), 0, s, spins, a);
    return hipGetLastError();
}

hipError_t launch_pairs3d_half(const Pairs3dArgs &b, bool ea, int c, int planes, const Tally &tally, hipStream_t s) {
    if (!pairs3d_supported(3, b.L) || b.n_rep < 1 || b.L % planes) return hipErrorInvalidValue;
    KArgs a = kargs(b, pairs3d_groups(b.L, planes));
    a.tally = tally;
    const int64_t blocks = (int64_t)a.groups * b.n_rep;
    if (const char *why = launch_config_error((uint64_t)blocks, kThreads, 0))
        return reject_launch("k_pairs3d_half", (uint64_t)blocks, kThreads, 0, why);
    const dim3 grid((unsigned)blocks);
    if (b.L % 16) {
        if (ea)
            SMC_LAUNCH(k_pairs3d_half_ragged<true>, grid, dim3(kThreads), 0, s, a, c);
        else
            SMC_LAUNCH(k_pairs3d_half_ragged<false>, grid, dim3(kThreads), 0, s, a, c);
        return hipGetLastError();
    }
#define SMC_PAIRS(EE, ZZ)                                                                       \
    if (ea == EE && planes == ZZ) {                                                             \
        SMC_LAUNCH((k_pairs3d_half<EE, ZZ>), grid, dim3(kThreads), 0, s, a, c);                 \
        return hipGetLastError();                                                               \
    }
    SMC_PAIRS(false, 1)
    SMC_PAIRS(false, 2)
    SMC_PAIRS(false, 4)
    SMC_PAIRS(true, 1)
    SMC_PAIRS(true, 2)
    SMC_PAIRS(true, 4)
#undef SMC_PAIRS
    return hipErrorInvalidValue;
}

}  // namespace smc
