// Half-sweeps of uniform 3D Ising / +-J EA batches on a packed copy of the
// lattice (Eq. 2 on the simple cubic lattice): half a byte per site, the two
// colours apart, eight sites per word (halves.hpp).
//
// A call packs its lattices once, runs all its half-sweeps in place on the copy and
// unpacks the spins.  A half-sweep writes one array and reads its neighbours
// from the other and no couplings: 0.75 bytes per site (0.76 measured at EA 512^3), 1.5
// per update, where the kernels on the caller's bytes move five and more; a Philox block's
// eight sites and each of their neighbours are one word, and the bond of a neighbour pair comes with the spins.
//
// Edges that are multiples of 16 (k_pairs3d_half): a word lies in one row; a thread
// takes the words of a few planes in z, all of them loaded before the first
// wait (the other array is not written, so nothing orders them).  Other edges
// (k_pairs3d_half_ragged): a word may hold the end of one row and the start of the next
// (at most two rows, the edge being at least 16); neighbours are shifted into place
// from two words, and masks merge what differs between the rows.
//
// Bound: VALU, and launches where the batch is small.
// Instructions per word: about 110 (130 where rows end inside words), 57 of them the
// Philox block; an array of pairs as bytes took 150, and read twice the bytes.
// Per sweep, on the caller's bytes, on pairs as bytes and now: EA 256^3 24.0 18.0 15.3 us,
// EA 384^3 70 47 39, EA 512^3 143 98 82, four Ising 100^3 18.4 13.9 10.9.  The XCD order
// of the workgroups is worth 3 % at 256^3 and 8 % at four of 100^3.
#include "pairs3d.hpp"

#include <stdlib.h>

#include "halves.hpp"
#include "rows.hpp"

namespace smc {
namespace {

using namespace seg3d;
using namespace halves;

constexpr int kThreads = 256;
constexpr int kMargin = 4;  // words before and after an array: reads beside a word stay inside

struct KArgs {
    Pairs3dArgs b;
    Tally tally;
    int words;       // words of an array
    int64_t span;    // words of an array with its margins
    int groups;      // workgroups per replica
    uint32_t blocks; // workgroups of the launch (gridDim would bring 256 bytes of hidden arguments, 0.35 us per launch)
    uint32_t one2;   // 0x00010001, opaque to the compiler
};

int words_in(int L) { return (int)(((int64_t)L * L * L + 15) / 16); }
int64_t span_of(int L) { return ((int64_t)words_in(L) + 3) / 4 * 4 + 2 * kMargin; }

__device__ __forceinline__ uint32_t *array_of(const KArgs &a, int r, int c) {
    return a.b.packed + (2 * (int64_t)r + c) * a.span + kMargin;
}

// Consecutive workgroups of a half-sweep on one XCD (the hardware deals them out in
// turn): rows and planes beside a workgroup's are then in the L2 that its neighbours fill.
__device__ __forceinline__ uint32_t block_of(const KArgs &a) {
    const uint32_t n = a.blocks, b = blockIdx.x, x = b & 7u, per = n >> 3, over = n & 7u;
    return x * per + min(x, over) + (b >> 3);
}

// Unsatisfied bonds of a word: own sites, their partners, the other x neighbours and
// those at y +- 1 and z +- 1; odd where the own sites are the odd ones.
template <bool EA>
__device__ __forceinline__ uint32_t unsatisfied(uint32_t odd, uint32_t own, uint32_t par, uint32_t side, uint32_t yp,
                                                uint32_t ym, uint32_t zp, uint32_t zm) {
    if constexpr (EA) {
        // bond of the pair itself: the even site's; of the side pair: the lower site's
        const uint32_t jp = pick(odd, par, own), js = pick(odd, own, side);
        return x3(own, par, jp >> 1) + x3(own, side, js >> 1) + x3(own, yp, own >> 2) + x3(own, ym, ym >> 2) +
               x3(own, zp, own >> 3) + x3(own, zm, zm >> 3);
    } else {
        return x2(own, par) + x2(own, side) + x2(own, yp) + x2(own, ym) + x2(own, zp) + x2(own, zm);
    }
}

// Flips (bit 0 of each half-byte) of word g with n unsatisfied bonds.
__device__ __forceinline__ uint32_t decide(uint32_t n, uint32_t g, uint32_t c, uint32_t r, const ThrRow &th,
                                           const Lut3 &K, const KArgs &a) {
    const uint4 w = philox4x32_10(make_uint4(g, a.b.t, r, 2 * kTagHead + c), a.b.key);
    const uint2 by = to_bytes(n);
    RowOut o;
    o.n0 = by.x;
    o.n1 = by.y;
    uint32_t eq = 0xFFFFFFFFu;
    o.F0 = decide4(o.n0, w.x, w.y, K, a.one2, eq);
    o.F1 = decide4(o.n1, w.z, w.w, K, a.one2, eq);
    if (__builtin_expect(__any(has_tie(eq)), 0)) exact_decisions(o, w, th, K, 8u * g, c, a.b.t, r, a.b.key, has_tie(eq));
    return flags_of(o.F0, o.F1);
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

// Edges that are multiples of 16; Z planes per thread.
template <bool EA, int Z>
__global__ __launch_bounds__(kThreads) void k_pairs3d_half(KArgs a, int c) {
    __shared__ int red[kThreads / 64];
    const uint32_t L = (uint32_t)a.b.L, K = L / 16, P = L * K;  // words per row and plane
    const uint32_t block = block_of(a);
    const int r = (int)(block / (uint32_t)a.groups);
    const uint32_t idx = (block - (uint32_t)r * (uint32_t)a.groups) * kThreads + threadIdx.x;
    const int row = a.b.row_of_rep ? a.b.row_of_rep[r] : r;
    uint32_t cnt = 0, nsum = 0;
    if (row >= 0 && idx < P * (L / Z)) {
        uint32_t *__restrict__ const mine = array_of(a, r, c);
        const uint32_t *__restrict__ const other = array_of(a, r, 1 - c);
        const uint32_t yz = idx / K, k = idx - yz * K, zq = yz / L, y = yz - zq * L, z0 = zq * Z;
        const uint32_t g0 = z0 * P + y * K + k;
        const uint32_t up = y == L - 1 ? K - P : K, down = y == 0 ? P - K : 0u - K;
        const uint32_t next = k == K - 1 ? 1u - K : 1u, prev = k == 0 ? K - 1u : 0u - 1u;
        const bool odd0 = ((y + z0 + (uint32_t)c) & 1u) != 0u;
        uint32_t own[Z], yp[Z], ym[Z], beside[Z], col[Z + 2];
        col[0] = other[z0 == 0 ? g0 + P * (L - 1) : g0 - P];
        col[Z + 1] = other[z0 + Z == L ? y * K + k : g0 + Z * P];
#pragma unroll
        for (int j = 0; j < Z; ++j) {
            const uint32_t g = g0 + j * P;
            own[j] = mine[g];
            col[j + 1] = other[g];
            yp[j] = other[g + up];
            ym[j] = other[g + down];
            beside[j] = other[g + ((j & 1) != (int)odd0 ? next : prev)];
        }
        const uint32_t rr = (uint32_t)r >> a.b.rng_shift;
        const ThrRow th = a.b.thr[row];
        const Lut3 lut = lut_of(th);
#pragma unroll
        for (int j = 0; j < Z; ++j) {
            const bool odd = (j & 1) != (int)odd0;
            const uint32_t g = g0 + j * P, par = col[j + 1];
            const uint32_t side =
                __builtin_amdgcn_alignbit(odd ? beside[j] : par, odd ? par : beside[j], odd ? 4u : 28u);
            const uint32_t n =
                unsatisfied<EA>(odd ? ~0u : 0u, own[j], par, side, yp[j], ym[j], col[j + 2], col[j]);
            const uint32_t f = decide(n, g, (uint32_t)c, rr, th, lut, a);
            if (f) mine[g] = own[j] ^ f;
            cnt += (uint32_t)__builtin_popcount(f);
            nsum = __builtin_amdgcn_udot8(n, f, nsum, false);
        }
    }
    put_tally(a, block, r, cnt, nsum, red);
}

// Where the pairs of word g lie in a lattice of edge L: pairs below `left` in row
// (y1, z1), the others in (y2, z2).
struct Place {
    int left, y1, z1, y2, z2;
    uint32_t second;  // mask of the pairs of the second row
    __device__ __forceinline__ Place(int g, int L) {
        const int Lh = L / 2, h0 = 8 * g, q = (int)((uint32_t)h0 / (uint32_t)Lh);
        left = Lh - (h0 - q * Lh);
        z1 = (int)((uint32_t)q / (uint32_t)L);
        y1 = q - z1 * L;
        y2 = y1 == L - 1 ? 0 : y1 + 1;
        z2 = y1 == L - 1 ? z1 + 1 : z1;
        second = left >= 8 ? 0u : ~0u << (4 * left);
    }
    // Mask of the pairs whose colour-c site is the odd one.
    __device__ __forceinline__ uint32_t odd(uint32_t c) const {
        const bool o1 = (((uint32_t)(y1 + z1) ^ c) & 1u) != 0u, o2 = (((uint32_t)(y2 + z2) ^ c) & 1u) != 0u;
        return (o1 ? ~second : 0u) | (o2 ? second : 0u);
    }
};

// Any even edge from 16.
template <bool EA>
__global__ __launch_bounds__(kThreads) void k_pairs3d_half_ragged(KArgs a, int c) {
    __shared__ int red[kThreads / 64];
    const int L = a.b.L, Lh = L / 2, P = L * Lh, H = P * L;  // pairs per row, plane and replica
    const uint32_t block = block_of(a);
    const int r = (int)(block / (uint32_t)a.groups);
    const int g = (int)(block - (uint32_t)r * (uint32_t)a.groups) * kThreads + (int)threadIdx.x;
    const int row = a.b.row_of_rep ? a.b.row_of_rep[r] : r;
    uint32_t cnt = 0, nsum = 0;
    if (row >= 0 && g < a.words) {
        uint32_t *__restrict__ const mine = array_of(a, r, c);
        const uint32_t *__restrict__ const other = array_of(a, r, 1 - c);
        const int h0 = 8 * g, n_pairs = min(8, H - h0);  // 4 or 8
        const Place w(g, L);
        auto off = [&](int k, int y, int z) -> int {
            if (k == 0) return y == L - 1 ? Lh - P : Lh;
            if (k == 1) return y == 0 ? P - Lh : -Lh;
            if (k == 2) return z == L - 1 ? P - H : P;
            return z == 0 ? H - P : -P;
        };
        // the eight half-bytes d pairs away (of those that run past the arrays' ends none is used)
        auto load2 = [&](int d) -> uint2 { return make_uint2(other[g + (d >> 3)], other[g + (d >> 3) + 1]); };
        auto shifted = [](const uint2 &v, int d) -> uint32_t {
            return __builtin_amdgcn_alignbit(v.y, v.x, 4u * ((uint32_t)d & 7u));
        };
        auto one = [&](int h) -> uint32_t { return (other[h >> 3] >> (4 * (h & 7))) & 0xFu; };
        int d1[4];
        uint2 raw[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            d1[k] = off(k, w.y1, w.z1);
            raw[k] = load2(d1[k]);
        }
        const uint32_t own = mine[g], par = other[g];
        uint32_t before = __builtin_amdgcn_alignbit(par, other[g - 1], 28u);
        uint32_t after = __builtin_amdgcn_alignbit(other[g + 1], par, 4u);
        uint32_t nb[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) nb[k] = shifted(raw[k], d1[k]);
        // ends of the rows: periodic neighbours
        if (w.left == Lh) before = pick(0xFu, one(h0 + Lh - 1), before);
        if (w.left <= 8) {
            const int s = 4 * (w.left - 1);
            after = pick(0xFu << s, one(h0 + w.left - Lh) << s, after);
            if (w.left < n_pairs) {
                before = pick(0xFu << (s + 4), one(h0 + w.left + Lh - 1) << (s + 4), before);
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const int d2 = off(k, w.y2, w.z2);
                    if (d2 != d1[k]) nb[k] = pick(w.second, shifted(load2(d2), d2), nb[k]);
                }
            }
        }
        const uint32_t odd = w.odd((uint32_t)c);
        const uint32_t n = unsatisfied<EA>(odd, own, par, pick(odd, after, before), nb[0], nb[1], nb[2], nb[3]);
        const ThrRow th = a.b.thr[row];
        uint32_t f = decide(n, (uint32_t)g, (uint32_t)c, (uint32_t)r >> a.b.rng_shift, th, lut_of(th), a);
        if (n_pairs < 8) f &= 0xFFFFu;
        if (f) mine[g] = own ^ f;
        cnt = (uint32_t)__builtin_popcount(f);
        nsum = __builtin_amdgcn_udot8(n, f, 0u, false);
    }
    put_tally(a, block, r, cnt, nsum, red);
}

// Row-major +-1 bytes (and bonds) to the packed arrays, and the spins back.
template <bool EA>
__global__ __launch_bounds__(kThreads) void k_pairs3d_pack(const int8_t *spins, const int8_t *coup, KArgs a) {
    const int64_t N = (int64_t)a.b.L * a.b.L * a.b.L;
    const int r = (int)(blockIdx.x / (uint32_t)a.groups);
    const int g = (int)(blockIdx.x - (uint32_t)r * (uint32_t)a.groups) * kThreads + (int)threadIdx.x;
    if (g >= a.words) return;
    const int64_t i = 16 * (int64_t)g;
    uint4 s = load_inside<int64_t>(spins + (int64_t)r * N, i, N), j[3];
    if constexpr (EA) {
        const int8_t *J = coup + (int64_t)(r / a.b.rep_per_sample) * 3 * N;
#pragma unroll
        for (int mu = 0; mu < 3; ++mu) j[mu] = load_inside<int64_t>(J + mu * N, i, N);
    }
    if (__builtin_expect(i > N - 16, 0)) {
        into_place<int64_t>(s, i, N);
        if constexpr (EA)
#pragma unroll
            for (int mu = 0; mu < 3; ++mu) into_place<int64_t>(j[mu], i, N);
    }
    const uint2 eo = words_of(s, j, EA ? 3 : 0);
    const uint32_t odd = Place(g, a.b.L).odd(0u);
    array_of(a, r, 0)[g] = pick(odd, eo.y, eo.x);
    array_of(a, r, 1)[g] = pick(odd, eo.x, eo.y);
}

__global__ __launch_bounds__(kThreads) void k_pairs3d_unpack(int8_t *spins, KArgs a) {
    const int64_t N = (int64_t)a.b.L * a.b.L * a.b.L;
    const int r = (int)(blockIdx.x / (uint32_t)a.groups);
    const int g = (int)(blockIdx.x - (uint32_t)r * (uint32_t)a.groups) * kThreads + (int)threadIdx.x;
    if (g >= a.words) return;
    const uint32_t odd = Place(g, a.b.L).odd(0u), c0 = array_of(a, r, 0)[g], c1 = array_of(a, r, 1)[g];
    const uint4 w = spins_of(pick(odd, c1, c0), pick(odd, c0, c1));
    const int64_t i = 16 * (int64_t)g;
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
    a.words = words_in(b.L);
    a.span = span_of(b.L);
    a.groups = groups;
    a.blocks = (uint32_t)groups * (uint32_t)b.n_rep;
    a.one2 = 0x00010001u;
    return a;
}

int word_groups(int L) { return (words_in(L) + kThreads - 1) / kThreads; }

}  // namespace

bool pairs3d_supported(int dim, int L) { return dim == 3 && L >= 16 && L <= 1024 && L % 2 == 0; }

bool pairs3d_launchable(int L, int n_rep) {
    return launch_config_error((uint64_t)word_groups(L) * (uint64_t)n_rep, kThreads, 0) == nullptr;
}

size_t pairs3d_bytes(int L, int n_rep) { return (size_t)n_rep * 8 * (size_t)span_of(L); }

// Planes of a thread: more of them read the planes beside less often and start with more
// loads in flight, fewer spread a small batch wider.  Per sweep with 1, 2, 4 and 8: EA 128^3
// 7.9 8.9 9.9 11.7 us, 16 Ising 64^3 8.9 8.5 9.3 11.5, EA 256^3 20.1 16.5 15.3 15.9, EA 384^3
// 56.8 44.2 39.9 38.9, EA 1024^3 1057 852 734 702.
int pairs3d_planes(int L, int n_rep) {
    if (L % 16) return 1;
    if (const char *e = getenv("SPINMC_PAIRS3D_PLANES")) {
        const int z = atoi(e);
        if (z == 1 || z == 2 || z == 4 || z == 8) return z;
    }
    const int64_t sites = (int64_t)n_rep * L * L * L;
    return sites >= (int64_t)1 << 25 ? 8 : sites >= (int64_t)1 << 23 ? 4 : sites >= (int64_t)1 << 22 ? 2 : 1;
}

int pairs3d_groups(int L, int planes) {
    if (L % 16) return word_groups(L);
    const int64_t threads = (int64_t)(L / 16) * L * (L / planes);
    return (int)((threads + kThreads - 1) / kThreads);
}

hipError_t launch_pairs3d_pack(const int8_t *spins, const int8_t *coup, const Pairs3dArgs &b, hipStream_t s) {
    if (!pairs3d_supported(3, b.L) || b.n_rep < 1 || b.rep_per_sample < 1) return hipErrorInvalidValue;
    const KArgs a = kargs(b, word_groups(b.L));
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
    const KArgs a = kargs(b, word_groups(b.L));
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
    SMC_PAIRS(false, 8)
    SMC_PAIRS(true, 8)
#undef SMC_PAIRS
    return hipErrorInvalidValue;
}

}  // namespace smc
