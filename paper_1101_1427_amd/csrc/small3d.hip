// Sweeps and parallel tempering of small 3D Ising / +-J EA lattices (even
// edges 4 .. 24, and 32) with whole replicas in LDS for every sweep and exchange
// round of a call (Eq. 2, Sec. 6, Eq. 12).
//
// A workgroup holds n replicas: the replicas of one tempering chain, or as
// many independent ones as fill it.  Bound: VALU of the compute units that hold
// a replica.
//
// Layout (halves.hpp): half a byte per site, eight sites of one colour per word, so
// a neighbour pair's bond comes with the spins and replicas of different samples can
// share a workgroup.
// The eight sites that share Philox block g are word g of C_c.  Their
// neighbours are all in the other array, at fixed distances in h: the partner at
// h, the other x neighbour at h + 1 or h - 1 (by the site's parity in x), y
// neighbours at h -+ L/2, z neighbours at h -+ L^2/2, and at other fixed distances
// where the lattice wraps.
//
// Edges 16 and 32 (LOG = log2 L): a word lies in one row, so each neighbour
// word is one read at a distance that the thread works out once.  Other edges
// (LOG = 0): a thread has, in registers, a mask for each wrap; it shifts two words into
// place for the ordinary and for the wrapped distance and merges them.
//
// Instructions per word and half-sweep: about 120 (LOG > 0) and 160, 57 of them
// the Philox block.  A byte per site took 355 issue slots (edge 10).  Edges 16 and 32 are
// held to 64 registers, for two workgroups per compute unit; the others spill then.
//
// Per step of tempering, before (edge 16: a kernel of its own, with a byte per site
// and couplings apart; else half-sweep launches) and now: 1024 chains of 32 at edge
// 16 65 -> 48 us, 1024 of 16 40 -> 28, 128 of 24 at edge 10 37 -> 4.5, 512 of 8 at
// edge 32 147 -> 61.  Per sweep of EA replicas, against half-sweep launches: 64 of
// 16^3 7.8 -> 1.2, 4096 of 16^3 31 -> 9.7, one of 24^3 7.2 -> 2.5, 1024 of 24^3 31 -> 14,
// one of 32^3 6.8 -> 3.4, 2048 of 32^3 94 -> 33.
#include "small3d.hpp"

#include <stdlib.h>

#include <algorithm>

#include "halves.hpp"
#include "rows.hpp"

namespace smc {
namespace {

using namespace seg3d;
using namespace halves;

constexpr int kMaxThreads = 1024;
constexpr int kMaxReps = kSmall3dMaxReps;
constexpr int kSums = 8;  // energy sums per replica

struct KArgs {
    Small3dArgs b;
    int G;          // Philox blocks (words of eight pairs) per replica
    int per_pass;   // replicas updated at once
    int swap0;      // first thread of the wavefront that runs the exchange rounds
    uint32_t one2;  // 0x00010001, opaque to the compiler
};

struct State {
    ThrRow thr[kMaxReps];        // by temperature
    uint2 lut[kMaxReps];         // by replica: its temperature's table
    double beta[kMaxReps];
    long long E[kMaxReps];       // by replica: its energy at the start (tempering), else 0
    __align__(16) int dE[kMaxReps][kSums];  // and its change since, in units of 4 modulo 2^32, in parts
    int temp_of_slot[kMaxReps];
    int slot_of_temp[kMaxReps];
    unsigned acc[kMaxReps];
    int bad;
};

// The energy of a replica.  The parts are sums modulo 2^32, and so is theirs, which is
// less than 2^31 in magnitude (a replica has fewer than 2^17 bonds).
__device__ __forceinline__ long long energy_of(const State &st, int rep) {
    const int4 a = *(const int4 *)&st.dE[rep][0], b = *(const int4 *)&st.dE[rep][4];
    const uint32_t d = (uint32_t)a.x + (uint32_t)a.y + (uint32_t)a.z + (uint32_t)a.w + (uint32_t)b.x + (uint32_t)b.y +
                       (uint32_t)b.z + (uint32_t)b.w;
    return st.E[rep] + 4ll * (int)d;
}

// The eight half-bytes at distance d (any) from word p.
__device__ __forceinline__ uint32_t at(const uint32_t *p, int d) {
    const uint32_t *q = p + (d >> 3);
    return __builtin_amdgcn_alignbit(q[1], q[0], 4u * ((uint32_t)d & 7u));
}

// Masks of the eight pairs of a word.
struct Masks {
    uint32_t odd;          // the colour-0 site is the odd one of its pair (the colour-1 site the even one)
    uint32_t first, last;  // first and last pair of a row
    uint32_t y0, y1;       // first and last row of a plane
    uint32_t z0, z1;       // first and last plane
    uint32_t in;           // inside the replica
};

__device__ __forceinline__ Masks masks_of(int g, int L) {
    Masks m{};
    const int Lh = L / 2, H = L * L * Lh;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const int h = 8 * g + j;
        const int row = h / Lh, x = h - row * Lh, z = row / L, y = row - z * L;
        const uint32_t b = 0xFu << (4 * j);
        m.odd |= ((y + z) & 1) ? b : 0u;
        m.first |= x == 0 ? b : 0u;
        m.last |= x == Lh - 1 ? b : 0u;
        m.y0 |= y == 0 ? b : 0u;
        m.y1 |= y == L - 1 ? b : 0u;
        m.z0 |= z == 0 ? b : 0u;
        m.z1 |= z == L - 1 ? b : 0u;
        m.in |= h < H ? b : 0u;
    }
    return m;
}

// Distances in words of the neighbours of word g of an edge 2^LOG, whose rows are kRow words.
template <int LOG>
struct Dist {
    static constexpr int kL = 1 << LOG, kRow = kL / 16, kPlane = kL * kRow, kG = kL * kPlane;
    int yp, ym;
    uint32_t odd;  // as in Masks: all bits or none
    __device__ __forceinline__ explicit Dist(int g) {
        const int y = (g / kRow) % kL, z = g / kPlane;
        yp = y == kL - 1 ? kRow - kPlane : kRow;
        ym = y == 0 ? kPlane - kRow : -kRow;
        odd = ((y + z) & 1) ? ~0u : 0u;
    }
    static __device__ __forceinline__ int zp(int g) { return g >= kG - kPlane ? kPlane - kG : kPlane; }
    static __device__ __forceinline__ int zm(int g) { return g < kPlane ? kG - kPlane : -kPlane; }
};

// 2^32 thresholds enter the table as 0xFFFF (see lut_of).
__device__ __forceinline__ uint2 packed_lut(const ThrRow &row) {
    const Lut3 k = lut_of(row);
    return make_uint2(k.lo, k.hi);
}

template <bool EA, int LOG>
__global__ __launch_bounds__(kMaxThreads, LOG ? 8 : 4) void k_small3d(KArgs a) {
    extern __shared__ __align__(16) uint8_t smem[];
    __shared__ State st;
    const int L = LOG ? 1 << LOG : a.b.L, G = LOG ? (1 << (3 * LOG)) / 16 : a.G, tid = (int)threadIdx.x;
    const int q = (int)blockIdx.x;
    const int n = min(a.b.n, a.b.n_rep - q * a.b.n);  // replicas of this workgroup
    const int r0 = q * a.b.n;
    const int64_t N = (int64_t)L * L * L;
    const int Lh = L / 2, P2 = L * Lh, H = P2 * L;  // pairs per row, plane and replica
    uint32_t *const T = (uint32_t *)smem + small3d_pad(L);
    const bool temper = a.b.slot_of_temp != nullptr;

    // ---- tables; a chain whose slot_of_temp row is no permutation is left as it is
    if (tid == 0) st.bad = 0;
    for (int i = tid; i < n * kSums; i += (int)blockDim.x) (&st.dE[0][0])[i] = 0;
    __syncthreads();
    if (tid < n) {
        const int64_t i = (int64_t)r0 + tid;
        st.thr[tid] = a.b.thr[temper && !a.b.beta_per_chain ? tid : i];
        if (temper) {
            const int s = a.b.slot_of_temp[i];
            st.slot_of_temp[tid] = s;
            st.beta[tid] = a.b.beta[a.b.beta_per_chain ? i : tid];
            st.acc[tid] = 0u;
            st.E[tid] = (int64_t)a.b.energy[i];
            if ((unsigned)s >= (unsigned)n) atomicOr(&st.bad, 1);
        } else {
            st.temp_of_slot[tid] = tid;
            st.lut[tid] = packed_lut(st.thr[tid]);
            st.E[tid] = 0;
        }
    }
    __syncthreads();
    if (temper) {
        if (tid < n) {
            int seen = 0;
            for (int k = 0; k < n; ++k) seen += st.slot_of_temp[k] == tid ? 1 : 0;
            if (seen != 1) atomicOr(&st.bad, 1);
            if (st.bad == 0) {
                const int s = st.slot_of_temp[tid];
                st.temp_of_slot[s] = tid;
                st.lut[s] = packed_lut(st.thr[tid]);
            }
        }
        __syncthreads();
        if (st.bad) return;
    }

    // ---- this thread's words (kSlices of them, kMaxThreads apart) and the replicas it serves
    constexpr int kSlices = LOG == 5 ? 2 : 1;
    const int lanes = G / kSlices;  // threads per replica
    int rep0 = tid / lanes;
    const int g0 = tid - rep0 * lanes;
    if constexpr (LOG != 0) rep0 = __builtin_amdgcn_readfirstlane(rep0);  // lanes is a multiple of 64
    const bool active = rep0 < a.per_pass;
    Masks m{};
    if constexpr (LOG == 0) m = masks_of(g0, L);
    const Dist<LOG ? LOG : 4> dist(g0);

    // ---- replicas in: row-major +-1 bytes to the two arrays
    auto colour0_odd = [&]() -> uint32_t { return LOG ? dist.odd : m.odd; };
    if (active)
        for (int rep = rep0; rep < n; rep += a.per_pass)
#pragma unroll
            for (int sl = 0; sl < kSlices; ++sl) {
                const int g = g0 + sl * lanes;
                const int64_t i = 16 * (int64_t)g;
                const int8_t *S = a.b.spins + (int64_t)(r0 + rep) * N;
                const uint4 w = load16(S, i, N);
                uint4 bonds[3];
                if constexpr (EA) {
                    const int8_t *J = a.b.coup + (int64_t)((r0 + rep) / a.b.rep_per_sample) * 3 * N;
#pragma unroll
                    for (int mu = 0; mu < 3; ++mu) bonds[mu] = load16(J + mu * N, i, N);
                }
                const uint2 eo = words_of(w, bonds, EA ? 3 : 0);
                uint32_t *p = T + rep * 2 * G + g;
                p[0] = pick(colour0_odd(), eo.y, eo.x);
                p[G] = pick(colour0_odd(), eo.x, eo.y);
            }
    __syncthreads();

    // ---- the steps
    int *const sum = &st.dE[0][0] + (tid & (kSums - 1));
    const int k = tid - a.swap0;  // the exchange round's pair (k, k + 1)
    const bool swapper = temper && k >= 0 && k < n - 1;
    for (int step = 0; step < a.b.n_steps; ++step) {
        const uint32_t t = a.b.t0 + (uint32_t)step;
        const bool mine_to_swap = swapper && (((uint32_t)k ^ t) & 1u) == 0u;
        double u = 0.0;
        if (mine_to_swap) {
            const uint4 w = philox4x32_10(make_uint4((uint32_t)k, t, (uint32_t)q, 2 * kTagSwap), a.b.key);
            u = unit53(w.x, w.y);
        }
        for (int j = 0; j < a.b.m; ++j) {
            const uint32_t ts = temper ? t * (uint32_t)a.b.m + (uint32_t)j : a.b.t0 + (uint32_t)j;
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                const uint32_t odd = c ? ~colour0_odd() : colour0_odd();
                if (active)
                    for (int rep = rep0; rep < n; rep += a.per_pass)
#pragma unroll
                        for (int sl = 0; sl < kSlices; ++sl) {
                            const int g = g0 + sl * lanes;
                            const uint32_t r = (uint32_t)(r0 + rep) >> a.b.rng_shift;
                            const uint4 w =
                                philox4x32_10(make_uint4((uint32_t)g, ts, r, 2 * kTagHead + (uint32_t)c), a.b.key);
                            uint32_t *mine = T + rep * 2 * G + c * G + g;
                            const uint32_t *other = T + rep * 2 * G + (1 - c) * G + g;
                            const uint32_t own = *mine, par = *other;
                            uint32_t side, yp, ym, zp, zm;
                            if constexpr (LOG != 0) {
                                using D = Dist<LOG ? LOG : 4>;
                                // a row is a ring of one or two words
                                const uint32_t beside = D::kRow == 1 ? par : T[rep * 2 * G + (1 - c) * G + (g ^ 1)];
                                side = __builtin_amdgcn_alignbit(pick(odd, beside, par), pick(odd, par, beside),
                                                                 odd ? 4u : 28u);
                                yp = other[dist.yp];
                                ym = other[dist.ym];
                                zp = other[D::zp(g)];
                                zm = other[D::zm(g)];
                            } else {
                                const uint32_t right =
                                    pick(m.last, at(other, 1 - Lh), __builtin_amdgcn_alignbit(other[1], par, 4u));
                                const uint32_t left =
                                    pick(m.first, at(other, Lh - 1), __builtin_amdgcn_alignbit(par, other[-1], 28u));
                                side = pick(odd, right, left);
                                yp = pick(m.y1, at(other, Lh - P2), at(other, Lh));
                                ym = pick(m.y0, at(other, P2 - Lh), at(other, -Lh));
                                zp = pick(m.z1, at(other, P2 - H), at(other, P2));
                                zm = pick(m.z0, at(other, H - P2), at(other, -P2));
                            }
                            uint32_t cnt;  // unsatisfied bonds
                            if constexpr (EA) {
                                // bond of the pair itself: the even site's; of the side pair: the lower site's
                                const uint32_t jp = pick(odd, par, own), js = pick(odd, own, side);
                                cnt = x3(own, par, jp >> 1) + x3(own, side, js >> 1) + x3(own, yp, own >> 2) +
                                      x3(own, ym, ym >> 2) + x3(own, zp, own >> 3) + x3(own, zm, zm >> 3);
                            } else {
                                cnt = x2(own, par) + x2(own, side) + x2(own, yp) + x2(own, ym) + x2(own, zp) +
                                      x2(own, zm);
                            }
                            const uint2 lu = st.lut[rep], by = to_bytes(cnt);
                            const Lut3 K{lu.x, lu.y};
                            uint32_t eq = 0xFFFFFFFFu;
                            RowOut o;
                            o.n0 = by.x;
                            o.n1 = by.y;
                            o.F0 = decide4(o.n0, w.x, w.y, K, a.one2, eq);
                            o.F1 = decide4(o.n1, w.z, w.w, K, a.one2, eq);
                            if (__builtin_expect(__any(has_tie(eq)), 0))
                                exact_decisions(o, w, st.thr[st.temp_of_slot[rep]], K, 8u * (uint32_t)g, (uint32_t)c,
                                                ts, r, a.b.key, has_tie(eq));
                            uint32_t f = flags_of(o.F0, o.F1);
                            if constexpr (LOG == 0) f &= m.in;
                            *mine = own ^ f;
                            // Delta E of a flip with n unsatisfied bonds is 4 (3 - n)
                            const int d = 3 * __builtin_popcount(f) - (int)__builtin_amdgcn_udot8(cnt, f, 0u, false);
                            atomicAdd(sum + rep * kSums, d);
                        }
                __syncthreads();
            }
        }
        if (!temper) continue;
        // exchange round: pairs (k, k + 1) with k = t mod 2, one thread each
        if (mine_to_swap) {
#pragma clang fp contract(off)
            const int A = st.slot_of_temp[k], B = st.slot_of_temp[k + 1];
            const double x = (st.beta[k + 1] - st.beta[k]) * (double)(energy_of(st, B) - energy_of(st, A));
            if (x >= 0.0 || below_exp(u, x)) {
                st.slot_of_temp[k] = B;
                st.slot_of_temp[k + 1] = A;
                st.temp_of_slot[B] = k;
                st.temp_of_slot[A] = k + 1;
                const uint2 l = st.lut[A];
                st.lut[A] = st.lut[B];
                st.lut[B] = l;
                st.acc[k] += 1u;
            }
        }
        __syncthreads();
    }

    // ---- back to HBM
    if (active)
        for (int rep = rep0; rep < n; rep += a.per_pass)
#pragma unroll
            for (int sl = 0; sl < kSlices; ++sl) {
                const int g = g0 + sl * lanes;
                const uint32_t *p = T + rep * 2 * G + g;
                const uint4 w = spins_of(pick(colour0_odd(), p[G], p[0]), pick(colour0_odd(), p[0], p[G]));
                int8_t *D = a.b.spins + (int64_t)(r0 + rep) * N + 16 * (int64_t)g;
                if (16 * (int64_t)g + 16 <= N)  // N is a multiple of 8
                    __builtin_memcpy(D, &w, 16);
                else
                    __builtin_memcpy(D, &w, 8);
            }
    if (tid < n) {
        const int64_t i = (int64_t)r0 + tid;
        if (temper) {
            a.b.slot_of_temp[i] = st.slot_of_temp[tid];
            a.b.energy[i] = (double)energy_of(st, tid);
            if (a.b.acc && tid < n - 1) a.b.acc[(int64_t)q * (n - 1) + tid] += (unsigned long long)st.acc[tid];
        } else if (a.b.dE) {
            atomicAdd((unsigned long long *)&a.b.dE[i], (unsigned long long)energy_of(st, tid));
        }
    }
}

int groups_of(int L) { return (L * L * L / 2 + 7) / 8; }

using Kernel = void (*)(KArgs);

Kernel kernel_of(bool ea, int L) {
    if (L == 16) return ea ? k_small3d<true, 4> : k_small3d<false, 4>;
    if (L == 32) return ea ? k_small3d<true, 5> : k_small3d<false, 5>;
    return ea ? k_small3d<true, 0> : k_small3d<false, 0>;
}

}  // namespace

bool small3d_supported(int dim, int L) { return dim == 3 && L % 2 == 0 && ((L >= 4 && L <= 24) || L == 32); }

size_t small3d_lds_bytes(int L, int n) { return 4 * ((size_t)n * 2 * groups_of(L) + 2 * (size_t)small3d_pad(L)); }

int small3d_max_reps(int L) {
    const size_t room = kMaxLdsBytes - sizeof(State) - 1024 - 8 * (size_t)small3d_pad(L);
    return (int)std::min<size_t>(kMaxReps, room / (8 * (size_t)groups_of(L)));
}

// A step takes a compute unit 1 us and 1.6 ns (edges 16 and 32) or 2.8 ns per
// Philox block of its chain; half-sweep launches take 12 us per step and 28 ps per
// block of all chains (140 ps below edge 16, a thread per pair of sites).  So 16
// chains of 20 at edge 24 run apart (18 us per step against 51), 128 of 10 together
// (25 against 41); one chain of 32 at edge 16 would gain 1 us apart.
bool small3d_tempers(int L, int n, int n_chains) {
    const char *env = getenv("SPINMC_SMALL3D");
    if (env && env[0] == '1') return true;
    const double blocks = (double)n * groups_of(L);
    const double together = (1.0 + (L % 16 ? 2.8e-3 : 1.6e-3) * blocks) * ((n_chains + 255) / 256);
    return together < 12.0 + (L < 16 ? 140e-6 : 28e-6) * blocks * n_chains;
}

hipError_t launch_small3d(const Small3dArgs &b, hipStream_t s) {
    if (!small3d_supported(3, b.L) || b.n < 1 || b.n > small3d_max_reps(b.L) || b.n_rep < 1 || b.rep_per_sample < 1 ||
        (b.slot_of_temp && b.n_rep % b.n))
        return hipErrorInvalidValue;
    KArgs a;
    a.b = b;
    a.G = groups_of(b.L);
    // as many replicas at once as 1024 threads hold, evenly over the passes; the exchange
    // rounds on a wavefront of their own where there is room
    const int lanes = std::min(a.G, kMaxThreads), most = kMaxThreads / lanes, passes = (b.n + most - 1) / most;
    a.per_pass = (b.n + passes - 1) / passes;
    a.one2 = 0x00010001u;
    int threads = std::max((a.per_pass * lanes + 63) / 64 * 64, (b.n + 63) / 64 * 64);
    if (b.slot_of_temp && threads < kMaxThreads) threads += 64;
    a.swap0 = threads - 64;
    const size_t lds = small3d_lds_bytes(b.L, b.n);
    const unsigned blocks = (unsigned)((b.n_rep + b.n - 1) / b.n);
    const Kernel kernel = kernel_of(b.coup != nullptr, b.L);
    if (lds > 65536 - sizeof(State))
        (void)hipFuncSetAttribute((const void *)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    SMC_LAUNCH(kernel, dim3(blocks), dim3(threads), lds, s, a);
    return hipGetLastError();
}

}  // namespace smc
