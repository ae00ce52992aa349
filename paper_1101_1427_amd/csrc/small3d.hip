// Sweeps and parallel tempering of small 3D Ising / +-J EA lattices (even
// edges 4 .. 24) with whole replicas in LDS for every sweep and exchange round of
// a call (Eq. 2, Sec. 6, Eq. 12).
//
// A workgroup holds n replicas: the replicas of one tempering chain, or as
// many independent ones as fill it.  Bound: latency (a half-sweep of one chain
// is one or two Philox blocks per thread between two barriers); launches, three
// per step before, are gone.
//
// Layout.  Pair h of a replica is the sites (2h, 2h + 1); each pair holds one
// site of either colour, so array C_c[h] keeps the colour-c site of pair h,
// and the eight sites that share Philox block g are the bytes 8 g .. 8 g + 7 of
// C_c.  Their neighbours are all in the other array, at fixed distances in h:
// the partner at h, the other x neighbour at h + 1 or h - 1 (by the site's
// parity in x), y neighbours at h -+ L/2, z neighbours at h -+ L^2/2, and at
// other fixed distances where the lattice wraps.  A thread keeps one g for the
// whole call and has, in registers, a byte mask for each of these cases; it reads
// eight bytes at the ordinary and at the wrapped distance and merges them.
//
// A byte holds the spin in bit 0 and, for EA, the bonds to x + 1, y + 1, z + 1
// in bits 1 .. 3 (1: -1), so a neighbour pair's bond comes with the spins and
// replicas of different samples can share a workgroup.
//
// 128 chains of 24 temperatures at edge 10, 20 steps: 886 -> 140 us.  Sweeps of
// EA replicas against half-sweep launches: 64 of 16^3 2.1 us per sweep (7.9),
// 4096 of 16^3 21 (32), one of 24^3 3.8 (7.0), 1024 of 24^3 19 (32).
#include "small3d.hpp"

#include <stdlib.h>

#include <algorithm>

#include "rows.hpp"
#include "segment3d.hpp"

namespace smc {
namespace {

using namespace seg3d;

constexpr int kMaxThreads = 1024;
constexpr int kMaxReps = kSmall3dMaxReps;

struct KArgs {
    Small3dArgs b;
    int G;          // Philox blocks (groups of eight pairs) per replica
    int per_pass;   // replicas updated at once
    uint32_t one2;  // 0x00010001, opaque to the compiler
};

struct State {
    ThrRow thr[kMaxReps];        // by temperature
    uint2 lut[kMaxReps];         // by replica: its temperature's table
    double beta[kMaxReps];
    long long E[kMaxReps];       // by replica: energy (tempering) or energy change
    int temp_of_slot[kMaxReps];
    int slot_of_temp[kMaxReps];
    unsigned acc[kMaxReps];
    int bad;
};

__device__ __forceinline__ uint32_t pick(uint32_t m, uint32_t one, uint32_t zero) { return (one & m) | (zero & ~m); }
__device__ __forceinline__ uint2 pick(uint2 m, uint2 one, uint2 zero) {
    return make_uint2(pick(m.x, one.x, zero.x), pick(m.y, one.y, zero.y));
}
// The eight bytes at p moved by one: the byte after them enters, or the one before.
__device__ __forceinline__ uint2 bytes_after(const uint2 &v, const uint8_t *p) {
    return make_uint2(alignbyte(v.y, v.x, 1), alignbyte(lds4(p + 8), v.y, 1));
}
__device__ __forceinline__ uint2 bytes_before(const uint2 &v, const uint8_t *p) {
    return make_uint2(alignbyte(v.x, lds4(p - 4), 3), alignbyte(v.y, v.x, 3));
}
// Bits 0 of four bytes: (a ^ b) & 1, (a ^ b ^ c) & 1.
__device__ __forceinline__ uint32_t x2(uint32_t a, uint32_t b) {
    return __builtin_amdgcn_bitop3_b32(a, b, 0x01010101u, 0x28);
}
__device__ __forceinline__ uint32_t x3(uint32_t a, uint32_t b, uint32_t c) { return x2(a ^ b, c); }

// Byte masks of the eight pairs of a group.
struct Masks {
    uint2 odd;         // the colour-0 site is the odd one of its pair (the colour-1 site the even one)
    uint2 first, last; // first and last pair of a row
    uint2 y0, y1;      // first and last row of a plane
    uint2 z0, z1;      // first and last plane
    uint2 in;          // inside the replica
};

__device__ __forceinline__ Masks masks_of(int g, int L) {
    Masks m{};
    const int Lh = L / 2, H = L * L * Lh;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const int h = 8 * g + j;
        const int row = h / Lh, x = h - row * Lh, z = row / L, y = row - z * L;
        const uint32_t b = 0xFFu << (8 * (j & 3));
        auto set = [&](uint2 &v, bool on) {
            if (j < 4)
                v.x |= on ? b : 0u;
            else
                v.y |= on ? b : 0u;
        };
        set(m.odd, ((y + z) & 1) != 0);
        set(m.first, x == 0);
        set(m.last, x == Lh - 1);
        set(m.y0, y == 0);
        set(m.y1, y == L - 1);
        set(m.z0, z == 0);
        set(m.z1, z == L - 1);
        set(m.in, h < H);
    }
    return m;
}

// 2^32 thresholds enter the table as 0xFFFF (see lut_of).
__device__ __forceinline__ uint2 packed_lut(const ThrRow &row) {
    const Lut3 k = lut_of(row);
    return make_uint2(k.lo, k.hi);
}

// Inclusive sums over the lanes of a wavefront (all lanes active).
__device__ __forceinline__ int wave_scan(int v) {
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xF, 0xF, false);  // row_shr:1
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xF, 0xF, false);  // row_shr:2
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xF, 0xF, false);  // row_shr:4
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xF, 0xF, false);  // row_shr:8
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xA, 0xF, false);  // row_bcast:15
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xC, 0xF, false);  // row_bcast:31
    return v;
}

// Adds the lanes' energy changes to their replicas, given the inclusive sums
// over the wavefront: the lanes of a replica are consecutive and replicas
// ascend, so the last lane of each adds the sum up to itself, which the next
// replica takes back.  (An LDS addition per lane, 64 to one address, took about
// as long as the rest of the update.)
__device__ __forceinline__ void add_energies(State &st, int upto, int rep, bool valid) {
    const int lane = (int)threadIdx.x & 63;
    const int next = __builtin_amdgcn_ds_bpermute(4 * ((lane + 1) & 63), valid ? rep : -1);
    if (valid && (lane == 63 || next != rep)) {
        atomicAdd((unsigned long long *)&st.E[rep], (unsigned long long)(long long)upto);
        if (lane != 63 && next > rep) atomicAdd((unsigned long long *)&st.E[next], (unsigned long long)(long long)-upto);
    }
}

template <bool EA>
__global__ __launch_bounds__(kMaxThreads) void k_small3d(KArgs a) {
    extern __shared__ __align__(16) uint8_t smem[];
    __shared__ State st;
    const int L = a.b.L, G = a.G, tid = (int)threadIdx.x, q = (int)blockIdx.x;
    const int n = min(a.b.n, a.b.n_rep - q * a.b.n);  // replicas of this workgroup
    const int r0 = q * a.b.n;
    const int64_t N = (int64_t)L * L * L;
    const int Lh = L / 2, P2 = L * Lh, H = P2 * L;  // pairs per row, plane and replica
    const int half = 8 * G;                         // bytes of one array
    uint8_t *const T = smem + small3d_pad(L);
    const bool temper = a.b.slot_of_temp != nullptr;

    // ---- tables; a chain whose slot_of_temp row is no permutation is left as it is
    if (tid == 0) st.bad = 0;
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

    // ---- this thread's group and the replicas it serves
    const int rep0 = tid / G, g = tid - rep0 * G;
    const bool active = rep0 < a.per_pass;
    const Masks m = masks_of(g, L);

    // ---- replicas in: row-major +-1 bytes to the two arrays
    if (active)
        for (int rep = rep0; rep < n; rep += a.per_pass) {
            const int64_t i = 16 * (int64_t)g;
            const int8_t *S = a.b.spins + (int64_t)(r0 + rep) * N;
            auto word = [](uint32_t v, int shift) -> uint32_t {
                return shift ? (v << (shift - 1)) & (0x01010101u << shift) : (v >> 1) & 0x01010101u;
            };
            auto bits = [&](const uint4 &v, int shift) -> uint4 {
                return make_uint4(word(v.x, shift), word(v.y, shift), word(v.z, shift), word(v.w, shift));
            };
            uint4 w = bits(load16(S, i, N), 0);
            if constexpr (EA) {
                const int8_t *J = a.b.coup + (int64_t)((r0 + rep) / a.b.rep_per_sample) * 3 * N;
#pragma unroll
                for (int mu = 0; mu < 3; ++mu) {
                    const uint4 j = bits(load16(J + mu * N, i, N), mu + 1);
                    w = make_uint4(w.x | j.x, w.y | j.y, w.z | j.z, w.w | j.w);
                }
            }
            const uint2 e = half_of(w, 0x06040200u), o = half_of(w, 0x07050301u);
            uint8_t *p = T + rep * 2 * half + 8 * g;
            *(uint2 *)__builtin_assume_aligned(p, 8) = pick(m.odd, o, e);
            *(uint2 *)__builtin_assume_aligned(p + half, 8) = pick(m.odd, e, o);
        }
    __syncthreads();

    // ---- the steps
    for (int step = 0; step < a.b.n_steps; ++step) {
        const uint32_t t = a.b.t0 + (uint32_t)step;
        for (int j = 0; j < a.b.m; ++j) {
            const uint32_t ts = temper ? t * (uint32_t)a.b.m + (uint32_t)j : a.b.t0 + (uint32_t)j;
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                const uint2 odd = c ? make_uint2(~m.odd.x, ~m.odd.y) : m.odd;
                for (int first = 0; first < n; first += a.per_pass) {
                    const int rep = first + rep0;
                    int dE = 0;
                    if (active && rep < n) {
                        const uint32_t r = (uint32_t)(r0 + rep) >> a.b.rng_shift;
                        const uint4 w =
                            philox4x32_10(make_uint4((uint32_t)g, ts, r, 2 * kTagHead + (uint32_t)c), a.b.key);
                        uint8_t *mine = T + rep * 2 * half + c * half + 8 * g;
                        const uint8_t *other = T + rep * 2 * half + (1 - c) * half + 8 * g;
                        const uint2 own = lds8(mine), par = lds8(other);
                        const uint2 right = pick(m.last, lds8_at(other, 1 - Lh), bytes_after(par, other));
                        const uint2 left = pick(m.first, lds8_at(other, Lh - 1), bytes_before(par, other));
                        const uint2 side = pick(odd, right, left);
                        const uint2 yp = pick(m.y1, lds8_at(other, Lh - P2), lds8_at(other, Lh));
                        const uint2 ym = pick(m.y0, lds8_at(other, P2 - Lh), lds8_at(other, -Lh));
                        const uint2 zp = pick(m.z1, lds8_at(other, P2 - H), lds8_at(other, P2));
                        const uint2 zm = pick(m.z0, lds8_at(other, H - P2), lds8_at(other, -P2));
                        RowOut o;
                        if constexpr (EA) {
                            // bond of the pair itself: the even site's; of the side pair: the lower site's
                            const uint2 jp = pick(odd, par, own), js = pick(odd, own, side);
                            o.n0 = x3(own.x, par.x, jp.x >> 1) + x3(own.x, side.x, js.x >> 1) +
                                   x3(own.x, yp.x, own.x >> 2) + x3(own.x, ym.x, ym.x >> 2) +
                                   x3(own.x, zp.x, own.x >> 3) + x3(own.x, zm.x, zm.x >> 3);
                            o.n1 = x3(own.y, par.y, jp.y >> 1) + x3(own.y, side.y, js.y >> 1) +
                                   x3(own.y, yp.y, own.y >> 2) + x3(own.y, ym.y, ym.y >> 2) +
                                   x3(own.y, zp.y, own.y >> 3) + x3(own.y, zm.y, zm.y >> 3);
                        } else {
                            o.n0 = x2(own.x, par.x) + x2(own.x, side.x) + x2(own.x, yp.x) + x2(own.x, ym.x) +
                                   x2(own.x, zp.x) + x2(own.x, zm.x);
                            o.n1 = x2(own.y, par.y) + x2(own.y, side.y) + x2(own.y, yp.y) + x2(own.y, ym.y) +
                                   x2(own.y, zp.y) + x2(own.y, zm.y);
                        }
                        const uint2 lu = st.lut[rep];
                        const Lut3 K{lu.x, lu.y};
                        uint32_t eq = 0xFFFFFFFFu;
                        o.F0 = decide4(o.n0, w.x, w.y, K, a.one2, eq);
                        o.F1 = decide4(o.n1, w.z, w.w, K, a.one2, eq);
                        if (__builtin_expect(__any(has_tie(eq)), 0))
                            exact_decisions(o, w, st.thr[st.temp_of_slot[rep]], K, 8u * (uint32_t)g, (uint32_t)c, ts,
                                            r, a.b.key, has_tie(eq));
                        o.F0 &= m.in.x;
                        o.F1 &= m.in.y;
                        *(uint2 *)__builtin_assume_aligned(mine, 8) = make_uint2(own.x ^ o.F0, own.y ^ o.F1);
                        dE = (int)flip_energy(o);
                    }
                    add_energies(st, wave_scan(dE), rep, active && rep < n);
                }
                __syncthreads();
            }
        }
        if (!temper) continue;
        // exchange round: pairs (k, k + 1) with k = t mod 2, one thread each
        if (tid < n - 1 && (((uint32_t)tid ^ t) & 1u) == 0u) {
#pragma clang fp contract(off)
            const int k = tid;
            const int A = st.slot_of_temp[k], B = st.slot_of_temp[k + 1];
            const double x = (st.beta[k + 1] - st.beta[k]) * (double)(st.E[B] - st.E[A]);
            bool accept = x >= 0.0;
            if (!accept) {
                const uint4 w = philox4x32_10(make_uint4((uint32_t)k, t, (uint32_t)q, 2 * kTagSwap), a.b.key);
                accept = unit53(w.x, w.y) < exp(x);
            }
            if (accept) {
                st.slot_of_temp[k] = B;
                st.slot_of_temp[k + 1] = A;
                st.temp_of_slot[B] = k;
                st.temp_of_slot[A] = k + 1;
                const uint2 u = st.lut[A];
                st.lut[A] = st.lut[B];
                st.lut[B] = u;
                st.acc[k] += 1u;
            }
        }
        __syncthreads();
    }

    // ---- back to HBM
    if (active)
        for (int rep = rep0; rep < n; rep += a.per_pass) {
            const uint8_t *p = T + rep * 2 * half + 8 * g;
            const uint2 c0 = lds8(p), c1 = lds8(p + half);
            const uint2 e = pick(m.odd, c1, c0), o = pick(m.odd, c0, c1);
            auto out = [](uint32_t od, uint32_t ev, uint32_t sel) {
                return bytes_pm1(perm(od, ev, sel) & 0x01010101u);
            };
            const uint4 w = make_uint4(out(o.x, e.x, 0x05010400u), out(o.x, e.x, 0x07030602u),
                                       out(o.y, e.y, 0x05010400u), out(o.y, e.y, 0x07030602u));
            int8_t *D = a.b.spins + (int64_t)(r0 + rep) * N + 16 * (int64_t)g;
            if (m.in.y)  // N is a multiple of 8
                __builtin_memcpy(D, &w, 16);
            else
                __builtin_memcpy(D, &w, 8);
        }
    if (tid < n) {
        const int64_t i = (int64_t)r0 + tid;
        if (temper) {
            a.b.slot_of_temp[i] = st.slot_of_temp[tid];
            a.b.energy[i] = (double)st.E[tid];
            if (a.b.acc && tid < n - 1) a.b.acc[(int64_t)q * (n - 1) + tid] += (unsigned long long)st.acc[tid];
        } else if (a.b.dE) {
            a.b.dE[i] += st.E[tid];
        }
    }
}

int groups_of(int L) { return (L * L * L / 2 + 7) / 8; }

}  // namespace

bool small3d_supported(int dim, int L) { return dim == 3 && L >= 4 && L <= 24 && L % 2 == 0; }

size_t small3d_lds_bytes(int L, int n) { return (size_t)n * 16 * groups_of(L) + 2 * (size_t)small3d_pad(L); }

int small3d_max_reps(int L) {
    const size_t room = kMaxLdsBytes - sizeof(State) - 1024 - 2 * (size_t)small3d_pad(L);
    return (int)std::min<size_t>(kMaxReps, room / (16 * (size_t)groups_of(L)));
}

// A step takes a compute unit about 4 ns per Philox block of its chain; half-
// sweep launches take 12 us per step and 28 ps per block of all chains (140 ps
// below edge 16, a thread per pair of sites).  So 8 chains of 32 at edge 14 run
// apart (17 us per step against 22), 128 of them together (23 against 107).
bool small3d_tempers(int L, int n, int n_chains) {
    const char *env = getenv("SPINMC_SMALL3D");
    if (env && env[0] == '1') return true;
    const double blocks = (double)n * groups_of(L);
    const double together = 4.0e-3 * blocks * ((n_chains + 511) / 512) * (n_chains > 256 ? 1.25 : 1.0);
    return together < 12.0 + (L < 16 ? 140e-6 : 28e-6) * blocks * n_chains;
}

hipError_t launch_small3d(const Small3dArgs &b, hipStream_t s) {
    if (!small3d_supported(3, b.L) || b.n < 1 || b.n > small3d_max_reps(b.L) || b.n_rep < 1 || b.rep_per_sample < 1 ||
        (b.slot_of_temp && b.n_rep % b.n))
        return hipErrorInvalidValue;
    KArgs a;
    a.b = b;
    a.G = groups_of(b.L);
    // as many replicas at once as 1024 threads hold, evenly over the passes
    const int most = std::max(1, kMaxThreads / a.G), passes = (b.n + most - 1) / most;
    a.per_pass = (b.n + passes - 1) / passes;
    a.one2 = 0x00010001u;
    const int threads = std::max((a.per_pass * a.G + 63) / 64 * 64, (b.n + 63) / 64 * 64);
    const size_t lds = small3d_lds_bytes(b.L, b.n);
    const unsigned blocks = (unsigned)((b.n_rep + b.n - 1) / b.n);
    if (b.coup) {
        if (lds > 65536 - sizeof(State))
            (void)hipFuncSetAttribute((const void *)k_small3d<true>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                      (int)lds);
        SMC_LAUNCH(k_small3d<true>, dim3(blocks), dim3(threads), lds, s, a);
    } else {
        if (lds > 65536 - sizeof(State))
            (void)hipFuncSetAttribute((const void *)k_small3d<false>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                      (int)lds);
        SMC_LAUNCH(k_small3d<false>, dim3(blocks), dim3(threads), lds, s, a);
    }
    return hipGetLastError();
}

}  // namespace smc
