// Sweeps of tempering batches of 2D Ising / +-J EA lattices with edges in
// {16, 32, ..., 256}, uniform or uneven (Sec. 6, Eq. 12; many independent
// instances at once): one launch per step for all edges.
//
// A workgroup sweeps a bin: one replica, or several of one edge that fill 5 to
// 10 KB (two of 96^2, sixteen of 32^2).  At most 36 KB, so four workgroups
// share a compute unit: some load while the others sweep (with a byte per
// site and two workgroups all of them loaded at once: 82 us per step below).
// The largest edges go first and the small bins fill the end of the launch
// (bins of 36 KB throughout: 66 us).  Waves divide the replicas of a bin among themselves, each wave
// staying within one replica, whose index, thresholds and random key are then
// wave-uniform.
//
// LDS layout of a replica of edge L (L^2 / 2 bytes): byte i of row y is the pair
// (2i, 2i + 1), the even site in the low four bits, the odd one in the high
// four; each holds the spin and, for EA, the bonds to x + 1 and y + 1 (1: -1)
// in bits 0, 1 and 2, so a half-sweep reads no couplings.  Even sites of row y
// have colour y & 1, so the own sites of a piece of 16 are the low or the high
// halves of its eight bytes, and their row neighbours the other halves.
// The first step of a call builds the bytes from the caller's arrays, the steps
// between keep them in a packed copy in the same layout (half a byte per site
// in and out, copied as it is), the last one writes the spins back.
//
// Bound: VALU (about 0.45 ps per update at full issue), then the HBM traffic
// of 1 B per site and step.
// 256 chains of 16 temperatures, edges 32 .. 256 (77.6e6 sites): 61 us per step
// (0.78 ps per update) and 5 us for the exchange round; a launch per edge in a
// graph with couplings read from global memory took about 85 us, and 2 ms per
// call to build the graph for arrays it had not met.
#include "bins2d.hpp"

#include <algorithm>

#include "rows.hpp"
#include "segment3d.hpp"

namespace smc {
namespace {

using namespace seg3d;

constexpr int kThreads = 512;
constexpr int kWaves = kThreads / 64;
constexpr size_t kBinBytes = 36 * 1024;  // four workgroups and their tables in 160 KB
constexpr size_t kSmallBin = 10 * 1024;  // most bytes of a bin of several replicas

struct RepRow {
    uint2 lut;
    int r, row;
};

// Bits 0 of four bytes: (a ^ b) & 1, (a ^ b ^ c) & 1.
__device__ __forceinline__ uint32_t x2(uint32_t a, uint32_t b) {
    return __builtin_amdgcn_bitop3_b32(a, b, 0x01010101u, 0x28);
}
__device__ __forceinline__ uint32_t x3(uint32_t a, uint32_t b, uint32_t c) { return x2(a ^ b, c); }

// In 2D the entries move up by one (a count of 2 reads a threshold of 2^32).
__device__ __forceinline__ ThrRow table2d(const ThrRow &th) {
    ThrRow t;
    t.m[0] = th.m[0];
    t.m[3] = th.m[2];
    t.m[2] = th.m[1];
    t.m[1] = make_uint2(65536u, 0u);
    return t;
}

// Row-major +-1 bytes of 16 sites (and their bonds) to the bytes of their pairs.
template <bool EA>
__device__ __forceinline__ uint2 pairs16(const uint4 &s, const uint4 &jx, const uint4 &jy) {
    auto word = [](uint32_t v, uint32_t x, uint32_t y) -> uint32_t {
        uint32_t w = (v >> 1) & 0x01010101u;
        if constexpr (EA) w |= (x & 0x02020202u) | ((y << 1) & 0x04040404u);
        return w;
    };
    const uint4 w =
        make_uint4(word(s.x, jx.x, jy.x), word(s.y, jx.y, jy.y), word(s.z, jx.z, jy.z), word(s.w, jx.w, jy.w));
    const uint2 e = half_of(w, 0x06040200u), o = half_of(w, 0x07050301u);
    return make_uint2(e.x | (o.x << 4), e.y | (o.y << 4));
}

// Colour-c sites of piece k of row y (yH = y L/2) of the replica at S; adds the
// flips and the unsatisfied bonds of the flipped sites.
template <bool EA>
__device__ __forceinline__ void update(uint8_t *S, int L, int y, int yH, int k, uint32_t c, uint32_t t, uint32_t r,
                                       Key key, const Lut3 &K, const ThrRow *thr, uint32_t one2, uint32_t &cnt,
                                       uint32_t &nsum) {
    const int half = L >> 1, bytes = L * half;
    const bool odd = ((uint32_t)y & 1u) != c;  // own sites are the odd ones
    const int below = yH == 0 ? bytes - half : yH - half, above = yH == bytes - half ? 0 : yH + half;
    uint8_t *at = S + yH + 8 * k;
    const uint2 p = lds8(at);
    // the word before the piece (even own sites) or after it (odd), periodic in the row
    const uint32_t ext = lds4(S + yH + (odd ? (8 * k + 8 == half ? 0 : 8 * k + 8) : (k == 0 ? half - 4 : 8 * k - 4)));
    const uint2 dn = lds8(S + below + 8 * k), up = lds8(S + above + 8 * k);
    const uint32_t g = (uint32_t)((yH >> 3) + k);
    const uint4 w = philox4x32_10(make_uint4(g, t, r, 2 * kTagHead + c), key);
    // the pairs before (even own sites) or after (odd)
    const uint32_t s = odd ? 1u : 3u;
    const uint32_t mx = alignbyte(odd ? p.y : p.x, odd ? p.x : ext, s), my = alignbyte(odd ? ext : p.y, odd ? p.y : p.x, s);
    // u: the x + 1 neighbours (own bond), v: the x - 1 neighbours (their bond)
    const uint2 u = make_uint2(odd ? mx : p.x, odd ? my : p.y), v = make_uint2(odd ? p.x : mx, odd ? p.y : my);
    const uint32_t mine = odd ? 4u : 0u, other = 4u - mine;
    auto count = [&](uint32_t own, uint32_t u1, uint32_t v1, uint32_t up1, uint32_t dn1) -> uint32_t {
        const uint32_t o1 = own >> mine;
        if constexpr (EA)
            return x3(o1, u1 >> other, own >> (mine + 1u)) + x3(o1, v1 >> other, v1 >> (other + 1u)) +
                   x3(o1, up1 >> mine, own >> (mine + 2u)) + x3(o1, dn1 >> mine, dn1 >> (mine + 2u));
        else
            return x2(o1, u1 >> other) + x2(o1, v1 >> other) + x2(o1, up1 >> mine) + x2(o1, dn1 >> mine);
    };
    RowOut o;
    o.n0 = count(p.x, u.x, v.x, up.x, dn.x);
    o.n1 = count(p.y, u.y, v.y, up.y, dn.y);
    uint32_t eq = 0xFFFFFFFFu;
    o.F0 = decide4(o.n0, w.x, w.y, K, one2, eq);
    o.F1 = decide4(o.n1, w.z, w.w, K, one2, eq);
    if (__builtin_expect(__any(has_tie(eq)), 0))
        exact_decisions(o, w, table2d(*thr), K, 8u * g, c, t, r, key, has_tie(eq));
    *(uint2 *)__builtin_assume_aligned(at, 8) = make_uint2(p.x ^ (o.F0 << mine), p.y ^ (o.F1 << mine));
    // Delta E of a flip with n unsatisfied bonds is 4 (2 - n)
    cnt = __builtin_amdgcn_sad_u8(o.F0, 0u, __builtin_amdgcn_sad_u8(o.F1, 0u, cnt));
    nsum = __builtin_amdgcn_sad_u8(o.n0 & bytes_ff(o.F0), 0u, __builtin_amdgcn_sad_u8(o.n1 & bytes_ff(o.F1), 0u, nsum));
}

// (replica, row, piece) of index tid + j * threads over the pieces of a bin,
// advanced without divisions.
struct Walk {
    int rep, y, k;
    int drep, dy, dk, L, G;
    __device__ __forceinline__ Walk(int L_, int tid, int nt) : L(L_), G(L_ >> 4) {
        const int P = L * G;
        rep = tid / P;
        y = (tid - rep * P) / G;
        k = tid - rep * P - y * G;
        drep = nt / P;
        dy = (nt - drep * P) / G;
        dk = nt - drep * P - dy * G;
    }
    __device__ __forceinline__ void next() {
        k += dk;
        y += dy;
        rep += drep;
        if (k >= G) {
            k -= G;
            ++y;
        }
        if (y >= L) {
            y -= L;
            ++rep;
        }
    }
};

template <bool EA>
__global__ __launch_bounds__(kThreads, 8) void k_bins2d(Bins2dArgs a, int raw_in, int raw_out, uint32_t one2) {
    extern __shared__ __align__(16) uint8_t smem[];
    __shared__ RepRow tab[kBinReps];
    __shared__ int64_t spin_off[kBinReps], coup_off[kBinReps];
    __shared__ int dE[kBinReps];
    // consecutive bins (the replicas of one chain) on one XCD, sharing its L2
    const uint32_t nblk = gridDim.x, b = blockIdx.x;
    const Bin2d bin = a.bins[(nblk & 7u) ? b : (b & 7u) * (nblk >> 3) + (b >> 3)];
    const int L = bin.L, N = L * L, half = L >> 1, bytes = N >> 1, tid = (int)threadIdx.x, reps = bin.count;
    if (tid < reps) {
        RepRow t;
        t.r = a.work[bin.first + tid];
        t.row = a.row_of_rep[t.r];
        const ThrRow th = table2d(a.thr[t.row < 0 ? 0 : t.row]);
        const Lut3 K = lut_of(th);
        t.lut = make_uint2(K.lo, K.hi);
        tab[tid] = t;
        spin_off[tid] = a.inst[t.r].spin_off;
        coup_off[tid] = EA ? a.inst[t.r].coup_off : 0;
        dE[tid] = 0;
    }

    // ---- in, four pieces of loads in flight per thread
    if (raw_in) {
        __syncthreads();
        constexpr int kBatch = 4;
        Walk wk(L, tid, kThreads);
        while (wk.rep < reps) {
            uint4 v[kBatch], jx[kBatch], jy[kBatch];
            int at[kBatch];
#pragma unroll
            for (int j = 0; j < kBatch; ++j) {
                at[j] = -1;
                if (wk.rep < reps) {
                    const int i = wk.y * L + 16 * wk.k;
                    at[j] = wk.rep * bytes + wk.y * half + 8 * wk.k;
                    v[j] = *(const uint4 *)(a.spins + spin_off[wk.rep] + i);
                    if constexpr (EA) {
                        jx[j] = *(const uint4 *)(a.coup + coup_off[wk.rep] + i);
                        jy[j] = *(const uint4 *)(a.coup + coup_off[wk.rep] + N + i);
                    }
                }
                wk.next();
            }
#pragma unroll
            for (int j = 0; j < kBatch; ++j)
                if (at[j] >= 0)
                    *(uint2 *)__builtin_assume_aligned(smem + at[j], 8) = pairs16<EA>(v[j], jx[j], jy[j]);
        }
    } else {
        const uint4 *src = (const uint4 *)(a.packed + bin.packed);
        uint4 *dst = (uint4 *)smem;
        const int n = reps * (N >> 5);
#pragma unroll 4
        for (int i = tid; i < n; i += kThreads) dst[i] = src[i];
    }
    __syncthreads();

    // ---- the sweeps: a wave (or several) per replica
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int share = reps >= kWaves ? 1 : kWaves / reps;  // waves per replica
    const int G = L >> 4, step = 64 * share, i0 = 64 * (wave % share) + lane;
    const int y0 = i0 / G, k0 = i0 - y0 * G, dy = step / G, dk = step - dy * G;
    const int rep0 = wave / share, reps_step = share > 1 ? kBinReps : kWaves;
    uint32_t cnt = 0, nsum = 0;
    auto flush = [&](int rep) {
        int d = 2 * (int)cnt - (int)nsum;
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) d += __shfl_xor(d, o, 64);
        if (lane == 0) atomicAdd(&dE[rep], d);
        cnt = nsum = 0;
    };
    for (int sw = 0; sw < a.sweeps; ++sw) {
        const uint32_t t = a.t + (uint32_t)sw;
#pragma unroll 1
        for (uint32_t c = 0; c < 2; ++c) {
            for (int rep = rep0; rep < reps; rep += reps_step) {
                const int row = __builtin_amdgcn_readfirstlane(tab[rep].row);
                if (row < 0) continue;  // a chain without a valid permutation: unchanged
                const uint32_t r = (uint32_t)__builtin_amdgcn_readfirstlane(tab[rep].r);
                Lut3 K;
                K.lo = __builtin_amdgcn_readfirstlane(tab[rep].lut.x);
                K.hi = __builtin_amdgcn_readfirstlane(tab[rep].lut.y);
                uint8_t *S = smem + rep * bytes;
                for (int y = y0, k = k0; y < L;) {
                    update<EA>(S, L, y, y * half, k, c, t, r, a.key, K, a.thr + row, one2, cnt, nsum);
                    y += dy;
                    k += dk;
                    if (k >= G) {
                        k -= G;
                        ++y;
                    }
                }
                if (reps > kWaves) flush(rep);
            }
            __syncthreads();
        }
    }
    if (reps <= kWaves && rep0 < reps) flush(rep0);

    // ---- out
    if (raw_out) {
        Walk wk(L, tid, kThreads);
        for (; wk.rep < reps; wk.next()) {
            const uint2 e = lds8(smem + wk.rep * bytes + wk.y * half + 8 * wk.k), o = make_uint2(e.x >> 4, e.y >> 4);
            auto word = [](uint32_t od, uint32_t ev, uint32_t sel) {
                return bytes_pm1(perm(od, ev, sel) & 0x01010101u);
            };
            *(uint4 *)(a.spins + spin_off[wk.rep] + wk.y * L + 16 * wk.k) =
                make_uint4(word(o.x, e.x, 0x05010400u), word(o.x, e.x, 0x07030602u), word(o.y, e.y, 0x05010400u),
                           word(o.y, e.y, 0x07030602u));
        }
    } else {
        uint4 *dst = (uint4 *)(a.packed + bin.packed);
        const uint4 *src = (const uint4 *)smem;
        const int n = reps * (N >> 5);
#pragma unroll 4
        for (int i = tid; i < n; i += kThreads) dst[i] = src[i];
    }
    __syncthreads();
    if (tid < reps && dE[tid] != 0) a.E[tab[tid].r] += 4ll * dE[tid];
}

}  // namespace

// Share of the lanes that have a piece in the rounds of a half-sweep, with
// per replicas in a bin.
static double lanes_used(int L, int per) {
    const int pieces = L * L / 16, lanes = 64 * (per >= kWaves ? 1 : kWaves / per);
    return (double)pieces / ((pieces + lanes - 1) / lanes * lanes);
}

size_t make_bins2d(const std::vector<smc_inst> &rows, std::vector<Bin2d> *bins, std::vector<int32_t> *work) {
    constexpr int kEdges = 17;  // edge / 16, 1 .. 16
    std::vector<int32_t> of[kEdges];
    for (size_t r = 0; r < rows.size(); ++r) of[rows[r].L / 16].push_back((int32_t)r);
    // (several replicas per bin only once there are four workgroups per compute unit)
    const size_t most = std::min<size_t>(kBinReps, rows.size() / 1024);
    int64_t packed = 0;
    size_t lds = 0;
    bins->clear();
    work->clear();
    for (int e = kEdges - 1; e > 0; --e) {
        const int L = 16 * e;
        const size_t N = (size_t)L * L / 2;  // bytes
        size_t per = 1;
        for (size_t p = 2; p <= most && p * N <= kSmallBin; p *= 2)
            if (2 * p * N <= kSmallBin || lanes_used(L, (int)p) > lanes_used(L, (int)per)) per = p;
        for (size_t i = 0; i < of[e].size(); i += per) {
            const size_t n = std::min(per, of[e].size() - i);
            bins->push_back(Bin2d{packed, (int32_t)work->size(), (int32_t)n, L, 0});
            work->insert(work->end(), of[e].begin() + i, of[e].begin() + i + n);
            packed += (int64_t)(n * N);
            lds = std::max(lds, n * N);
        }
    }
    return lds;
}

double bins2d_ns(int L, int n_rep) {
    const int pieces = L * L / 16, rounds = (pieces + kThreads - 1) / kThreads;
    const double per_cu = ((n_rep + 255) / 256) * (double)pieces;
    return 2.0 * std::max(700.0 * rounds * ((n_rep + 1023) / 1024), 1.3 * per_cu);
}

hipError_t launch_bins2d(const Bins2dArgs &a, int n_bins, size_t lds, bool raw_in, bool raw_out, hipStream_t s) {
    if (a.sweeps < 1 || ((!raw_in || !raw_out) && !a.packed)) return hipErrorInvalidValue;
    const uint32_t one2 = 0x00010001u;
    if (a.coup) {
        if (lds > 60000)
            (void)hipFuncSetAttribute((const void *)k_bins2d<true>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                      (int)kBinBytes);
        SMC_LAUNCH(k_bins2d<true>, dim3((unsigned)n_bins), dim3(kThreads), lds, s, a, raw_in ? 1 : 0, raw_out ? 1 : 0,
                   one2);
    } else {
        if (lds > 60000)
            (void)hipFuncSetAttribute((const void *)k_bins2d<false>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                      (int)kBinBytes);
        SMC_LAUNCH(k_bins2d<false>, dim3((unsigned)n_bins), dim3(kThreads), lds, s, a, raw_in ? 1 : 0, raw_out ? 1 : 0,
                   one2);
    }
    return hipGetLastError();
}

}  // namespace smc
