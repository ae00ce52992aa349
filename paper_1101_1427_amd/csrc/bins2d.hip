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
// LDS layout of a replica of edge L (L^2 / 2 bytes, halves.hpp): two arrays of half-bytes
// by colour, eight sites to a word, so the own sites, their partners and each kind
// of neighbour of a Philox block are one word, and the bonds come with them.  Even
// sites of row y have colour y & 1.
// The first step of a call builds the words from the caller's arrays, the steps
// between keep them in a packed copy in the same layout (half a byte per site
// in and out, copied as it is), the last one writes the spins back.
//
// Bound: VALU (about 0.45 ps per update at full issue), then the HBM traffic
// of 1 B per site and step.
// 256 chains of 16 temperatures, edges 32 .. 256 (77.6e6 sites): 48 us per step
// (0.62 ps per update) and 4 us for the exchange round (a byte per two sites: 61; lanes
// that walk over columns and rows of both parities: 53);
// a launch per edge in a graph with couplings read from global memory took about 85 us,
// and 2 ms per call to build the graph for arrays it had not met.
//
// Batches of up to kBinsAtOnce bins, all resident at once, make the exchange round of a step at
// the start of the next launch (SWAP), each replica for its own pair, instead of in a
// launch of its own: 16 temperatures of one 64^2 chain 8.3 -> 7.0 us per step, of 64 chains
// of 128^2 21.2 -> 19.5. In larger batches the round's four dependent loads stand before
// the sweeps of every workgroup that follows: 57 -> 58 us in the batch above (before
// the lanes kept their columns).
#include "bins2d.hpp"

#include <algorithm>

#include "halves.hpp"

namespace smc {
namespace {

using namespace seg3d;
using namespace halves;

constexpr int kThreads = 512;
constexpr int kWaves = kThreads / 64;
constexpr int kMost = (1 << 23) - 1;     // bins of a launch: fewer than 2^32 work-items
constexpr size_t kBinBytes = 36 * 1024;  // four workgroups and their tables in 160 KB
constexpr size_t kSmallBin = 10 * 1024;  // most bytes of a bin of several replicas

struct RepRow {
    uint2 lut;
    int r, row;
};

// In 2D the entries move up by one (a count of 2 reads a threshold of 2^32).
__device__ __forceinline__ ThrRow table2d(const ThrRow &th) {
    ThrRow t;
    t.m[0] = th.m[0];
    t.m[3] = th.m[2];
    t.m[2] = th.m[1];
    t.m[1] = make_uint2(65536u, 0u);
    return t;
}

// Colour-c sites of word k of the row whose first word is yG: mine and row point to word
// k of row 0 of the own array and of the other, to_beside is the distance of the word after (odd:
// the own sites are the odd ones) or before it, periodic in the row; adds the flips and the
// unsatisfied bonds of the flipped sites.
template <bool EA>
__device__ __forceinline__ void update(uint32_t *mine, const uint32_t *row, int G, int words, int yG, int k, bool odd,
                                       int to_beside, uint32_t c, uint32_t t, uint32_t r, Key key, const Lut3 &K,
                                       const ThrRow *thr, uint32_t one2, uint32_t &cnt, uint32_t &nsum) {
    const uint32_t own = mine[yG], par = row[yG];
    const uint32_t up = row[yG == words - G ? 0 : yG + G], dn = row[yG == 0 ? words - G : yG - G];
    const uint32_t beside = row[yG + to_beside];
    const uint32_t g = (uint32_t)(yG + k);
    const uint4 w = philox4x32_10(make_uint4(g, t, r, 2 * kTagHead + c), key);
    const uint32_t side = __builtin_amdgcn_alignbit(odd ? beside : par, odd ? par : beside, odd ? 4u : 28u);
    uint32_t n;  // unsatisfied bonds
    if constexpr (EA) {
        // bond of the pair itself: the even site's; of the side pair: the lower site's
        const uint32_t jp = odd ? par : own, js = odd ? own : side;
        n = x3(own, par, jp >> 1) + x3(own, side, js >> 1) + x3(own, up, own >> 2) + x3(own, dn, dn >> 2);
    } else {
        n = x2(own, par) + x2(own, side) + x2(own, up) + x2(own, dn);
    }
    const uint2 by = to_bytes(n);
    RowOut o;
    o.n0 = by.x;
    o.n1 = by.y;
    uint32_t eq = 0xFFFFFFFFu;
    o.F0 = decide4(o.n0, w.x, w.y, K, one2, eq);
    o.F1 = decide4(o.n1, w.z, w.w, K, one2, eq);
    if (__builtin_expect(__any(has_tie(eq)), 0))
        exact_decisions(o, w, table2d(*thr), K, 8u * g, c, t, r, key, has_tie(eq));
    const uint32_t f = flags_of(o.F0, o.F1);
    mine[yG] = own ^ f;
    // Delta E of a flip with n unsatisfied bonds is 4 (2 - n)
    cnt += (uint32_t)__builtin_popcount(f);
    nsum = __builtin_amdgcn_udot8(n, f, nsum, false);
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

// The threshold row of replica r after the exchange round: its pair's decision, which
// both replicas of the pair make alike from the state before it, and its entries of the
// state after it.
__device__ __forceinline__ int exchanged_row(const Bins2dArgs &a, int r, int row) {
#pragma clang fp contract(off)
    const int n = a.n_temps, q = r / n, s = r - q * n, base = a.beta_per_chain ? q * n : 0;
    const int32_t *slot = a.slot_in + (int64_t)q * n;
    if (row < 0) {
        a.slot_out[r] = slot[s];
    } else {
        const int k = row - base, other = ((uint32_t)k ^ a.swap_t) & 1u ? k - 1 : k + 1;
        int now = k;
        if (other >= 0 && other < n) {
            const int lo = min(k, other), t = slot[other], A = lo == k ? s : t, B = lo == k ? t : s;
            const uint4 w = philox4x32_10(make_uint4((uint32_t)lo, a.swap_t, (uint32_t)q, 2 * kTagSwap), a.key);
            const double x = (a.beta[base + lo + 1] - a.beta[base + lo]) *
                             (double)(a.E_in[(int64_t)q * n + B] - a.E_in[(int64_t)q * n + A]);
            if (x >= 0.0 || below_exp(unit53(w.x, w.y), x)) {
                now = other;
                if (lo == k && a.acc) a.acc[(int64_t)q * (n - 1) + k] += 1ull;
            }
        }
        a.slot_out[(int64_t)q * n + now] = s;
        row = base + now;
    }
    a.row_out[r] = row;
    return row;
}

template <bool EA, bool SWAP>
__global__ __launch_bounds__(kThreads, 8) void k_bins2d(Bins2dArgs a, int raw_in, int raw_out, uint32_t one2) {
    extern __shared__ __align__(16) uint32_t smem[];
    __shared__ RepRow tab[kBinReps];
    __shared__ int64_t spin_off[kBinReps], coup_off[kBinReps];
    __shared__ int dE[kBinReps];
    // consecutive bins (the replicas of one chain) on one XCD, sharing its L2
    const uint32_t nblk = gridDim.x, blk = blockIdx.x;
    const Bin2d bin = a.bins[(nblk & 7u) ? blk : (blk & 7u) * (nblk >> 3) + (blk >> 3)];
    const int L = bin.L, N = L * L, G = L >> 4, words = N >> 4, tid = (int)threadIdx.x, reps = bin.count;
    if (tid < reps) {
        RepRow t;
        t.r = a.work[bin.first + tid];
        t.row = a.row_in[t.r];
        if constexpr (SWAP) t.row = exchanged_row(a, t.r, t.row);
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
            uint4 v[kBatch], j[kBatch][2];
            int at[kBatch];  // word of the colour-0 array, twice, plus 1 where it takes the odd sites
#pragma unroll
            for (int b = 0; b < kBatch; ++b) {
                at[b] = -1;
                if (wk.rep < reps) {
                    const int i = wk.y * L + 16 * wk.k;
                    at[b] = 2 * (2 * wk.rep * words + wk.y * G + wk.k) + (wk.y & 1);
                    v[b] = *(const uint4 *)(a.spins + spin_off[wk.rep] + i);
                    if constexpr (EA) {
                        j[b][0] = *(const uint4 *)(a.coup + coup_off[wk.rep] + i);
                        j[b][1] = *(const uint4 *)(a.coup + coup_off[wk.rep] + N + i);
                    }
                }
                wk.next();
            }
#pragma unroll
            for (int b = 0; b < kBatch; ++b)
                if (at[b] >= 0) {
                    const uint2 eo = words_of(v[b], j[b], EA ? 2 : 0);
                    uint32_t *p = smem + (at[b] >> 1);
                    p[0] = (at[b] & 1) ? eo.y : eo.x;
                    p[words] = (at[b] & 1) ? eo.x : eo.y;
                }
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
    // (an even number of rows at a time: a lane stays in its column and on rows of one
    // parity, so that where its neighbours lie does not change from word to word)
    const int dy = (64 * share / G) & ~1, i0 = 64 * (wave % share) + lane;
    const int y0 = i0 / G, k0 = i0 - y0 * G, first = y0 < dy ? y0 * G : words;
    const int to_next = k0 == G - 1 ? 1 - G : 1, to_prev = k0 == 0 ? G - 1 : -1;
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
            const bool odd = ((uint32_t)y0 & 1u) != c;  // own sites are the odd ones
            const int to_beside = odd ? to_next : to_prev;
            for (int rep = rep0; rep < reps; rep += reps_step) {
                const int row = __builtin_amdgcn_readfirstlane(tab[rep].row);
                if (row < 0) continue;  // a chain without a valid permutation: unchanged
                const uint32_t r = (uint32_t)__builtin_amdgcn_readfirstlane(tab[rep].r);
                Lut3 K;
                K.lo = __builtin_amdgcn_readfirstlane(tab[rep].lut.x);
                K.hi = __builtin_amdgcn_readfirstlane(tab[rep].lut.y);
                uint32_t *mine = smem + (2 * rep + (int)c) * words + k0;
                const uint32_t *other = smem + (2 * rep + 1 - (int)c) * words + k0;
                for (int yG = first; yG < words; yG += dy * G)
                    update<EA>(mine, other, G, words, yG, k0, odd, to_beside, c, t, r, a.key, K, a.thr + row, one2, cnt,
                               nsum);
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
            const uint32_t *p = smem + 2 * wk.rep * words + wk.y * G + wk.k;
            const uint32_t c0 = p[0], c1 = p[words];
            *(uint4 *)(a.spins + spin_off[wk.rep] + wk.y * L + 16 * wk.k) =
                (wk.y & 1) ? spins_of(c1, c0) : spins_of(c0, c1);
        }
    } else {
        uint4 *dst = (uint4 *)(a.packed + bin.packed);
        const uint4 *src = (const uint4 *)smem;
        const int n = reps * (N >> 5);
#pragma unroll 4
        for (int i = tid; i < n; i += kThreads) dst[i] = src[i];
    }
    __syncthreads();
    if (tid < reps) a.E_out[tab[tid].r] = a.E_in[tab[tid].r] + 4ll * dE[tid];
}

}  // namespace

// Share of the lanes that have a piece in the rounds of a half-sweep, with
// per replicas in a bin.
static double lanes_used(int L, int per) {
    const int G = L / 16, pieces = L * G, lanes = 64 * (per >= kWaves ? 1 : kWaves / per), used = (lanes / G & ~1) * G;
    return (double)pieces / ((pieces + used - 1) / used * lanes);
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

int bins2d_launches(int n_bins) { return (n_bins + kMost - 1) / kMost; }

hipError_t launch_bins2d(const Bins2dArgs &a, int n_bins, size_t lds, bool raw_in, bool raw_out, hipStream_t s) {
    if (a.sweeps < 1 || ((!raw_in || !raw_out) && !a.packed)) return hipErrorInvalidValue;
    const uint32_t one2 = 0x00010001u;
    using Kernel = void (*)(Bins2dArgs, int, int, uint32_t);
    const Kernel kernel = a.coup ? (a.swap ? k_bins2d<true, true> : k_bins2d<true, false>)
                                 : (a.swap ? k_bins2d<false, true> : k_bins2d<false, false>);
    if (lds > 60000)
        (void)hipFuncSetAttribute((const void *)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kBinBytes);
    for (int first = 0; first < n_bins; first += kMost) {
        Bins2dArgs part = a;
        part.bins += first;
        SMC_LAUNCH(kernel, dim3((unsigned)std::min(kMost, n_bins - first)), dim3(kThreads), lds, s, part, raw_in ? 1 : 0,
                   raw_out ? 1 : 0, one2);
        if (hipError_t e = hipGetLastError()) return e;
    }
    return hipSuccess;
}

}  // namespace smc
