// Sweeps of uniform 2D Ising / +-J EA batches of any even edge, several per
// launch (Eq. 2, Sec. 3.2); the kernel for edges that are no multiples of 16 (the
// others: tiles2d.hip) and the choice of the shape for both.
//
// A workgroup owns a band of rows (all x) and holds it in LDS with 2 S halo
// rows on either side for S sweeps: half-sweep h updates the rows that are h + 1
// or more from the staged edge, so after 2 S half-sweeps the band's own rows
// are final.  The halo rows are recomputed by the neighbouring bands with the
// same random numbers (every draw is keyed by the site), so bands never
// exchange data within a launch; launches alternate between two lattices.  A
// lattice that fits in LDS as a whole needs no halo, wraps its rows in LDS and
// runs all sweeps of a call in place.
//
// Bound: for small batches the latency of a half-sweep (Philox, LDS round
// trip, barrier) and the launches, so as many sweeps per launch as the halo
// allows; for large ones the VALU.  bands2d_shape weighs the two.
//
// Layout.  The 16 consecutive sites 16 g .. 16 g + 15 of a replica hold the
// eight in-colour indices of Philox block g for either colour.  Row y starts at
// offset p = (y L) mod 16 of its first such piece; in LDS site x of the row has
// position q = p + x, piece k = q / 16, and the even positions (array E) and the
// odd ones (array O) lie apart, one byte per site at q / 2, so the own sites of a
// piece are eight consecutive bytes.  A row that starts or ends inside a piece
// shares it with another row; each row holds its own copy and masks the
// positions that are not its own.  Rows y - 1 and y + 1 have other offsets,
// so their bytes are read shifted by half the difference.
// One byte before array O holds a copy of the row's last site and the byte after
// the row's end in array E one of its first, so that x neighbours never wrap.
// Where these bytes lie in a piece that a thread updates, flips are
// applied with LDS exclusive-or, which leaves them alone.
//
// A byte holds the spin in bit 0 and, for EA, the bonds to x + 1 and y + 1 in
// bits 1 and 2 (1: -1), so the bond of a neighbour pair comes with the spin.
//
// Per sweep, against two half-sweep launches: 64 EA lattices of 200^2 4.6 us
// (14.3), 16 Ising lattices of 1000^2 15.0 us (28.5).
#include <stdlib.h>

#include <algorithm>

#include "bands2d.hpp"
#include "rows.hpp"
#include "segment3d.hpp"

namespace smc {
namespace {

using namespace seg3d;

constexpr int kMaxThreads = 1024;
constexpr int kPad = 16;  // bytes before and after the staged rows (shifted reads of the first and last row)

struct KArgs {
    Bands2dArgs b;
    Tally tally;
    int K, pitch;      // pieces and bytes per staged row
    int rows, halo;    // own rows per band (the last one may have fewer), halo rows on either side
    int bands, sweeps;
    uint32_t one2;     // 0x00010001, opaque to the compiler
};

// Pieces of a staged row: offset 0 when 16 divides L, at most 14 otherwise.
__host__ __device__ constexpr int pieces_of(int L) { return L % 16 == 0 ? L / 16 : (L + 14 + 15) / 16; }
// E (8 K bytes), eight bytes with the two copies, O (8 K bytes).
__host__ __device__ constexpr int pitch_of(int L) { return 16 * pieces_of(L) + 8; }


// Bits 0 of four bytes: (a ^ b) & 1, (a ^ b ^ c) & 1.
__device__ __forceinline__ uint32_t x2(uint32_t a, uint32_t b) {
    return __builtin_amdgcn_bitop3_b32(a, b, 0x01010101u, 0x28);
}
__device__ __forceinline__ uint32_t x3(uint32_t a, uint32_t b, uint32_t c) { return x2(a ^ b, c); }

// Where a piece of a staged row lies.
struct At {
    int y;           // lattice row
    uint32_t p;      // its offset in its first piece
    uint32_t g;      // Philox block of the piece
    uint32_t base;   // LDS byte of the row
    int k;
};

template <bool EA>
struct Band {
    const KArgs &a;
    uint8_t *T;      // the first staged row
    Lut3 K3;
    ThrRow th;
    uint32_t rr;     // replica index of the draws
    uint32_t cnt = 0, nsum = 0;

    __device__ __forceinline__ At at(int row, int k, int y_first) const {
        const int L = a.b.L;
        At t;
        t.y = y_first + row;
        t.y += t.y < 0 ? L : t.y >= L ? -L : 0;
        const uint32_t yL = (uint32_t)t.y * (uint32_t)L;
        t.p = yL & 15u;
        t.g = (yL >> 4) + (uint32_t)k;
        t.base = (uint32_t)row * (uint32_t)a.pitch;
        t.k = k;
        return t;
    }

    // Colour-c sites of a piece with the draw w.  up / down: LDS bytes of the
    // rows y + 1 and y - 1.
    __device__ __forceinline__ void update(const At &t, uint32_t down, uint32_t up, uint32_t c, uint32_t time,
                                           const uint4 &w, bool own_row) {
        const uint32_t L = (uint32_t)a.b.L, K8 = 8u * (uint32_t)a.K, k8 = 8u * (uint32_t)t.k;
        const bool odd = ((uint32_t)t.y & 1u) != c;  // own sites in array O
        const uint32_t mine = (odd ? K8 + 8u : 0u) + k8;
        uint8_t *own_at = T + t.base + mine;
        const uint2 own = lds8(own_at);
        const uint2 oth = lds8(T + t.base + (odd ? 0u : K8 + 8u) + k8);
        // the word before (even own sites: array O) or after (odd: array E)
        const uint32_t ext = lds4(T + t.base + (odd ? k8 + 8u : K8 + 8u + k8 - 4u));
        const uint32_t pd = t.y == 0 ? ((L - 1u) * L) & 15u : (t.p - L) & 15u;
        const uint32_t pu = t.y == (int)L - 1 ? 0u : (t.p + L) & 15u;
        const uint2 dn = lds8_at(T + down + mine, (int)(pd - t.p) >> 1);
        const uint2 un = lds8_at(T + up + mine, (int)(pu - t.p) >> 1);
        // the other array moved by one site: x - 1 of even own sites, x + 1 of odd ones
        const uint32_t s = odd ? 1u : 3u;
        uint2 sh;
        sh.x = alignbyte(odd ? oth.y : oth.x, odd ? oth.x : ext, s);
        sh.y = alignbyte(odd ? ext : oth.y, odd ? oth.y : oth.x, s);
        // u: the x + 1 neighbours (own bond), v: the x - 1 neighbours (their bond)
        const uint2 u = make_uint2(odd ? sh.x : oth.x, odd ? sh.y : oth.y);
        const uint2 v = make_uint2(odd ? oth.x : sh.x, odd ? oth.y : sh.y);
        RowOut o;
        if constexpr (EA) {
            o.n0 = x3(own.x, own.x >> 1, u.x) + x3(own.x, v.x, v.x >> 1) + x3(own.x, own.x >> 2, un.x) +
                   x3(own.x, dn.x, dn.x >> 2);
            o.n1 = x3(own.y, own.y >> 1, u.y) + x3(own.y, v.y, v.y >> 1) + x3(own.y, own.y >> 2, un.y) +
                   x3(own.y, dn.y, dn.y >> 2);
        } else {
            o.n0 = x2(own.x, u.x) + x2(own.x, v.x) + x2(own.x, un.x) + x2(own.x, dn.x);
            o.n1 = x2(own.y, u.y) + x2(own.y, v.y) + x2(own.y, un.y) + x2(own.y, dn.y);
        }
        uint32_t eq = 0xFFFFFFFFu;
        o.F0 = decide4(o.n0, w.x, w.y, K3, a.one2, eq);
        o.F1 = decide4(o.n1, w.z, w.w, K3, a.one2, eq);
        if (__builtin_expect(__any(has_tie(eq)), 0))
            exact_decisions(o, w, th, K3, 8u * t.g, c, time, rr, a.b.key, has_tie(eq));
        uint8_t *row = T + t.base;
        // positions p / 2 .. (p + L) / 2 - 1 of either array are the row's
        const uint32_t first = t.p >> 1, end = (t.p + L) >> 1;
        const uint32_t lo = first > k8 ? min(first - k8, 8u) : 0u, hi = end > k8 ? min(end - k8, 8u) : 0u;
        const uint64_t m = (hi > lo ? ~0ull >> (64u - 8u * (hi - lo)) : 0ull) << (8u * (lo & 7u));
        o.F0 &= (uint32_t)m;
        o.F1 &= (uint32_t)(m >> 32);
        const uint64_t F = ((uint64_t)o.F1 << 32) | o.F0;
        (void)__hip_atomic_fetch_xor((unsigned long long *)__builtin_assume_aligned(own_at, 8),
                                     (unsigned long long)F, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        // the copies: the first site after the row's end in E, the last one before its start in O
        if (lo < hi && (odd ? end - k8 <= 8u : t.k == 0)) {
            const uint32_t f = (uint32_t)(F >> (8u * (odd ? hi - 1u : lo))) & 1u;
            uint8_t *copy = row + (odd ? K8 + 8u + first - 1u : end);
            const uint32_t sub = (uint32_t)(uintptr_t)copy & 3u;
            (void)__hip_atomic_fetch_xor((unsigned int *)__builtin_assume_aligned(copy - sub, 4), f << (8u * sub),
                                         __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        }
        // Delta E of a flip with n unsatisfied bonds is 4 (2 - n)
        if (own_row) {
            cnt = __builtin_amdgcn_sad_u8(o.F0, 0u, __builtin_amdgcn_sad_u8(o.F1, 0u, cnt));
            nsum = __builtin_amdgcn_sad_u8(o.n0 & bytes_ff(o.F0), 0u,
                                           __builtin_amdgcn_sad_u8(o.n1 & bytes_ff(o.F1), 0u, nsum));
        }
    }
};

// ONE: a thread per staged piece, which it keeps for the whole launch; the
// draws of both colours are made together at the start of a sweep.
template <bool EA, bool ONE>
__global__ __launch_bounds__(kMaxThreads) void k_bands2d(KArgs a) {
    extern __shared__ __align__(16) uint8_t smem[];
    __shared__ long long red[kMaxThreads / 64];
    // consecutive workgroups (the bands of one replica share halo rows) on one XCD
    const uint32_t nblk = gridDim.x, b = blockIdx.x;
    const uint32_t lb = (nblk & 7u) ? b : (b & 7u) * (nblk >> 3) + (b >> 3);
    const int r = (int)(lb / (uint32_t)a.bands), band = (int)(lb % (uint32_t)a.bands);
    const int L = a.b.L, K = a.K, tid = (int)threadIdx.x, nt = (int)blockDim.x;
    const int64_t N = (int64_t)L * L;
    const int y_own = band * a.rows, own = min(a.rows, L - y_own), halo = a.halo, R = own + 2 * halo;
    const int y_first = y_own - halo;
    const bool whole = halo == 0;
    const int8_t *S = a.b.src + (int64_t)r * N;
    int8_t *D = a.b.dst + (int64_t)r * N;
    const int trow = a.b.row_of_rep ? a.b.row_of_rep[r] : r;
    uint8_t *T = smem + kPad;
    Band<EA> bd{a, T};
    bd.rr = (uint32_t)r >> a.b.rng_shift;

    // (row, piece) of index i = tid + j * nt, advanced without divisions
    const int dr = nt / K, dk = nt % K;
    const int row0 = tid / K, k0 = tid % K;

    // rows in: +-1 bytes to bits, four pieces of loads in flight per thread
    constexpr int kBatch = 4;
    for (int row = row0, k = k0; row < R;) {
        uint4 v[kBatch], jx[kBatch], jy[kBatch];
        int rw[kBatch], kk[kBatch];
#pragma unroll
        for (int j = 0; j < kBatch; ++j) {
            rw[j] = row;
            kk[j] = k;
            if (row < R) {
                const At t = bd.at(row, k, y_first);
                const int64_t i = (int64_t)16 * t.g;
                v[j] = load_inside<int64_t>(S, i, N);
                if constexpr (EA) {
                    const int8_t *J = a.b.coup + (int64_t)(r / a.b.rep_per_sample) * 2 * N;
                    jx[j] = load_inside<int64_t>(J, i, N);
                    jy[j] = load_inside<int64_t>(J + N, i, N);
                }
            }
            row += dr;
            k += dk;
            if (k >= K) {
                k -= K;
                ++row;
            }
        }
#pragma unroll
        for (int j = 0; j < kBatch; ++j)
            if (rw[j] < R) {
                const At t = bd.at(rw[j], kk[j], y_first);
                const int64_t i = (int64_t)16 * t.g;
                if (__builtin_expect(i > N - 16, 0)) {
                    into_place<int64_t>(v[j], i, N);
                    if constexpr (EA) {
                        into_place<int64_t>(jx[j], i, N);
                        into_place<int64_t>(jy[j], i, N);
                    }
                }
                auto word = [&](uint32_t s, uint32_t x, uint32_t y) -> uint32_t {
                    uint32_t w = (s >> 1) & 0x01010101u;
                    if constexpr (EA) w |= (x & 0x02020202u) | ((y << 1) & 0x04040404u);
                    return w;
                };
                uint4 w;
                if constexpr (EA)
                    w = make_uint4(word(v[j].x, jx[j].x, jy[j].x), word(v[j].y, jx[j].y, jy[j].y),
                                   word(v[j].z, jx[j].z, jy[j].z), word(v[j].w, jx[j].w, jy[j].w));
                else
                    w = make_uint4(word(v[j].x, 0, 0), word(v[j].y, 0, 0), word(v[j].z, 0, 0), word(v[j].w, 0, 0));
                uint8_t *e = T + t.base + 8 * t.k;
                *(uint2 *)__builtin_assume_aligned(e, 8) = half_of(w, 0x06040200u);
                *(uint2 *)__builtin_assume_aligned(e + 8 * K + 8, 8) = half_of(w, 0x07050301u);
            }
    }
    // threshold table: in 2D the entries move up by one (count 2 reads 2^32)
    if (trow >= 0) {
        const ThrRow th = a.b.thr[trow];
        bd.th.m[0] = th.m[0];
        bd.th.m[3] = th.m[2];
        bd.th.m[2] = th.m[1];
        bd.th.m[1] = make_uint2(65536u, 0u);
        bd.K3 = lut_of(bd.th);
    }
    __syncthreads();
    for (int row = tid; row < R; row += nt) {
        const At t = bd.at(row, 0, y_first);
        uint8_t *e = T + t.base, *o = e + 8 * K + 8;
        const uint32_t first = t.p >> 1, end = (t.p + (uint32_t)L) >> 1;
        e[end] = e[first];
        o[(int)first - 1] = o[end - 1];
    }
    __syncthreads();

    if (trow >= 0) {
        const uint32_t pitch = (uint32_t)a.pitch;
        if constexpr (ONE) {
            const bool mine = row0 < R;
            const At t = bd.at(mine ? row0 : 0, k0, y_first);
            const uint32_t down = row0 == 0 ? (uint32_t)(R - 1) * pitch : t.base - pitch;
            const uint32_t up = row0 == R - 1 ? 0u : t.base + pitch;
            const bool own_row = row0 >= halo && row0 < halo + own;
            for (int sw = 0; sw < a.sweeps; ++sw) {
                const uint32_t time = a.b.t + (uint32_t)sw;
                uint4 w[2] = {make_uint4(t.g, time, bd.rr, 2 * kTagHead), make_uint4(t.g, time, bd.rr, 2 * kTagHead + 1)};
                philox4x32_10_multi<2>(w, a.b.key);
#pragma unroll
                for (int c = 0; c < 2; ++c) {
                    const int h = 2 * sw + c;
                    const int lo = whole ? 0 : h + 1, hi = whole ? R : R - 1 - h;
                    if (mine && row0 >= lo && row0 < hi) bd.update(t, down, up, (uint32_t)c, time, w[c], own_row);
                    __syncthreads();
                }
            }
        } else {
            for (int sw = 0; sw < a.sweeps; ++sw) {
                const uint32_t time = a.b.t + (uint32_t)sw;
#pragma unroll 1
                for (int c = 0; c < 2; ++c) {
                    const int h = 2 * sw + c;
                    const int lo = whole ? 0 : h + 1, hi = whole ? R : R - 1 - h;
                    for (int row = lo + row0, k = k0; row < hi;) {
                        const At t = bd.at(row, k, y_first);
                        const uint32_t down = row == 0 ? (uint32_t)(R - 1) * pitch : t.base - pitch;
                        const uint32_t up = row == R - 1 ? 0u : t.base + pitch;
                        const uint4 w =
                            philox4x32_10(make_uint4(t.g, time, bd.rr, 2 * kTagHead + (uint32_t)c), a.b.key);
                        bd.update(t, down, up, (uint32_t)c, time, w, row >= halo && row < halo + own);
                        row += dr;
                        k += dk;
                        if (k >= K) {
                            k -= K;
                            ++row;
                        }
                    }
                    __syncthreads();
                }
            }
        }
    }

    // own rows out
    for (int row = halo + row0, k = k0; row < halo + own;) {
        const At t = bd.at(row, k, y_first);
        const uint8_t *e = T + t.base + 8 * k;
        const uint2 ev = lds8(e), od = lds8(e + 8 * K + 8);
        const uint4 w =
            make_uint4(bytes_pm1(perm(od.x, ev.x, 0x05010400u) & 0x01010101u),
                       bytes_pm1(perm(od.x, ev.x, 0x07030602u) & 0x01010101u),
                       bytes_pm1(perm(od.y, ev.y, 0x05010400u) & 0x01010101u),
                       bytes_pm1(perm(od.y, ev.y, 0x07030602u) & 0x01010101u));
        int8_t *out = D + (int64_t)16 * t.g;
        const int lo = max((int)t.p - 16 * k, 0), hi = min((int)t.p + L - 16 * k, 16);
        if (lo == 0 && hi == 16) {
            __builtin_memcpy(out, &w, 16);
        } else {
            // the row's part of a shared piece, two sites at a time
            const uint32_t ws[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const uint16_t two = (uint16_t)(ws[j >> 1] >> (16 * (j & 1)));
                if (2 * j >= lo && 2 * j < hi) __builtin_memcpy(out + 2 * j, &two, 2);
            }
        }
        row += dr;
        k += dk;
        if (k >= K) {
            k -= K;
            ++row;
        }
    }
    if (tally_wanted(a.tally)) {
        long long v = 2ll * (long long)bd.cnt - (long long)bd.nsum;
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
        if ((tid & 63) == 0) red[tid >> 6] = v;
        __syncthreads();
        if (tid == 0) {
            long long tot = 0;
            for (int w = 0; w < (nt + 63) >> 6; ++w) tot += red[w];
            tally_put(a.tally, lb, r, 4 * tot);
        }
    }
}

// Fills the rest of a shape from (rows, sweeps per launch, whole) and
// estimates its time per sweep; false if it does not fit.
bool complete(BandShape &sh, int L, int n_rep, bool ea, int n_sweeps, bool even) {
    const bool tiles = L % 16 == 0, cut = tiles && sh.words < L / 16;  // halo pieces beside the tile
    const int halo = sh.rows >= L ? 0 : 2 * sh.sweeps, R = sh.rows + 2 * halo;
    const int K = tiles ? sh.words + (cut ? 2 : 0) : pieces_of(L);
    const size_t lds = tiles ? 8 * (size_t)R * K : (size_t)R * pitch_of(L) + 2 * kPad;
    if (lds > kMaxLdsBytes - 1024 || halo > L || (cut && sh.sweeps > 8)) return false;
    const int launches = bands2d_launches(sh, n_sweeps, even);
    if (launches > n_sweeps) return false;
    const int64_t pieces = (int64_t)R * K;
    const int rounds = (int)((pieces + kMaxThreads - 1) / kMaxThreads);
    sh.threads = (int)std::max<int64_t>(64, ((pieces + rounds - 1) / rounds + 63) / 64 * 64);
    if (tiles)  // whole rows of threads with 1, 2 or 4 words each, where they suffice
        for (const int n : {4, 2, 1}) {
            const int lanes = (R + n - 1) / n * K;
            if (lanes <= kMaxThreads) sh.threads = (lanes + 63) / 64 * 64;
        }
    if (sh.threads > kMaxThreads) sh.threads = kMaxThreads;
    if (sh.whole)
        if (const int tuned = small2d_threads(L, ea)) sh.threads = tuned;
    // Workgroups per compute unit, and how many run there at once.
    const int64_t groups = (int64_t)n_rep * bands2d_groups(L, sh);
    const double per_cu = (double)((groups + 255) / 256);
    const double at_once = std::max(1.0, std::min({per_cu, (double)(kMaxLdsBytes / lds), 2048.0 / sh.threads}));
    // A half-sweep of one round takes about `latency` ns from barrier to barrier,
    // a busy compute unit updates a piece in about `piece` ns, a launch costs
    // about 3 us and its first loads and last stores 2 us more.  The shapes this
    // picks are within 7 % of the best measured over bands of 2 .. 128 rows and
    // 1 .. 8 sweeps (edges 130 .. 3000, 1 .. 64 replicas) and tiles of 2 .. 256 rows and
    // 1 .. 256 words (edges 64 .. 4096).
    const double latency = (sh.threads >= pieces ? 450.0 : 550.0) * (tiles ? 0.75 : 1.0) * rounds;
    // (a tile's words in registers, at most four per thread, or all of them in LDS)
    const double piece = !tiles ? (ea ? 1.1 : 0.9) : (R + 3) / 4 * K <= sh.threads ? (ea ? 0.75 : 0.68) : ea ? 1.2 : 1.1;
    const double half = std::max(latency * per_cu / at_once, per_cu * (sh.rows + halo) * K * piece);
    const double memory = per_cu * R * 16.0 * K * (ea ? 4.0 : 2.0) / 20.0;
    sh.ns_per_sweep = (5000.0 + memory) * launches / n_sweeps + 2.0 * half;
    return true;
}

}  // namespace

bool bands2d_shape(int L, int n_rep, bool ea, int n_sweeps, bool even, BandShape *out) {
    BandShape best;
    const int all = L % 16 == 0 ? L / 16 : 0;  // pieces per row, where tiles are cut along rows
    auto offer = [&](int rows, int words, int sweeps) {
        BandShape sh;
        sh.rows = std::min(rows, L);
        sh.words = words;
        sh.sweeps = sweeps;
        sh.whole = rows >= L && words >= all;
        if (complete(sh, L, n_rep, ea, n_sweeps, even) && (best.rows == 0 || sh.ns_per_sweep < best.ns_per_sweep)) best = sh;
    };
    offer(L, all, std::min(n_sweeps, 256));
    for (int sweeps : {1, 2, 3, 4, 6, 8})
        if (sweeps <= (even ? (n_sweeps + 1) / 2 : n_sweeps)) {
            if (!all)
                for (int rows = 2; rows < L; rows += rows < 16 ? 2 : rows < 64 ? 8 : 32) offer(rows, 0, sweeps);
            // tiles: rows that give each compute unit 1, 2, 4 or 8 of them, and a few sizes
            for (int parts = 1; parts <= all; ++parts) {
                if (all % parts) continue;
                for (int per_cu : {1, 2, 4, 8}) {
                    const int strips = 256 * per_cu / std::min(256 * 8, n_rep * parts);
                    if (strips > 0) offer(std::max(2, (L + strips - 1) / strips), all / parts, sweeps);
                }
                for (int rows : {32, 128})
                    if (rows < L) offer(rows, all / parts, sweeps);
            }
        }
    const char *er = getenv("SPINMC_BANDS2D_ROWS"), *es = getenv("SPINMC_BANDS2D_SWEEPS");
    const char *ew = getenv("SPINMC_BANDS2D_WORDS");
    if (er && es && atoi(er) > 0 && atoi(es) > 0) {
        best = BandShape{};
        offer(std::min(atoi(er), L), ew && atoi(ew) > 0 ? std::min(atoi(ew), all) : all,
              std::min(atoi(es), std::max(1, n_sweeps)));
    }
    *out = best;
    return best.rows > 0;
}

int bands2d_launches(const BandShape &sh, int n_sweeps, bool even) {
    const int n = (n_sweeps + sh.sweeps - 1) / sh.sweeps;
    return sh.whole || !even ? n : n + (n & 1);
}

int bands2d_groups(int L, const BandShape &sh) {
    return ((L + sh.rows - 1) / sh.rows) * (L % 16 == 0 ? (L / 16 + sh.words - 1) / sh.words : 1);
}

hipError_t launch_bands2d(const Bands2dArgs &b, const BandShape &sh, int sweeps, const Tally &tally, hipStream_t s) {
    if (sweeps < 1 || sh.rows < 1 || (!sh.whole && (sweeps > sh.sweeps || b.src == b.dst)) || b.L < 4 || b.L % 2 ||
        b.rep_per_sample < 1)
        return hipErrorInvalidValue;
    if (b.L % 16 == 0) return launch_tiles2d(b, sh, sweeps, tally, s);
    KArgs a;
    a.b = b;
    a.tally = tally;
    a.K = pieces_of(b.L);
    a.pitch = pitch_of(b.L);
    a.rows = sh.rows;
    a.halo = sh.whole ? 0 : 2 * sweeps;
    a.bands = bands2d_groups(b.L, sh);
    a.sweeps = sweeps;
    a.one2 = 0x00010001u;
    const int R = sh.rows + 2 * a.halo;
    const size_t lds = (size_t)R * a.pitch + 2 * kPad;
    const bool one = (int64_t)R * a.K <= sh.threads, ea = b.coup != nullptr;
    const int64_t blocks = (int64_t)b.n_rep * a.bands;
    if (const char *why = launch_config_error((uint64_t)blocks, (uint64_t)sh.threads, lds))
        return reject_launch("k_bands2d", (uint64_t)blocks, (uint64_t)sh.threads, lds, why);
    void (*kernel)(KArgs) = ea ? (one ? k_bands2d<true, true> : k_bands2d<true, false>)
                               : (one ? k_bands2d<false, true> : k_bands2d<false, false>);
    if (lds > 65536)
        if (hipError_t e = hipFuncSetAttribute((const void *)kernel, hipFuncAttributeMaxDynamicSharedMemorySize,
                                               (int)kMaxLdsBytes - 1024))
            return e;
    SMC_LAUNCH(kernel, dim3((unsigned)blocks), dim3(sh.threads), lds, s, a);
    return hipGetLastError();
}

}  // namespace smc
