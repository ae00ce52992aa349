// Sweeps of uniform 2D Ising / +-J EA batches of edges that are multiples of 16,
// several per launch (Eq. 2, Sec. 3.2): bands2d.hip's scheme on tiles.
//
// A workgroup owns a tile of rows and of 16-site pieces of them, and holds it in LDS
// with 2 S halo rows above and below and a halo piece on either side for S <= 8
// sweeps: half-sweep h updates the rows that are h + 1 or more from the staged edge,
// and the sites of the halo pieces become wrong one per half-sweep from
// outside, so after 2 S <= 16 half-sweeps the tile's own sites are final.  Halo sites are
// recomputed by the neighbouring tiles with the same random numbers (every draw is
// keyed by the site).  A tile of whole rows or columns wraps there in LDS and needs
// no halo; a whole lattice runs all sweeps of a call in place.
//
// Layout (halves.hpp): half a byte per site, the colours apart, a piece's eight
// sites of a colour per word, so each neighbour of a Philox block is one word.
//
// Bound: for small batches the latency of a half-sweep (Philox, LDS round trip,
// barrier) and the launches, for large ones the VALU (about 105 instructions per
// word).  bands2d_shape weighs them.
//
// A thread keeps one, two or four words of a column in registers for the whole launch
// where the tile has at most 4096 (0.70 ns of a compute unit per word and half-sweep), and
// reads three words per update; larger tiles are all in LDS (1.1 ns).  Against
// bands of whole rows at a byte per site, per sweep: one 64^2 Ising lattice 0.88 -> 0.66 us,
// 512^2 2.0 -> 1.3 (tiles of 32 rows x 2 words, 8 sweeps per launch), 1024^2 3.0 -> 1.7, 2048^2
// 5.7 -> 3.2, 4096^2 EA 18.7 -> 11.9, 256 EA lattices of 256^2 10.9 -> 6.9, 64 of 208^2
// 3.7 -> 2.5.
#include <algorithm>

#include "bands2d.hpp"
#include "halves.hpp"
#include "rows.hpp"

namespace smc {
namespace {

using namespace seg3d;
using namespace halves;

constexpr int kMaxThreads = 1024;

struct KArgs {
    Bands2dArgs b;
    Tally tally;
    int K;                 // pieces per row of the lattice
    int words, W;          // pieces per row of a tile: its own, staged
    int rows, halo, side;  // own rows, halo rows on either side, halo pieces (0 or 1)
    int xtiles, tiles;     // tiles per row of tiles and per replica
    int sweeps;
    int lanes;             // threads that take words (NI > 0: whole rows of them)
    uint32_t one2;         // 0x00010001, opaque to the compiler
};

template <bool EA>
struct Tile {
    const KArgs &a;
    uint32_t *T;     // colour 0, then colour 1
    int cells;       // words of a colour
    Lut3 K3;
    ThrRow th;
    uint32_t rr;     // replica index of the draws
    uint32_t cnt = 0, nsum = 0;

    // Colour-c sites of a staged word: own and par its words of colour c and of the
    // other; returns the new own.
    __device__ __forceinline__ uint32_t update(uint32_t own, uint32_t par, int cell, int up, int down, int next,
                                               int prev, bool odd, uint32_t g, uint32_t c, uint32_t time,
                                               const uint4 &w, bool mine) {
        const uint32_t *other = T + (c ? 0 : cells) + cell;
        const uint32_t yp = other[up], ym = other[down], beside = other[odd ? next : prev];
        const uint32_t side = __builtin_amdgcn_alignbit(odd ? beside : par, odd ? par : beside, odd ? 4u : 28u);
        uint32_t n;  // unsatisfied bonds
        if constexpr (EA) {
            // bond of the pair itself: the even site's; of the side pair: the lower site's
            const uint32_t jp = odd ? par : own, js = odd ? own : side;
            n = x3(own, par, jp >> 1) + x3(own, side, js >> 1) + x3(own, yp, own >> 2) + x3(own, ym, ym >> 2);
        } else {
            n = x2(own, par) + x2(own, side) + x2(own, yp) + x2(own, ym);
        }
        const uint2 by = to_bytes(n);
        RowOut o;
        o.n0 = by.x;
        o.n1 = by.y;
        uint32_t eq = 0xFFFFFFFFu;
        o.F0 = decide4(o.n0, w.x, w.y, K3, a.one2, eq);
        o.F1 = decide4(o.n1, w.z, w.w, K3, a.one2, eq);
        if (__builtin_expect(__any(has_tie(eq)), 0))
            exact_decisions(o, w, th, K3, 8u * g, c, time, rr, a.b.key, has_tie(eq));
        const uint32_t f = flags_of(o.F0, o.F1);
        // Delta E of a flip with n unsatisfied bonds is 4 (2 - n)
        const uint32_t counted = mine ? f : 0u;
        cnt += (uint32_t)__builtin_popcount(counted);
        nsum = __builtin_amdgcn_udot8(n, counted, nsum, false);
        return own ^ f;
    }
};

// A cell of the staged tile.
struct Cell {
    int row, k;      // staged
    int y;           // lattice row
    uint32_t g;      // Philox block
    bool mine;       // of the tile itself
};

// NI > 0: a thread keeps NI staged words of one column in registers for the whole launch
// (the workgroup's threads are whole rows; with one word each, the draws of both
// colours are made together at the start of a sweep).  NI = 0: any number, in LDS.
template <bool EA, int NI>
__global__ __launch_bounds__(kMaxThreads) void k_tiles2d(KArgs a) {
    extern __shared__ __align__(16) uint32_t smem[];
    __shared__ long long red[kMaxThreads / 64];
    // consecutive workgroups (the tiles of one replica share halos) on one XCD
    const uint32_t nblk = gridDim.x, blk = blockIdx.x;
    const uint32_t lb = (nblk & 7u) ? blk : (blk & 7u) * (nblk >> 3) + (blk >> 3);
    const int r = (int)(lb / (uint32_t)a.tiles), tile = (int)(lb % (uint32_t)a.tiles);
    const int ty = tile / a.xtiles, tx = tile - ty * a.xtiles;
    const int L = a.b.L, K = a.K, W = a.W, tid = (int)threadIdx.x;
    const int64_t N = (int64_t)L * L;
    const int y_own = ty * a.rows, own_rows = min(a.rows, L - y_own), halo = a.halo, R = own_rows + 2 * halo;
    const int k_own = tx * a.words, own_words = min(a.words, K - k_own), side = a.side;
    const bool rings = halo == 0;  // the rows wrap in LDS
    const int8_t *S = a.b.src + (int64_t)r * N;
    int8_t *D = a.b.dst + (int64_t)r * N;
    const int trow = a.b.row_of_rep ? a.b.row_of_rep[r] : r;
    Tile<EA> t{a, smem, (a.rows + 2 * halo) * W};
    t.rr = (uint32_t)r >> a.b.rng_shift;
    auto cell_of = [&](int row, int k) -> Cell {
        Cell c;
        c.row = row;
        c.k = k;
        c.y = y_own - halo + row;
        c.y += c.y < 0 ? L : c.y >= L ? -L : 0;
        int kx = k_own - side + k;
        kx += kx < 0 ? K : kx >= K ? -K : 0;
        c.g = (uint32_t)(c.y * K + kx);
        c.mine = row >= halo && row < halo + own_rows && k >= side && k < side + own_words;
        return c;
    };

    // (row, piece) of index i = tid + j * lanes, advanced without divisions
    const int dr = a.lanes / W, dk = a.lanes - dr * W;
    const int q0 = tid / W, k0 = tid - q0 * W, row0 = tid < a.lanes ? q0 : R;
    auto advance = [&](int &row, int &k) {
        row += dr;
        k += dk;
        if (k >= W) {
            k -= W;
            ++row;
        }
    };
    const int8_t *J = nullptr;
    if constexpr (EA) J = a.b.coup + (int64_t)(r / a.b.rep_per_sample) * 2 * N;

    // tile in, up to four pieces of loads in flight per thread
    uint32_t mine[NI ? NI : 1][2];
    constexpr int kBatch = NI ? NI : 4;
    for (int row = row0, k = k0, first = 1; NI ? first : row < R; first = 0) {
        uint4 v[kBatch], j[kBatch][2];
        int at[kBatch];  // cell, twice, plus 1 where colour 0 takes the odd sites
#pragma unroll
        for (int b = 0; b < kBatch; ++b) {
            at[b] = -1;
            if (row < R) {
                const Cell c = cell_of(row, k);
                const int64_t i = 16 * (int64_t)c.g;
                at[b] = 2 * (row * W + k) + (c.y & 1);
                v[b] = load16_any(S + i);
                if constexpr (EA) {
                    j[b][0] = load16_any(J + i);
                    j[b][1] = load16_any(J + N + i);
                }
            }
            advance(row, k);
        }
#pragma unroll
        for (int b = 0; b < kBatch; ++b)
            if (at[b] >= 0) {
                const uint2 eo = words_of(v[b], j[b], EA ? 2 : 0);
                const uint32_t c0 = (at[b] & 1) ? eo.y : eo.x, c1 = (at[b] & 1) ? eo.x : eo.y;
                t.T[at[b] >> 1] = c0;
                t.T[(at[b] >> 1) + t.cells] = c1;
                if constexpr (NI != 0) {
                    mine[b][0] = c0;
                    mine[b][1] = c1;
                }
            }
    }
    // threshold table: in 2D the entries move up by one (count 2 reads 2^32)
    if (trow >= 0) {
        const ThrRow th = a.b.thr[trow];
        t.th.m[0] = th.m[0];
        t.th.m[3] = th.m[2];
        t.th.m[2] = th.m[1];
        t.th.m[1] = make_uint2(65536u, 0u);
        t.K3 = lut_of(t.th);
    }
    __syncthreads();

    if (trow >= 0) {
        const int wrap = (R - 1) * W;
        if constexpr (NI != 0) {
            const int next = k0 == W - 1 ? 1 - W : 1, prev = k0 == 0 ? W - 1 : -1;
            Cell c[NI];
#pragma unroll
            for (int b = 0; b < NI; ++b) c[b] = cell_of(min(row0 + b * dr, R - 1), k0);
            for (int sw = 0; sw < a.sweeps; ++sw) {
                const uint32_t time = a.b.t + (uint32_t)sw;
                uint4 both[2];
                if constexpr (NI == 1) {
                    both[0] = make_uint4(c[0].g, time, t.rr, 2 * kTagHead);
                    both[1] = make_uint4(c[0].g, time, t.rr, 2 * kTagHead + 1);
                    philox4x32_10_multi<2>(both, a.b.key);
                }
#pragma unroll
                for (int col = 0; col < 2; ++col) {
                    const int h = 2 * sw + col;
                    const int lo = rings ? 0 : h + 1, hi = rings ? R : R - 1 - h;
#pragma unroll
                    for (int b = 0; b < NI; ++b) {
                        const int row = row0 + b * dr;
                        if (row < lo || row >= hi) continue;
                        const int cell = row * W + k0;
                        const int up = row == R - 1 ? -wrap : W, down = row == 0 ? wrap : -W;
                        uint4 w;
                        if constexpr (NI == 1)
                            w = both[col];
                        else
                            w = philox4x32_10(make_uint4(c[b].g, time, t.rr, 2 * kTagHead + (uint32_t)col), a.b.key);
                        mine[b][col] = t.update(mine[b][col], mine[b][1 - col], cell, up, down, next, prev,
                                                ((uint32_t)c[b].y & 1u) != (uint32_t)col, c[b].g, (uint32_t)col, time, w,
                                                c[b].mine);
                        t.T[cell + (col ? t.cells : 0)] = mine[b][col];
                    }
                    __syncthreads();
                }
            }
        } else {
            for (int sw = 0; sw < a.sweeps; ++sw) {
                const uint32_t time = a.b.t + (uint32_t)sw;
#pragma unroll 1
                for (uint32_t col = 0; col < 2; ++col) {
                    const int h = 2 * sw + (int)col;
                    const int lo = rings ? 0 : h + 1, hi = rings ? R : R - 1 - h;
                    for (int row = lo + row0, k = k0; row < hi; advance(row, k)) {
                        const Cell c = cell_of(row, k);
                        const int cell = row * W + k;
                        const int up = row == R - 1 ? -wrap : W, down = row == 0 ? wrap : -W;
                        const int next = k == W - 1 ? 1 - W : 1, prev = k == 0 ? W - 1 : -1;
                        const uint4 w = philox4x32_10(make_uint4(c.g, time, t.rr, 2 * kTagHead + col), a.b.key);
                        uint32_t *own = t.T + cell + (col ? t.cells : 0);
                        const uint32_t par = t.T[cell + (col ? 0 : t.cells)];
                        *own = t.update(*own, par, cell, up, down, next, prev, ((uint32_t)c.y & 1u) != col, c.g, col, time,
                                        w, c.mine);
                    }
                    __syncthreads();
                }
            }
        }
    }

    // own pieces out
    for (int row = row0, k = k0; row < R; advance(row, k)) {
        const Cell c = cell_of(row, k);
        if (!c.mine) continue;
        const uint32_t c0 = t.T[row * W + k], c1 = t.T[row * W + k + t.cells];
        const uint4 w = (c.y & 1) ? spins_of(c1, c0) : spins_of(c0, c1);
        __builtin_memcpy(D + 16 * (int64_t)c.g, &w, 16);
    }
    if (tally_wanted(a.tally)) {
        long long v = 2ll * (long long)t.cnt - (long long)t.nsum;
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
        if ((tid & 63) == 0) red[tid >> 6] = v;
        __syncthreads();
        if (tid == 0) {
            long long tot = 0;
            for (int w = 0; w < ((int)blockDim.x + 63) >> 6; ++w) tot += red[w];
            tally_put(a.tally, lb, r, 4 * tot);
        }
    }
}

}  // namespace

hipError_t launch_tiles2d(const Bands2dArgs &b, const BandShape &sh, int sweeps, const Tally &tally, hipStream_t s) {
    KArgs a;
    a.b = b;
    a.tally = tally;
    a.K = b.L / 16;
    a.words = sh.words;
    a.side = sh.words < a.K ? 1 : 0;
    a.W = sh.words + 2 * a.side;
    a.rows = sh.rows;
    a.halo = sh.rows < b.L ? 2 * sweeps : 0;
    a.xtiles = (a.K + sh.words - 1) / sh.words;
    a.tiles = bands2d_groups(b.L, sh);
    a.sweeps = sweeps;
    a.one2 = 0x00010001u;
    if (b.L % 16 || sh.words < 1 || sh.words > a.K || sh.rows > b.L || a.halo > b.L || (a.side && sweeps > 8))
        return hipErrorInvalidValue;
    const int cells = (sh.rows + 2 * a.halo) * a.W;
    const size_t lds = 8 * (size_t)cells;
    const bool ea = b.coup != nullptr;
    // as few words per thread as the threads allow, in whole rows
    int per = 0;
    a.lanes = sh.threads;
    for (const int n : {4, 2, 1}) {
        const int lanes = (sh.rows + 2 * a.halo + n - 1) / n * a.W;
        if (lanes > sh.threads) break;
        per = n;
        a.lanes = lanes;
    }
    const int64_t blocks = (int64_t)b.n_rep * a.tiles;
    if (const char *why = launch_config_error((uint64_t)blocks, (uint64_t)sh.threads, lds))
        return reject_launch("k_tiles2d", (uint64_t)blocks, (uint64_t)sh.threads, lds, why);
    using Kernel = void (*)(KArgs);
    const Kernel kernel = per == 1   ? (ea ? k_tiles2d<true, 1> : k_tiles2d<false, 1>)
                          : per == 2 ? (ea ? k_tiles2d<true, 2> : k_tiles2d<false, 2>)
                          : per == 4 ? (ea ? k_tiles2d<true, 4> : k_tiles2d<false, 4>)
                                     : (ea ? k_tiles2d<true, 0> : k_tiles2d<false, 0>);
    if (lds > 65536)
        if (hipError_t e = hipFuncSetAttribute((const void *)kernel, hipFuncAttributeMaxDynamicSharedMemorySize,
                                               (int)kMaxLdsBytes - 1024))
            return e;
    SMC_LAUNCH(kernel, dim3((unsigned)blocks), dim3(sh.threads), lds, s, a);
    return hipGetLastError();
}

}  // namespace smc
