// Sweeps of uniform 2D Ising / +-J EA batches of any even edge, several per launch
// (Eq. 2, Sec. 3.2).
//
// A workgroup owns a tile of rows (and, where 16 divides the edge, of 16-site pieces
// of them) and holds it in LDS with 2 S halo rows above and below and a halo piece on
// either side for S sweeps: half-sweep h updates the rows that are h + 1 or more from
// the staged edge, and the sites of the halo pieces become wrong one per half-sweep
// from outside (so S <= 8 there); after 2 S half-sweeps the tile's own sites are final.
// Halo sites are recomputed by the neighbouring tiles with the same random numbers
// (every draw is keyed by the site), so tiles never exchange data within a launch;
// launches alternate between two lattices.  A tile of whole rows or columns wraps
// there in LDS and needs no halo; a whole lattice runs all sweeps of a call in place.
//
// Layout (halves.hpp): half a byte per site, the colours apart, the eight sites of a
// Philox block per word.  Where 16 divides the edge each neighbour of a block is one word.
// Other rows start and end inside pieces that they share (RAG): each row holds its own
// copy of those, masks what is not its own, shifts the rows beside it into place from two
// words and takes the neighbour across its ends from the word that holds it.
//
// Bound: for small batches the latency of a half-sweep (Philox, LDS round trip,
// barrier) and the launches, for large ones the VALU (about 105 instructions per
// word).  bands2d_shape weighs them.
//
// A thread keeps one, two or four words of a column in registers for the whole launch
// where the tile has at most 4096 (RAG: 2048), 0.70 ns of a compute unit per word and
// half-sweep, and reads three words per update; larger tiles are all in LDS (1.1 ns).
// Against bands of whole rows at a byte per site, per sweep: one 64^2 Ising lattice 0.88 ->
// 0.65 us, 512^2 2.0 -> 1.3 (tiles of 32 rows x 2 words, 8 sweeps per launch), 1024^2 3.0 -> 1.7,
// 2048^2 5.7 -> 3.3, 4096^2 EA 18.7 -> 11.9, 256 EA lattices of 256^2 10.9 -> 6.9, 64 of
// 200^2 4.9 -> 3.3, 16 of 500^2 6.1 -> 4.2, 20 Ising lattices of 106^2 1.87 -> 1.54, 16 of
// 1000^2 16.0 -> 14.8 (two half-sweep launches: 28.5), eight of 1502^2 17.0 -> 17.4.
#include <stdlib.h>

#include <algorithm>

#include "bands2d.hpp"
#include "bins2d.hpp"
#include "halves.hpp"
#include "rows.hpp"

namespace smc {
namespace {

using namespace seg3d;
using namespace halves;

constexpr int kMaxThreads = 1024;

constexpr int kPad = 4;  // words before and after the staged tile (reads beside the first and last row)

struct KArgs {
    Bands2dArgs b;
    Tally tally;
    int K;                 // pieces per row of the lattice (RAG: that a row may touch)
    int words, W;          // pieces per row of a tile: its own, staged
    int rows, halo, side;  // own rows, halo rows on either side, halo pieces (0 or 1)
    int xtiles, tiles;     // tiles per row of tiles and per replica
    int sweeps;
    int lanes;             // threads that take words (NI > 0: whole rows of them)
    uint32_t one2;         // 0x00010001, opaque to the compiler
};

// A cell of the staged tile.
struct Cell {
    int row, k;      // staged
    int y;           // lattice row
    uint32_t g;      // Philox block
    bool mine;       // of the tile itself
};

// RAG: where the sites of row y lie in its words and in those of the rows beside it.
// Pair x of the row is half-byte first + x of its words, counted from word 0.
struct Ragged {
    int first, last;   // the first and the last pair
    int up, down;      // how much later a pair lies in the rows y + 1 and y - 1
    __device__ __forceinline__ Ragged(int y, int L) {
        const int Lh = L / 2;
        first = (y * Lh) & 7;
        last = first + Lh - 1;
        up = (y == L - 1 ? 0 : (first + Lh) & 7) - first;
        down = (y == 0 ? ((L - 1) * Lh) & 7 : (first - Lh) & 7) - first;
    }
    // Mask of the row's pairs in its word k.
    __device__ __forceinline__ uint32_t in(int k) const {
        const int lo = max(first - 8 * k, 0), n = min(last + 1 - 8 * k, 8) - lo;
        return n > 0 ? (~0u >> (32 - 4 * n)) << (4 * lo) : 0u;
    }
};

// The eight half-bytes d later than word p (-7 .. 7).
__device__ __forceinline__ uint32_t later(const uint32_t *p, int d) {
    const uint32_t *q = p + (d < 0 ? -1 : 0);
    return __builtin_amdgcn_alignbit(q[1], q[0], 4u * ((uint32_t)d & 7u));
}

template <bool EA, bool RAG>
struct Tile {
    const KArgs &a;
    uint32_t *T;     // colour 0, then colour 1
    int cells;       // words of a colour
    Lut3 K3;
    ThrRow th;
    uint32_t rr;     // replica index of the draws
    uint32_t cnt = 0, nsum = 0;

    // Colour-c sites of a staged word: own and par its words of colour c and of the
    // other; returns the new own.  up, down, next, prev: distances of the cells beside it.
    __device__ __forceinline__ uint32_t update(uint32_t own, uint32_t par, const Cell &at, int up, int down, int next,
                                               int prev, uint32_t c, uint32_t time, const uint4 &w) {
        const bool odd = ((uint32_t)at.y & 1u) != c;  // own sites are the odd ones
        const uint32_t *other = T + (c ? 0 : cells) + at.row * a.W + at.k;
        uint32_t yp, ym, in = ~0u;
        const uint32_t beside = other[odd ? next : prev];
        uint32_t side = __builtin_amdgcn_alignbit(odd ? beside : par, odd ? par : beside, odd ? 4u : 28u);
        if constexpr (RAG) {
            const Ragged rg(at.y, a.b.L);
            yp = later(other + up, rg.up);
            ym = later(other + down, rg.down);
            // the row's ends: the neighbour of the last pair is the first one, and the reverse
            const int here = odd ? rg.last : rg.first, there = odd ? rg.first : rg.last;
            const uint32_t wrap = other[(there >> 3) - at.k];
            const uint32_t end = (here >> 3) == at.k ? 0xFu << (4 * (here & 7)) : 0u;
            side = pick(end, __builtin_amdgcn_alignbit(wrap, wrap, 4u * ((uint32_t)(there - here) & 7u)), side);
            in = rg.in(at.k);
        } else {
            yp = other[up];
            ym = other[down];
        }
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
            exact_decisions(o, w, th, K3, 8u * at.g, c, time, rr, a.b.key, has_tie(eq));
        uint32_t f = flags_of(o.F0, o.F1);
        if constexpr (RAG) f &= in;
        // Delta E of a flip with n unsatisfied bonds is 4 (2 - n)
        const uint32_t counted = at.mine ? f : 0u;
        cnt += (uint32_t)__builtin_popcount(counted);
        nsum = __builtin_amdgcn_udot8(n, counted, nsum, false);
        return own ^ f;
    }
};

// NI > 0: a thread keeps NI staged words of one column in registers for the whole launch
// (the workgroup's threads are whole rows; with one word each, the draws of both
// colours are made together at the start of a sweep).  NI = 0: any number, in LDS.
template <bool EA, bool RAG, int NI>
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
    Tile<EA, RAG> t{a, smem + kPad, (a.rows + 2 * halo) * W};
    t.rr = (uint32_t)r >> a.b.rng_shift;
    auto cell_of = [&](int row, int k) -> Cell {
        Cell c;
        c.row = row;
        c.k = k;
        c.y = y_own - halo + row;
        c.y += c.y < 0 ? L : c.y >= L ? -L : 0;
        c.mine = row >= halo && row < halo + own_rows;
        if constexpr (RAG) {
            c.g = ((uint32_t)(c.y * (L / 2)) >> 3) + (uint32_t)k;
        } else {
            int kx = k_own - side + k;
            kx += kx < 0 ? K : kx >= K ? -K : 0;
            c.g = (uint32_t)(c.y * K + kx);
            c.mine = c.mine && k >= side && k < side + own_words;
        }
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
                // (RAG: the last piece may run over the lattice's end, and one past it hold nothing)
                v[b] = RAG ? load_inside<int64_t>(S, i, N) : load16_any(S + i);
                if constexpr (EA) {
                    j[b][0] = RAG ? load_inside<int64_t>(J, i, N) : load16_any(J + i);
                    j[b][1] = RAG ? load_inside<int64_t>(J + N, i, N) : load16_any(J + N + i);
                }
            }
            advance(row, k);
        }
#pragma unroll
        for (int b = 0; b < kBatch; ++b)
            if (at[b] >= 0) {
                if constexpr (RAG) {
                    const int cell = at[b] >> 1, row = cell / W;
                    const int64_t i = 16 * (int64_t)cell_of(row, cell - row * W).g;
                    if (__builtin_expect(i > N - 16, 0)) {
                        into_place<int64_t>(v[b], i, N);
                        if constexpr (EA) {
                            into_place<int64_t>(j[b][0], i, N);
                            into_place<int64_t>(j[b][1], i, N);
                        }
                    }
                }
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
                        mine[b][col] = t.update(mine[b][col], mine[b][1 - col], c[b], up, down, next, prev, (uint32_t)col,
                                                time, w);
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
                        *own = t.update(*own, par, c, up, down, next, prev, col, time, w);
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
        int8_t *out = D + 16 * (int64_t)c.g;
        if constexpr (RAG) {
            const uint32_t in = Ragged(c.y, L).in(k);
            if (in == ~0u) {
                __builtin_memcpy(out, &w, 16);
            } else {
                // the row's part of a shared piece, two sites at a time
                const uint32_t ws[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
                for (int p = 0; p < 8; ++p) {
                    const uint16_t two = (uint16_t)(ws[p >> 1] >> (16 * (p & 1)));
                    if ((in >> (4 * p)) & 1u) __builtin_memcpy(out + 2 * p, &two, 2);
                }
            }
        } else {
            __builtin_memcpy(out, &w, 16);
        }
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

// Threads of a workgroup, at most `limit` of them (a multiple of 64), for R rows of K words:
// whole rows of threads with 1, 2 or `most` = 4 words each (2: rows that share pieces, of
// which 4 do not fit in the registers), as few words as the limit allows; else any number.
int threads_for(int R, int K, int most, int limit) {
    for (int n = 1; n <= most; n *= 2) {
        const int lanes = (R + n - 1) / n * K;
        if (lanes <= limit) return (lanes + 63) / 64 * 64;
    }
    const int64_t words = (int64_t)R * K, rounds = (words + limit - 1) / limit;
    return (int)std::max<int64_t>(64, ((words + rounds - 1) / rounds + 63) / 64 * 64);
}

// SPINMC_U2D_THREADS, for an edge that is a multiple of 16 up to 256; else 0.
int whole_threads_asked_for(int L) {
    const char *f = getenv("SPINMC_U2D_THREADS");
    const int v = f && uneven2d_edge_supported(L) ? atoi(f) : 0;
    return v == 64 || v == 128 || v == 256 || v == 512 ? v : 0;
}

// Fills the rest of a shape from (rows, sweeps per launch, whole) and
// estimates its time per sweep; false if it does not fit.
bool complete(BandShape &sh, int L, int n_rep, bool ea, int n_sweeps, bool even) {
    const bool rag = L % 16 != 0, cut = !rag && sh.words < L / 16;  // cut: halo pieces beside the tile
    const int halo = sh.rows >= L ? 0 : 2 * sh.sweeps, R = sh.rows + 2 * halo;
    const int K = rag ? bands2d_pieces(L) : sh.words + (cut ? 2 : 0);
    if ((int64_t)R * K > (int64_t)kMaxLdsBytes) return false;
    const size_t lds = bands2d_lds(R * K);
    if (lds > kMaxLdsBytes - 1024 || halo > L || (cut && sh.sweeps > 8)) return false;
    const int launches = bands2d_launches(sh, n_sweeps, even);
    if (launches > n_sweeps) return false;
    const int64_t pieces = (int64_t)R * K;
    const int rounds = (int)((pieces + kMaxThreads - 1) / kMaxThreads);
    const int most = rag ? 2 : 4;
    sh.threads = threads_for(R, K, most, kMaxThreads);
    if (sh.whole)
        if (const int asked = whole_threads_asked_for(L)) sh.threads = asked;
    // A launch has fewer than 2^32 work-items: of a great many lattices each gets fewer threads.
    const int64_t groups = (int64_t)n_rep * bands2d_groups(L, sh), room = 0xFFFFFFFFll / groups / 64 * 64;
    if (room < 64) return false;
    sh.threads = (int)std::min<int64_t>(sh.threads, room);
    // Workgroups per compute unit, and how many run there at once.
    const double per_cu = (double)((groups + 255) / 256);
    const double at_once = std::max(1.0, std::min({per_cu, (double)(kMaxLdsBytes / lds), 2048.0 / sh.threads}));
    // A half-sweep of one round takes about `latency` ns from barrier to barrier,
    // a busy compute unit updates a piece in about `piece` ns, a launch costs
    // about 3 us and its first loads and last stores 2 us more.  The shapes this
    // picks are within 7 % of the best measured over bands of 2 .. 128 rows and
    // 1 .. 8 sweeps (edges 130 .. 3000, 1 .. 64 replicas) and tiles of 2 .. 256 rows and
    // 1 .. 256 words (edges 64 .. 4096).
    const double latency = (sh.threads >= pieces ? 340.0 : 410.0) * (rag ? 1.2 : 1.0) * rounds;
    // (a tile's words in registers, at most four per thread, or all of them in LDS)
    const bool kept = (R + most - 1) / most * K <= sh.threads;
    const double piece = (kept ? (ea ? 0.75 : 0.68) : ea ? 1.2 : 1.1) * (rag ? 1.2 : 1.0);
    const double half = std::max(latency * per_cu / at_once, per_cu * (sh.rows + halo) * K * piece);
    const double memory = per_cu * R * 16.0 * K * (ea ? 4.0 : 2.0) / 20.0;
    sh.ns_per_sweep = (5000.0 + memory) * launches / n_sweeps + 2.0 * half;
    return true;
}

}  // namespace

// Pieces of 16 sites that a staged row has: where 16 does not divide the edge a row may
// share its first and its last one with others.
int bands2d_pieces(int L) { return L % 16 == 0 ? L / 16 : (L + 14 + 15) / 16; }
size_t bands2d_lds(int cells) { return 8 * (size_t)cells + 8 * kPad; }

bool bands2d_shape(int L, int n_rep, bool ea, int n_sweeps, bool even, BandShape *out) {
    BandShape best;
    const int all = L % 16 == 0 ? L / 16 : 0;  // pieces per row, where tiles are cut along rows
    // (of shapes with the same estimate the one with fewer sweeps per launch; the whole lattice before all)
    bool whole_first = false;
    auto offer = [&](int rows, int words, int sweeps) {
        BandShape sh;
        sh.rows = std::min(rows, L);
        sh.words = words;
        sh.sweeps = sweeps;
        sh.whole = rows >= L && words >= all;
        if (complete(sh, L, n_rep, ea, n_sweeps, even) &&
            (best.rows == 0 || sh.ns_per_sweep < best.ns_per_sweep ||
             (sh.ns_per_sweep == best.ns_per_sweep && !whole_first && sweeps < best.sweeps))) {
            best = sh;
            whole_first = false;
        }
    };
    offer(L, all, std::min(n_sweeps, 256));
    whole_first = best.rows > 0;
    // The search would take as long on the host as a short call on the chip, so what cannot win
    // is left out before its estimate is made: nothing takes less than its launches, its traffic and the
    // shortest half-sweeps or its updates (the figures are those of the estimate).
    const double slower = all ? 1.0 : 1.2, shortest = 340.0 * slower;
    const double kept = (ea ? 0.75 : 0.68) * slower, in_lds = (ea ? 1.2 : 1.1) * slower;
    const double traffic = 16.0 * (ea ? 4.0 : 2.0) / 20.0;
    const int most = all ? 4 : 2;
    const auto beaten = [&](double least) { return best.rows > 0 && least * (1.0 - 1e-9) > best.ns_per_sweep; };
    for (int sweeps : {8, 6, 5, 4, 3, 2, 1}) {
        if (sweeps > (even ? (n_sweeps + 1) / 2 : n_sweeps)) continue;
        BandShape any;
        any.sweeps = sweeps;
        const int launches = bands2d_launches(any, n_sweeps, even);
        const double per_sweep = (double)launches / n_sweeps;
        if (launches > n_sweeps || beaten(5000.0 * per_sweep + 2.0 * shortest)) continue;
        for (int parts = 1; parts <= std::max(all, 1); ++parts) {
            if (all && all % parts) continue;
            const int words = all / parts, K = all ? words + (parts > 1 ? 2 : 0) : bands2d_pieces(L);
            const int room = (int)((kMaxLdsBytes - 1024) / (8 * (size_t)K));  // rows in LDS
            // (of all heights: the sites once, with the halos of the tallest tiles)
            const double each = n_rep / 256.0 * parts * K * (1.0 + (room < L ? 2.0 * sweeps / room : 0.0)) * L;
            if (beaten((5000.0 + each * traffic) * per_sweep + 2.0 * each * kept)) continue;
            int last = 0;
            auto consider = [&](int rows) {
                rows = std::min(rows, L);
                const int halo = rows < L ? 2 * sweeps : 0, R = rows + 2 * halo;
                if (rows == last || R > room) return;
                last = rows;
                const int64_t per_cu = ((int64_t)n_rep * parts * ((L + rows - 1) / rows) + 255) / 256;
                const double memory = per_cu * R * K * traffic;
                const double at_once = std::min<int64_t>(per_cu, kMaxLdsBytes / bands2d_lds(R * K));
                const double piece = (R + most - 1) / most * K <= kMaxThreads ? kept : in_lds;
                const double half = std::max(shortest * per_cu / at_once, per_cu * (rows + halo) * K * piece);
                if (!beaten((5000.0 + memory) * per_sweep + 2.0 * half)) offer(rows, words, sweeps);
            };
            // rows that give each compute unit 1, 2, 4 or 8 tiles, and a few sizes
            const int strips_of = (int)std::min<int64_t>(256 * 8, (int64_t)n_rep * parts);
            for (int per_cu : {1, 2, 4, 8}) {
                const int strips = 256 * per_cu / strips_of;
                if (strips > 0) consider(std::max(2, (L + strips - 1) / strips));
            }
            for (int rows : {8, 16, 32, 64, 128})
                if (rows < L && (!all || rows == 32 || rows == 128)) consider(rows);
        }
    }
    const char *er = getenv("SPINMC_BANDS2D_ROWS"), *es = getenv("SPINMC_BANDS2D_SWEEPS");
    const char *ew = getenv("SPINMC_BANDS2D_WORDS");
    if (er && es && atoi(er) > 0 && atoi(es) > 0) {
        best = BandShape{};
        offer(std::min(atoi(er), L), ew && atoi(ew) > 0 ? std::min(atoi(ew), all) : all,
              std::min(atoi(es), std::max(1, n_sweeps)));
    }
    // (a measured limit of the workgroup holds for the shape, not for the choice of it)
    Shape tuned;
    if (best.whole && all && !whole_threads_asked_for(L) && tuned_shape(kShapeWhole2d, L, ea ? 1 : 0, n_rep, &tuned))
        best.threads = std::min(best.threads, threads_for(L, all, 4, tuned.v[0]));
    *out = best;
    return best.rows > 0;
}

bool bands2d_whole(int L, int n_rep, bool ea, int n_sweeps, int most_threads, BandShape *out) {
    BandShape sh;
    sh.rows = L;
    sh.words = L % 16 == 0 ? L / 16 : 0;
    sh.sweeps = std::min(n_sweeps, 256);
    sh.whole = true;
    if (!complete(sh, L, n_rep, ea, n_sweeps, true)) return false;
    sh.threads = std::min(sh.threads, threads_for(L, bands2d_pieces(L), L % 16 ? 2 : 4, most_threads));
    *out = sh;
    return true;
}

int bands2d_launches(const BandShape &sh, int n_sweeps, bool even) {
    const int n = (n_sweeps + sh.sweeps - 1) / sh.sweeps;
    return sh.whole || !even ? n : n + (n & 1);
}

int bands2d_groups(int L, const BandShape &sh) {
    return ((L + sh.rows - 1) / sh.rows) * (L % 16 == 0 ? (L / 16 + sh.words - 1) / sh.words : 1);
}

hipError_t launch_bands2d(const Bands2dArgs &b, const BandShape &sh, int sweeps, const Tally &tally, hipStream_t s) {
    const bool rag = b.L % 16 != 0, ea = b.coup != nullptr;
    KArgs a;
    a.b = b;
    a.tally = tally;
    a.K = bands2d_pieces(b.L);
    a.words = rag ? a.K : sh.words;
    a.side = a.words < a.K ? 1 : 0;
    a.W = a.words + 2 * a.side;
    a.rows = sh.rows;
    a.halo = sh.rows < b.L ? 2 * sweeps : 0;
    if (sweeps < 1 || sh.rows < 1 || sh.rows > b.L || (!sh.whole && (sweeps > sh.sweeps || b.src == b.dst)) || b.L < 4 ||
        b.L % 2 || b.rep_per_sample < 1 || a.words < 1 || a.words > a.K || a.halo > b.L || (a.side && sweeps > 8))
        return hipErrorInvalidValue;
    a.xtiles = (a.K + a.words - 1) / a.words;
    a.tiles = bands2d_groups(b.L, sh);
    a.sweeps = sweeps;
    a.one2 = 0x00010001u;
    const int R = sh.rows + 2 * a.halo;
    const size_t lds = bands2d_lds(R * a.W);
    // as few words per thread as the threads allow, in whole rows
    int per = 0;
    a.lanes = sh.threads;
    for (int n = rag ? 2 : 4; n > 0; n /= 2) {
        const int lanes = (R + n - 1) / n * a.W;
        if (lanes > sh.threads) break;
        per = n;
        a.lanes = lanes;
    }
    const int64_t blocks = (int64_t)b.n_rep * a.tiles;
    if (const char *why = launch_config_error((uint64_t)blocks, (uint64_t)sh.threads, lds))
        return reject_launch("k_tiles2d", (uint64_t)blocks, (uint64_t)sh.threads, lds, why);
#define SMC_TILES(EE, RR, NN)                                                                     \
    if (ea == EE && rag == RR && per == NN) {                                                     \
        if (lds > 65536)                                                                          \
            if (hipError_t e = hipFuncSetAttribute((const void *)k_tiles2d<EE, RR, NN>,           \
                                                   hipFuncAttributeMaxDynamicSharedMemorySize,    \
                                                   (int)kMaxLdsBytes - 1024))                     \
                return e;                                                                         \
        SMC_LAUNCH((k_tiles2d<EE, RR, NN>), dim3((unsigned)blocks), dim3(sh.threads), lds, s, a); \
        return hipGetLastError();                                                                 \
    }
#define SMC_TILES_NI(EE, RR) SMC_TILES(EE, RR, 0) SMC_TILES(EE, RR, 1) SMC_TILES(EE, RR, 2)
    SMC_TILES_NI(false, false)
    SMC_TILES_NI(false, true)
    SMC_TILES_NI(true, false)
    SMC_TILES_NI(true, true)
    SMC_TILES(false, false, 4)
    SMC_TILES(true, false, 4)
#undef SMC_TILES_NI
#undef SMC_TILES
    return hipErrorInvalidValue;
}

}  // namespace smc
