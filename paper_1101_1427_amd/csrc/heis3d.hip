// Heisenberg half-sweeps of uniform 3D batches whose edge is a power of two
// (Sec. 4, Eq. 10): the same update as the generic kernel (same proposal
// and acceptance functions, same float32 arithmetic in the same order, same
// random numbers), with 32-bit shift/mask indexing instead of 64-bit
// divisions and one 12-byte load per neighbour.  A thread handles the
// colour-c sites of site pairs (2p, 2p+1), whose in-colour index is p.
#include <stdlib.h>

#include "heis_math.hpp"
#include "internal.hpp"

namespace smc {
namespace {

constexpr int kThreads = 256;

struct Heis3dArgs {
    float *spins;       // [n_rep][N][3]
    const float *beta;  // per replica (float32)
    Tally acc;          // accepted moves
    Key key;
    uint32_t t;
    int lgL;            // log2 of the edge
    int64_t N;          // sites per replica
    int bpr;            // blocks per replica
};

struct F3 {
    float x, y, z;
};

__device__ __forceinline__ F3 ld(const float *s, uint32_t i) { return *(const F3 *)(s + 3 * (size_t)i); }

// The loads of one site: its six neighbours and itself.
struct SiteLoads {
    F3 nb[6];
    F3 so;
};

__device__ __forceinline__ SiteLoads load_site(const float *s, uint32_t p, int lgL, int c, uint32_t &i) {
    const uint32_t L = 1u << lgL, m = L - 1u;
    const uint32_t row = p >> (lgL - 1), pi = p & ((L >> 1) - 1u);
    const uint32_t y = row & m, z = row >> lgL;
    const uint32_t x = 2u * pi + (((y ^ z) & 1u) ^ (uint32_t)c);
    const uint32_t base = row << lgL;  // site (0, y, z)
    const uint32_t P = L << lgL;       // sites per z plane
    i = base + x;
    SiteLoads l;
    // neighbours in the order of the generic kernel: +x, -x, +y, -y, +z, -z
    l.nb[0] = ld(s, base + ((x + 1u) & m));
    l.nb[1] = ld(s, base + ((x - 1u) & m));
    l.nb[2] = ld(s, i - y * L + ((y + 1u) & m) * L);
    l.nb[3] = ld(s, i - y * L + ((y - 1u) & m) * L);
    l.nb[4] = ld(s, i - z * P + ((z + 1u) & m) * P);
    l.nb[5] = ld(s, i - z * P + ((z - 1u) & m) * P);
    l.so = ld(s, i);
    return l;
}

// Each thread updates kSitesPerThread sites (pairs p, p + kThreads, ...) and
// issues all their loads before the first update, so that a wave keeps
// several loads per lane in flight.
constexpr int kSitesPerThread = 4;

__global__ __launch_bounds__(kThreads) void k_heis3d_half(Heis3dArgs a, int c) {
    __shared__ int red[kThreads / 64];
    const int r = blockIdx.x / a.bpr;
    const uint32_t p0 = (uint32_t)(blockIdx.x % a.bpr) * (kThreads * kSitesPerThread) + threadIdx.x;
    float *s = a.spins + (size_t)r * 3 * (size_t)a.N;
    const int64_t pairs = a.N / 2;
    SiteLoads l[kSitesPerThread];
    uint32_t idx[kSitesPerThread];
#pragma unroll
    for (int q = 0; q < kSitesPerThread; ++q) {
        const uint32_t p = p0 + (uint32_t)(q * kThreads);
        if ((int64_t)p < pairs) l[q] = load_site(s, p, a.lgL, c, idx[q]);
    }
    const float beta = a.beta[r];
    int n_acc = 0;
#pragma unroll
    for (int q = 0; q < kSitesPerThread; ++q) {
        const uint32_t p = p0 + (uint32_t)(q * kThreads);
        if ((int64_t)p >= pairs) continue;
        float3 hf = make_float3(0.f, 0.f, 0.f);
#pragma unroll
        for (int k = 0; k < 6; ++k) {
            hf.x += l[q].nb[k].x;
            hf.y += l[q].nb[k].y;
            hf.z += l[q].nb[k].z;
        }
        const F3 so = l[q].so;
        const uint4 w = philox4x32_10(make_uint4(p, a.t, (uint32_t)r, 2 * kTagHeis + (uint32_t)c), a.key);
        const float3 sp = heis_proposal(unit23f(w.x), unit23f(w.y));
        const float dE = -((sp.x - so.x) * hf.x + (sp.y - so.y) * hf.y + (sp.z - so.z) * hf.z);
        if (dE <= 0.0f || unit23f(w.z) < heis_boltzmann(beta, dE)) {
            F3 v;
            v.x = sp.x;
            v.y = sp.y;
            v.z = sp.z;
            *(F3 *)(s + 3 * (size_t)idx[q]) = v;
            ++n_acc;
        }
    }
    if (tally_wanted(a.acc)) {
        int v = n_acc;
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
        if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
        __syncthreads();
        if (threadIdx.x == 0) {
            const int tot = red[0] + red[1] + red[2] + red[3];
            tally_put(a.acc, blockIdx.x, r, tot);
        }
    }
}

// ----------------------------------------------------------------------
// One-pass sweep (colour 0 then colour 1 in a single pass over the
// lattice), any even edge from 32 on.  A workgroup owns a tile of kTile x kTile
// sites in (x, y) (fewer at the end of an edge that is no multiple) over a
// segment of planes in z and streams down the planes: at step z it
// updates colour 0 of plane z on the tile plus a one-site ring, then colour 1
// of plane z-1 on the tile (its neighbours are then final), and writes plane
// z-1 of the tile.  The ring's colour-0 values are recomputed identically by
// the neighbouring tiles (every draw is keyed by the site), so tiles never
// exchange data; reads come from one buffer and writes go to the other.
// Planes live in LDS as structure-of-arrays float planes of
// (kTile+4) x (kTile+4) sites (two-site halo), five planes in a ring.
//
// Order within step z: request plane z+2 from global memory into
// registers, colour 0 of plane z, colour 1 of plane z-1, then wait for the
// requested plane, put it into the slot of plane z-3, and only then store
// the tile's plane z-1 to global memory.  Loads and stores share one
// completion counter on this target, so a wait for data also waits for
// every store issued before it; in this order the stores a wait covers were
// issued two update phases earlier and have completed.
//
// Bound: at 256^3 the HBM traffic (95 us per sweep, 5.3 TB/s with the halos);
// below, the latency of a plane step (1.5 us alone on a compute unit, the wait
// for the plane that it requests), so short segments fill the chip first.
// Per sweep: one 64^3 lattice 9.1 us (58 with segments of 32 planes), 128^3 19.6
// (58); on edges that took the half-sweep kernel 96^3 16 us (31), 160^3 36 (88),
// 200^3 74 (163).  Drawing for both half-steps at the start of a step was 0.5 % slower
// at 256^3 and 3 % at 64^3.
constexpr int kTile = 32;
constexpr int kMaxSeg = 32;
constexpr int kW = kTile + 4;       // staged width with the halo
constexpr int kPlane = kW * kW;     // sites per staged plane
constexpr int kRing = 5;
constexpr int kTiledThreads = 576;  // one colour-0 cell per thread (see update_colour0)
constexpr int kLoadsPerThread = (kPlane + kTiledThreads - 1) / kTiledThreads;

struct TiledArgs {
    const float *src;  // [n_rep][N][3]
    float *dst;
    const float *beta;
    Tally acc;  // accepted moves
    Key key;
    uint32_t t;
    int L, lgL;        // edge and, for a power of two, its logarithm
    int64_t N;
    int tiles, segs;   // tiles per row of tiles, segments per replica
    int D;             // planes per segment (the last one may have fewer)
    int xcd_remap;     // 1: consecutive tiles of a segment on one XCD (shared halo lines in its L2)
    int renorm;        // 1: the stored spins are renormalised (this sweep ends a renormalisation period)
};

struct PlaneRegs {
    F3 v[kLoadsPerThread];
};

// A coordinate in [-L, 2 L) in the lattice, and the index of a site.
template <bool POW2>
__device__ __forceinline__ uint32_t wrapped(int v, const TiledArgs &a) {
    if constexpr (POW2) return (uint32_t)v & ((1u << a.lgL) - 1u);
    return (uint32_t)(v < 0 ? v + a.L : v >= a.L ? v - a.L : v);
}
template <bool POW2>
__device__ __forceinline__ uint32_t site(uint32_t x, uint32_t y, uint32_t z, const TiledArgs &a) {
    if constexpr (POW2) return (((z << a.lgL) + y) << a.lgL) + x;
    return (z * (uint32_t)a.L + y) * (uint32_t)a.L + x;
}

template <bool POW2>
__device__ __forceinline__ void load_plane(const float *src, const TiledArgs &a, int x0, int y0, int z,
                                           PlaneRegs &pr) {
    const uint32_t zz = wrapped<POW2>(z, a);
#pragma unroll
    for (int j = 0; j < kLoadsPerThread; ++j) {
        const int q = (int)threadIdx.x + j * kTiledThreads;
        if (q < kPlane) {
            const int v = q / kW, u = q - v * kW;
            // (a tile that ends before its 32nd column or row stages its halo
            // next to it; what lies beyond is clamped and not used)
            const int ux = POW2 ? u : min(u, a.L - x0 + 3), vy = POW2 ? v : min(v, a.L - y0 + 3);
            pr.v[j] = ld(src, site<POW2>(wrapped<POW2>(x0 - 2 + ux, a), wrapped<POW2>(y0 - 2 + vy, a), zz, a));
        }
    }
}

__device__ __forceinline__ int slot_of(int z) { return (z + 2 * kRing) % kRing; }  // z >= -2 * kRing

__device__ __forceinline__ void store_plane(float *ring, int slot, const PlaneRegs &pr) {
    float *P = ring + slot * 3 * kPlane;
#pragma unroll
    for (int j = 0; j < kLoadsPerThread; ++j) {
        const int q = (int)threadIdx.x + j * kTiledThreads;
        if (q < kPlane) {
            P[q] = pr.v[j].x;
            P[kPlane + q] = pr.v[j].y;
            P[2 * kPlane + q] = pr.v[j].z;
        }
    }
}

__device__ __forceinline__ F3 lds3(const float *ring, int slot, int q) {
    const float *P = ring + slot * 3 * kPlane;
    F3 r;
    r.x = P[q];
    r.y = P[kPlane + q];
    r.z = P[2 * kPlane + q];
    return r;
}

// First staged column u >= lo of staged row v whose site has colour c in plane z.
__device__ __forceinline__ int first_cell(int lo, int v, int c, int x0, int y0, int z) {
    return lo + ((c - (x0 - 2 + lo) - (y0 - 2 + v) - z) & 1);
}

// A thread's cell of a half-step: staged column u and row v, and the
// in-colour index of its site (the counter of its draw).
struct Cell {
    int u, v;
    bool on, own;  // updated at all; a site of the tile (not of its ring)
    uint32_t h;
};

template <bool POW2>
__device__ __forceinline__ uint32_t pair_of(int u, int v, int z, int x0, int y0, const TiledArgs &a) {
    return site<POW2>(wrapped<POW2>(x0 - 2 + u, a), wrapped<POW2>(y0 - 2 + v, a), wrapped<POW2>(z, a), a) >> 1;
}

// Colour 0 of plane z on the tile and on the one-site ring around it without
// the ring's corners (no tile site neighbours them): staged rows 1 and kW-2
// over columns [2, kW-2), rows 2 .. kW-3 over columns [1, kW-1).  That is
// kTile/2 + kTile*(kTile/2 + 1) + kTile/2 cells, one per thread.
constexpr int kRingRowCells = kTile / 2;
constexpr int kMidRowCells = kTile / 2 + 1;
constexpr int kColour0Cells = 2 * kRingRowCells + kTile * kMidRowCells;
static_assert(kColour0Cells == kTiledThreads, "one colour-0 cell per thread");

template <bool POW2>
__device__ __forceinline__ Cell cell0(int x0, int y0, int z, const TiledArgs &a) {
    const int tw = POW2 ? kTile : min(kTile, a.L - x0), th = POW2 ? kTile : min(kTile, a.L - y0);
    const int k = (int)threadIdx.x;
    int lo, j;
    Cell c;
    if (k < kRingRowCells) {
        c.v = 1, lo = 2, j = k;
    } else if (k < kRingRowCells + kTile * kMidRowCells) {
        const int kk = k - kRingRowCells;
        c.v = 2 + kk / kMidRowCells, lo = 1, j = kk % kMidRowCells;
    } else {
        c.v = th + 2, lo = 2, j = k - kRingRowCells - kTile * kMidRowCells;
    }
    c.u = first_cell(lo, c.v, 0, x0, y0, z) + 2 * j;
    c.on = POW2 || (c.u <= (lo == 1 ? tw + 2 : tw + 1) && (lo != 1 || c.v <= th + 1));
    c.own = c.on && c.u >= 2 && c.u < 2 + tw && c.v >= 2 && c.v < 2 + th;
    c.h = c.on ? pair_of<POW2>(c.u, c.v, z, x0, y0, a) : 0u;
    return c;
}

// Colour 1 of plane z on the tile: kTile * kTile / 2 cells, one per thread
// of the first kTile * kTile / 2.
template <bool POW2>
__device__ __forceinline__ Cell cell1(int x0, int y0, int z, const TiledArgs &a) {
    const int k = (int)threadIdx.x;
    Cell c;
    c.v = 2 + k / (kTile / 2);
    c.u = first_cell(2, c.v, 1, x0, y0, z) + 2 * (k % (kTile / 2));
    c.on = k < kTile * kTile / 2;
    if constexpr (!POW2) c.on = c.on && c.u <= min(kTile, a.L - x0) + 1 && c.v <= min(kTile, a.L - y0) + 1;
    c.own = c.on;
    c.h = c.on ? pair_of<POW2>(c.u, c.v, z, x0, y0, a) : 0u;
    return c;
}

// Updates the site of cell c of the plane in ring slot sz with the draw w;
// the planes below and above sit in slots sm and sp.  Returns whether it moved.
__device__ __forceinline__ bool update_cell(float *ring, int sm, int sz, int sp, const Cell &c, const uint4 &w,
                                            float beta) {
    const int q = c.v * kW + c.u;
    const F3 nx1 = lds3(ring, sz, q + 1), nx0 = lds3(ring, sz, q - 1);
    const F3 ny1 = lds3(ring, sz, q + kW), ny0 = lds3(ring, sz, q - kW);
    const F3 nz1 = lds3(ring, sp, q), nz0 = lds3(ring, sm, q);
    const F3 so = lds3(ring, sz, q);
    float3 hf = make_float3(0.f, 0.f, 0.f);
    hf.x += nx1.x; hf.y += nx1.y; hf.z += nx1.z;
    hf.x += nx0.x; hf.y += nx0.y; hf.z += nx0.z;
    hf.x += ny1.x; hf.y += ny1.y; hf.z += ny1.z;
    hf.x += ny0.x; hf.y += ny0.y; hf.z += ny0.z;
    hf.x += nz1.x; hf.y += nz1.y; hf.z += nz1.z;
    hf.x += nz0.x; hf.y += nz0.y; hf.z += nz0.z;
    const float3 sp3 = heis_proposal(unit23f(w.x), unit23f(w.y));
    const float dE = -((sp3.x - so.x) * hf.x + (sp3.y - so.y) * hf.y + (sp3.z - so.z) * hf.z);
    if (dE <= 0.0f || unit23f(w.z) < heis_boltzmann(beta, dE)) {
        float *P = ring + sz * 3 * kPlane;
        P[q] = sp3.x;
        P[kPlane + q] = sp3.y;
        P[2 * kPlane + q] = sp3.z;
        return true;
    }
    return false;
}

// POW2: L is a power of two (shifts and masks; whole tiles).
template <bool POW2>
__global__ __launch_bounds__(kTiledThreads) void k_heis3d_tiled(TiledArgs a) {
    extern __shared__ __align__(16) float ring[];  // [kRing][3][kPlane]
    __shared__ int red[kTiledThreads / 64];
    const int L = a.L;
    const int per_rep = a.tiles * a.tiles * a.segs;
    // Workgroups go to the XCDs round-robin; with the remap, XCD k runs a
    // contiguous range of logical blocks (whole segments), so the halo rows
    // and columns that neighbouring tiles share are fetched once into its L2.
    const uint32_t nblk = gridDim.x, b = blockIdx.x;
    const int lb = (int)((a.xcd_remap && (nblk & 7u) == 0) ? (b & 7u) * (nblk >> 3) + (b >> 3) : b);
    const int r = lb / per_rep;
    const int rem = lb % per_rep;
    const int seg = rem / (a.tiles * a.tiles), tile = rem % (a.tiles * a.tiles);
    const int x0 = (tile % a.tiles) * kTile, y0 = (tile / a.tiles) * kTile;
    const int z0 = seg * a.D, z1 = min(z0 + a.D, L);
    const float *src = a.src + (size_t)r * 3 * (size_t)a.N;
    float *dst = a.dst + (size_t)r * 3 * (size_t)a.N;
    const float beta = a.beta[r];

    // planes z0-2 .. z0 into their slots
    PlaneRegs pr;
    for (int z = z0 - 2; z <= z0; ++z) {
        load_plane<POW2>(src, a, x0, y0, z, pr);
        store_plane(ring, slot_of(z), pr);
    }
    __syncthreads();
    int n_acc = 0;
    for (int z = z0 - 1; z <= z1; ++z) {
        const bool fetch = z + 2 <= z1 + 1;
        if (fetch) load_plane<POW2>(src, a, x0, y0, z + 2, pr);
        // colour 0 of plane z on the tile and a one-site ring (planes z-1 .. z+1)
        const Cell c0 = cell0<POW2>(x0, y0, z, a);
        if (c0.on) {
            const uint4 w = philox4x32_10_wide(make_uint4(c0.h, a.t, (uint32_t)r, 2 * kTagHeis), a.key);
            if (update_cell(ring, slot_of(z - 1), slot_of(z), slot_of(z + 1), c0, w, beta))
                n_acc += c0.own && z >= z0 && z < z1 ? 1 : 0;
        }
        __syncthreads();
        // colour 1 of plane z-1 on the tile (planes z-2 .. z)
        if (z >= z0 + 1) {
            const Cell c1 = cell1<POW2>(x0, y0, z - 1, a);
            if (c1.on) {
                const uint4 w = philox4x32_10_wide(make_uint4(c1.h, a.t, (uint32_t)r, 2 * kTagHeis + 1u), a.key);
                n_acc += update_cell(ring, slot_of(z - 2), slot_of(z - 1), slot_of(z), c1, w, beta) ? 1 : 0;
            }
        }
        // plane z+2 into the slot of plane z-3.  The wait is explicit and on
        // every path, so that no load is left pending across the loop (the
        // next step's request would otherwise wait behind this step's stores).
        __builtin_amdgcn_s_waitcnt(0 | (7 << 4) | (15 << 8));  // vmcnt(0)
        if (fetch) store_plane(ring, slot_of(z + 2), pr);
        __syncthreads();
        if (z >= z0 + 1) {
            // the tile's plane z-1 out
            const int zc = z - 1;
            for (int k = threadIdx.x; k < kTile * kTile; k += kTiledThreads) {
                const int v = 2 + k / kTile, u = 2 + k % kTile;
                if constexpr (!POW2)
                    if (x0 + u - 2 >= L || y0 + v - 2 >= L) continue;
                F3 val = lds3(ring, slot_of(zc), v * kW + u);
                if (a.renorm) {
                    const float3 n = heis_unit(val.x, val.y, val.z);
                    val.x = n.x;
                    val.y = n.y;
                    val.z = n.z;
                }
                *(F3 *)(dst + 3 * (size_t)site<POW2>((uint32_t)(x0 + u - 2), (uint32_t)(y0 + v - 2), (uint32_t)zc, a)) =
                    val;
            }
        }
    }
    if (tally_wanted(a.acc)) {
        int v = n_acc;
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
        if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
        __syncthreads();
        if (threadIdx.x == 0) {
            int tot = 0;
            for (int w = 0; w < kTiledThreads / 64; ++w) tot += red[w];
            tally_put(a.acc, lb, r, tot);
        }
    }
}

}  // namespace

bool heis3d_supported(int dim, int L) { return dim == 3 && L >= 4 && L <= 1024 && (L & (L - 1)) == 0; }

int heis3d_half_groups(int L) {
    const int64_t pairs = (int64_t)L * L * L / 2;
    return (int)((pairs + kThreads * kSitesPerThread - 1) / (kThreads * kSitesPerThread));
}

hipError_t launch_heis3d_half(float *spins, const float *beta, const Tally &acc, int n_rep, int L, Key key, uint32_t t,
                              int c, hipStream_t s) {
    Heis3dArgs a;
    a.spins = spins;
    a.beta = beta;
    a.acc = acc;
    a.key = key;
    a.t = t;
    a.lgL = 0;
    while ((1 << a.lgL) < L) ++a.lgL;
    a.N = (int64_t)L * L * L;
    a.bpr = heis3d_half_groups(L);
    SMC_LAUNCH(k_heis3d_half, dim3((unsigned)(a.bpr * n_rep)), dim3(kThreads), 0, s, a, c);
    return hipGetLastError();
}

bool heis3d_tiled_supported(int dim, int L) { return dim == 3 && L % 2 == 0 && L >= kTile && L <= 1024; }

static int tiles_of(int L) { return (L + kTile - 1) / kTile; }

// Planes per segment.  A segment of D planes takes D + 2 steps after the
// planes of its prologue, and two workgroups share a compute unit: long
// segments recompute and reload fewer planes, short ones fill the chip.  The
// shortest total of rounds over 512 workgroups, one round at half the cost
// when the workgroups have a compute unit each.
int heis3d_tiled_planes(int L, int n_rep) {
    if (const char *e = getenv("SPINMC_HEIS_PLANES"))
        if (atoi(e) >= 2 && atoi(e) <= 1024) return atoi(e);
    int best = kMaxSeg;
    double least = 1e30;
    for (int D : {2, 3, 4, 6, 8, 12, 16, 24, kMaxSeg}) {
        const int64_t groups = (int64_t)tiles_of(L) * tiles_of(L) * ((L + D - 1) / D) * n_rep;
        const double cost = (groups <= 256 ? 0.6 : (double)((groups + 511) / 512)) * (D + 4);
        if (cost < least) {
            least = cost;
            best = D;
        }
    }
    return best;
}

int heis3d_tiled_groups(int L, int planes) { return tiles_of(L) * tiles_of(L) * ((L + planes - 1) / planes); }

size_t heis3d_tiled_lds_bytes() { return (size_t)kRing * 3 * kPlane * sizeof(float); }

hipError_t launch_heis3d_tiled(const float *src, float *dst, const float *beta, const Tally &acc, int n_rep, int L, Key key,
                               uint32_t t, bool renorm, int planes, hipStream_t s) {
    if (!heis3d_tiled_supported(3, L) || n_rep < 1 || planes < 2 || src == dst) return hipErrorInvalidValue;
    TiledArgs a;
    a.renorm = renorm ? 1 : 0;
    a.src = src;
    a.dst = dst;
    a.beta = beta;
    a.acc = acc;
    a.key = key;
    a.t = t;
    a.L = L;
    a.lgL = 0;
    while ((1 << a.lgL) < L) ++a.lgL;
    a.N = (int64_t)L * L * L;
    a.tiles = tiles_of(L);
    a.D = planes;
    a.segs = (L + planes - 1) / planes;
    {
        const char *e = getenv("SPINMC_XCD_REMAP");
        a.xcd_remap = (e && e[0] == '0') ? 0 : 1;
    }
    const size_t lds = heis3d_tiled_lds_bytes();
    const int64_t blocks = (int64_t)a.tiles * a.tiles * a.segs * n_rep;
    if (const char *why = launch_config_error((uint64_t)blocks, kTiledThreads, lds))
        return reject_launch("k_heis3d_tiled", (uint64_t)blocks, kTiledThreads, lds, why);
    if (L == 1 << a.lgL) {
        (void)hipFuncSetAttribute((const void *)k_heis3d_tiled<true>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                  (int)lds);
        SMC_LAUNCH(k_heis3d_tiled<true>, dim3((unsigned)blocks), dim3(kTiledThreads), lds, s, a);
    } else {
        (void)hipFuncSetAttribute((const void *)k_heis3d_tiled<false>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                  (int)lds);
        SMC_LAUNCH(k_heis3d_tiled<false>, dim3((unsigned)blocks), dim3(kTiledThreads), lds, s, a);
    }
    return hipGetLastError();
}

}  // namespace smc
