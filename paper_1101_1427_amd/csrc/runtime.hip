// The host runtime of the C-ABI layer (declared in runtime.hpp).
#include <math.h>
#include <stdarg.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <map>
#include <mutex>
#include <string>
#include <utility>
#include <vector>

#include "pairs3d.hpp"
#include "runtime.hpp"
#include "small3d.hpp"

namespace smc {

thread_local std::string g_launch_rejection;

hipError_t reject_launch(const char *kernel, uint64_t grid, uint64_t block, uint64_t lds, const char *why) {
    char buf[256];
    snprintf(buf, sizeof buf, "launch of %s refused (%s): %llu workgroups of %llu, %llu bytes of LDS", kernel, why,
             (unsigned long long)grid, (unsigned long long)block, (unsigned long long)lds);
    g_launch_rejection = buf;
    return hipErrorInvalidConfiguration;
}

std::string take_launch_rejection() {
    std::string r;
    r.swap(g_launch_rejection);
    return r;
}

namespace {
thread_local std::string g_last_error;
}  // namespace

std::string &last_error() { return g_last_error; }

int fail(int code, const char *fmt, ...) {
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    g_last_error = buf;
    return code;
}

// ------------------------------------------------------------------ scratch --

namespace {
std::mutex g_ctx_mutex;
std::map<std::pair<int, hipStream_t>, StreamCtx> g_ctx;
}  // namespace

StreamCtx &ctx_for(hipStream_t s) {
    int dev = 0;
    (void)hipGetDevice(&dev);
    std::lock_guard<std::mutex> lk(g_ctx_mutex);
    StreamCtx &c = g_ctx[std::make_pair(dev, s)];
    c.stream = s;
    return c;
}

// Device buffer of at least `bytes`.  Only calls on this set's stream use
// the buffer, so growing waits for that stream (not the whole device)
// before the old allocation is freed.
int ensure(StreamCtx &c, Slot slot, size_t bytes, void **out) {
    Buffer &b = c.dev[slot];
    if (b.bytes < bytes) {
        if (b.p) {
            SMC_HIP(hipStreamSynchronize(c.stream));
            SMC_HIP(hipFree(b.p));
            b.p = nullptr;
            b.bytes = 0;
        }
        b.last.clear();
        size_t want = bytes < 256 ? 256 : bytes;
        if (hipMalloc(&b.p, want) != hipSuccess) {
            (void)hipGetLastError();
            b.p = nullptr;
            return fail(SMC_ENOMEM, "could not allocate %zu bytes of scratch", want);
        }
        b.bytes = want;
    }
    *out = b.p;
    return SMC_OK;
}

bool spare_fits(size_t bytes, size_t held, size_t free_bytes) {
    return bytes <= held || bytes <= (free_bytes + held) / 2;
}

int ensure_spare(StreamCtx &c, size_t bytes, void **out) {
    const size_t held = c.dev[kLattices].bytes;
    if (bytes > held) {
        size_t free_bytes = 0, total = 0;
        SMC_HIP(hipMemGetInfo(&free_bytes, &total));
        if (!spare_fits(bytes, held, free_bytes))
            return fail(SMC_ENOMEM, "a copy of %zu bytes would take more than half of the free memory", bytes);
    }
    return ensure(c, kLattices, bytes, out);
}

int release(StreamCtx &c, Slot slot) {
    Buffer &b = c.dev[slot];
    if (b.p) {
        SMC_HIP(hipStreamSynchronize(c.stream));
        SMC_HIP(hipFree(b.p));
    }
    b.p = nullptr;
    b.bytes = 0;
    b.last.clear();
    return SMC_OK;
}

// Copy host bytes into a device scratch slot through that slot's pinned
// staging area.  The staging area is reused only after its previous copy has
// completed; an upload identical to the slot's previous one is skipped (the
// device copy is only ever written by uploads, in stream order).
int upload(StreamCtx &c, hipStream_t s, Slot slot, const void *src, size_t bytes, void **dev_out) {
    int rc = ensure(c, slot, bytes, dev_out);
    if (rc) return rc;
    Buffer &b = c.dev[slot];
    if (b.last.size() == bytes && memcmp(b.last.data(), src, bytes) == 0) return SMC_OK;
    if (b.staged_pending) {
        SMC_HIP(hipEventSynchronize(b.staged));
        b.staged_pending = false;
    }
    if (b.pinned_bytes < bytes) {
        if (b.pinned) SMC_HIP(hipHostFree(b.pinned));
        b.pinned = nullptr;
        b.pinned_bytes = 0;
        size_t want = bytes < 4096 ? 4096 : bytes;
        if (hipHostMalloc(&b.pinned, want, hipHostMallocDefault) != hipSuccess) {
            (void)hipGetLastError();
            b.pinned = nullptr;
            return fail(SMC_ENOMEM, "could not allocate %zu bytes of pinned staging", want);
        }
        b.pinned_bytes = want;
    }
    if (!b.staged) SMC_HIP(hipEventCreateWithFlags(&b.staged, hipEventDisableTiming));
    memcpy(b.pinned, src, bytes);
    b.last.assign((const unsigned char *)src, (const unsigned char *)src + bytes);
    SMC_HIP(hipMemcpyAsync(*dev_out, b.pinned, bytes, hipMemcpyHostToDevice, s));
    SMC_HIP(hipEventRecord(b.staged, s));
    b.staged_pending = true;
    return SMC_OK;
}

// Calls stage host data (tables, instance lists) through pinned buffers and
// grow their scratch on demand; neither can be recorded into a caller's
// stream capture, so a call on a capturing stream is refused before anything
// is issued.
int refuse_capture(hipStream_t s) {
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    SMC_HIP(hipStreamIsCapturing(s, &cap));
    if (cap != hipStreamCaptureStatusNone)
        return fail(SMC_EINVAL, "the stream is capturing a graph: this call cannot be captured");
    return SMC_OK;
}

// ----------------------------------------------------------------- tables ----
// thr[m] = floor(2^32 exp(-4 m beta)) for Delta E = 4m > 0, computed in
// float64 with the C library's exp and split as (thr >> 16, thr & 0xffff).
ThrRow threshold_row(double beta, int dim) {
    ThrRow row;
    row.m[0] = make_uint2(65536u, 0u);
    for (int m = 1; m <= 3; ++m) {
        uint64_t thr = 0;
        if (m <= dim) {
            const double p = exp(-beta * (4.0 * m));
            thr = (uint64_t)floor(4294967296.0 * p);
        }
        row.m[m] = make_uint2((uint32_t)(thr >> 16), (uint32_t)(thr & 0xFFFFu));
    }
    return row;
}

// Uniform 3D Heisenberg batches with a power-of-two edge take the indexed
// kernel (SPINMC_HEIS3D=0 sends them to the generic one).
bool use_heis3d(const smc_desc *d) {
    const char *env = getenv("SPINMC_HEIS3D");
    if (env && env[0] == '0') return false;
    return d->model == SMC_HEISENBERG && d->L > 0 && heis3d_supported(d->dim, d->L);
}

// Small uniform Heisenberg lattices keep whole replicas in LDS for a call where an estimate
// says that it is faster: a sweep takes a compute unit 1 us and 0.95 ns per site of its
// replica (half as much again once for loads and stores), the half-sweep launches 8.5 us
// and 15 ps per site of the batch (one 22^3 lattice 11.1 against 9.2 us, 50 of them 11.3
// against 17.9).  SPINMC_HEIS_SMALL=0 and SPINMC_HEIS3D=0 keep the half-sweeps, =1 takes this
// kernel wherever it fits (same results).
bool use_heis_small(const smc_desc *d, int64_t n_sweeps) {
    for (const char *name : {"SPINMC_HEIS_SMALL", "SPINMC_HEIS3D"}) {
        const char *env = getenv(name);
        if (env && env[0] == '0') return false;
    }
    if (d->model != SMC_HEISENBERG || d->L <= 0 || !heis_small_supported(d->dim, d->L)) return false;
    const char *env = getenv("SPINMC_HEIS_SMALL");
    if (env && env[0] == '1') return true;
    const double N = d->dim == 3 ? (double)d->L * d->L * d->L : (double)d->L * d->L;
    const double small = (1.0 + 0.95e-3 * N + 0.5e-3 * N / (double)n_sweeps) * ((d->n_rep + 255) / 256);
    return small < 8.5 + 15e-6 * N * d->n_rep;
}

// ... and those with any even edge of at least 32 the one-pass tiled kernel
// (SPINMC_HEIS_TILED=0 keeps the two half-sweep launches).
bool use_heis3d_tiled(const smc_desc *d, int64_t n_sweeps) {
    const char *env = getenv("SPINMC_HEIS_TILED");
    if (env && env[0] == '0') return false;
    const char *all = getenv("SPINMC_HEIS3D");
    if (all && all[0] == '0') return false;
    if (d->model != SMC_HEISENBERG || d->L <= 0 || !heis3d_tiled_supported(d->dim, d->L)) return false;
    // few sites: two small half-sweep launches are as fast as the tiles' plane
    // steps (46^3: 9.7 against 11.3 us per sweep; 64^3 level, 96^3 31 against 16)
    if (heis3d_supported(d->dim, d->L)) return true;
    // an odd number of sweeps ends with a copy back, which edges that waste most of their tiles
    // do not make up for in one sweep, nor, where the batch fills the chip, in three (64 of 34^3
    // 85 against 75 and 224 against 208 us, ten sweeps 708 against 740; eight of 34^3, three
    // sweeps, 60 against 77; 64 of 40^3, one sweep, 88 against 109)
    const int64_t tiled = (d->L + 31) / 32 * 32, sites = (int64_t)d->n_rep * d->L * d->L * d->L;
    if (tiled * tiled * 10 > (int64_t)d->L * d->L * 28 &&
        (n_sweeps == 1 || (n_sweeps == 3 && sites >= (int64_t)1 << 21)))
        return false;
    return sites >= (int64_t)1 << 18;
}

// Uniform 3D Ising / EA batches with an edge of 4 .. 24 or 32 keep whole replicas
// in LDS for a call (any alignment, any beta); SPINMC_SMALL3D=0 keeps them on
// the half-sweep launches, =1 tempering here whatever the estimate (same
// results).
bool use_small3d(const smc_desc *d) {
    const char *env = getenv("SPINMC_SMALL3D");
    if (env && env[0] == '0') return false;
    return (d->model == SMC_ISING || d->model == SMC_EA) && d->L > 0 && small3d_supported(d->dim, d->L);
}

bool use_pt3d(const smc_desc *d, int n_temps) {
    const char *env = getenv("SPINMC_PT3D");
    if (env && env[0] == '0') return false;
    return (d->model == SMC_ISING || d->model == SMC_EA) && d->dim == 3 && d->L == 16 && n_temps >= 2 &&
           n_temps <= 32 && !(d->model == SMC_EA && d->rep_per_sample % n_temps);
}

bool use_small3d_pt(const smc_desc *d, int n_temps, int n_chains) {
    if (use_pt3d(d, n_temps)) return true;
    const char *env = getenv("SPINMC_PT3D");
    if (d->L == 16 && env && env[0] == '0') return false;
    return use_small3d(d) && n_temps <= small3d_max_reps(d->L) && small3d_tempers(d->L, n_temps, n_chains);
}

// The one-pass split-layout kernel serves uniform 2D Ising batches whose
// edge it supports, with 16-byte aligned spins and thresholds below 2^32
// (beta > 0 up to rounding; the generic kernels cover the rest).
bool use_lattice2d(const smc_desc *d, const void *spins, const std::vector<ThrRow> &rows) {
    if (d->model != SMC_ISING || d->dim != 2 || d->L <= 0 || !lattice2d_supported(d->L)) return false;
    if (((uintptr_t)spins & 15u) != 0) return false;
    for (const ThrRow &r : rows)
        if (r.m[1].x > 0xFFFFu || r.m[2].x > 0xFFFFu) return false;
    return true;
}

// Edges that the one-pass kernel (lattice2d.hip) serves: up to 2^25 sites and edge
// 4096 the tiles are faster, because they move the lattice once per several
// sweeps and need one launch for them (1024^2: 1.7 against 6.4 us per sweep,
// eight of 2048^2: 18.8 against 32.6, 4096^2: 9.8 against 13.3); above, the one-pass kernel's
// fewer instructions per site win (16 of 2048^2: 36.3 against 39.2, 8192^2: 34 against 40).
// A call needs sweeps enough for the tiles' even number of launches, the more the fuller they
// are.  2048^2 from 2^23 sites on 3 (2 sweeps of 4 lattices 46 against 41 us, 3 of them 55 and
// 60) and from 2^24 on 4 (3 of 6 lattices 70 and 61, 4 of 8 115 and 134); 1024^2, where the one-pass
// kernel is a quarter faster per site, 2, 3 and from 24 2^20 on 6 (2 of 24 lattices 58 and 52, 3
// of them 67 and 76; 5 of 32 130 and 126, 6 of them 146 and 151); 4096^2 8 and from 2^24 on 12 (two
// lattices: 10 sweeps 212 and 208, 12 of them 242 and 249).  Tempering, where the one-pass kernel
// needs four more launches per step, takes tiles from one sweep per step on (4096^2: 8).
// A launch shape asked for in the environment is the one-pass kernel's.
bool bands_before_lattice2d(const smc_desc *d, int32_t n_sweeps, bool tempering) {
    for (const char *name : {"SPINMC_L2D_CHUNKS", "SPINMC_L2D_H", "SPINMC_L2D_H1", "SPINMC_L2D_H2", "SPINMC_L2D_PAD",
                             "SPINMC_L2D_FUSE"})
        if (getenv(name)) return false;
    const char *env = getenv("SPINMC_BANDS2D");
    if (env && env[0] == '1') return true;
    const int64_t sites = (int64_t)d->n_rep * d->L * d->L, M = 1 << 20;
    if (d->L > 4096 || sites > 32 * M) return false;
    if (d->L > 2048) return n_sweeps >= (tempering || sites <= 16 * M ? 8 : 12);
    if (tempering || sites <= 8 * M) return true;
    return n_sweeps >= (d->L > 1024 ? (sites <= 16 * M ? 3 : 4) : (sites <= 16 * M ? 2 : sites <= 24 * M ? 3 : 6));
}

// Uniform 3D Ising / EA batches with an edge that is a multiple of 16 take
// the segment-per-thread half-sweeps when spins (and couplings) are 16-byte
// aligned and every threshold has a 16-bit high half; SPINMC_SWEEP3D=0 keeps
// them on the generic kernels (same results).
bool sweep3d_shape(const smc_desc *d) {
    const char *env = getenv("SPINMC_SWEEP3D");
    if (env && env[0] == '0') return false;
    return d->dim == 3 && d->L > 0 && (d->model == SMC_ISING || d->model == SMC_EA) && sweep3d_supported(d->L);
}

// ... and, with an edge of 512 .. 1024, the one-pass sweep (below 512 its
// strips are too few to fill the chip and the two half-sweep launches are
// faster; SPINMC_SWEEP3D_PASS=1 takes it for every edge of 32 .. 1024 it
// supports, SPINMC_SWEEP3D_PASS=0 never).
bool pass3d_enabled(const smc_desc *d) {
    const char *env = getenv("SPINMC_SWEEP3D_PASS");
    if (env && env[0] == '0') return false;
    if (!(env && env[0] == '1') && d->L < 512) return false;
    return pass3d_supported(d->L);
}

bool use_sweep3d(const smc_desc *d, const void *spins, const int8_t *coup, const std::vector<ThrRow> &rows) {
    if (!sweep3d_shape(d)) return false;
    if (((uintptr_t)spins & 15u) != 0 || (d->model == SMC_EA && ((uintptr_t)coup & 15u) != 0)) return false;
    for (const ThrRow &r : rows)
        if (r.m[1].x > 0xFFFFu || r.m[2].x > 0xFFFFu || r.m[3].x > 0xFFFFu) return false;
    return true;
}

// 3D batches of edge 16 and more run calls of several sweeps on a packed copy
// of their lattices (packing and unpacking take about as long as one
// sweep saves two or three times over; against the one-pass kernel of Ising edges from
// 512, five times).  Per sweep, packing included, against the kernels on the caller's
// bytes: EA 256^3 24.0 -> 15.3 us (20 sweeps), 512^3 143 -> 82 (10), 1024^3 1000 -> 702 (6),
// Ising 512^3 92 -> 68 (10), 768^3 290 -> 226 (6); Ising 1024^3 stays (565 and, with tuned
// strips, 545 against 544 and more).
// Short calls on small lattices are bound by their launches, of which packing and unpacking
// are two: up to seven sweeps of fewer than 2^22 sites in all, of ragged rows 2^20, stay on the
// caller's bytes (three of one 48^3 Ising lattice, call and wait: 60 us with the copy, 39
// without; five of one 96^3 90 and 66, throughput 43 and 47; eight of one 64^3 110 and 82,
// throughput 60 and 65; three of 32 of 26^3 EA 61 and 53, throughput 31 and 40).
// SPINMC_PAIRS3D=0 keeps the kernels on the caller's bytes (same results), and
// so does a launch shape of those asked for in the environment.
bool sweep3d_asked_for() {
    for (const char *name : {"SPINMC_SWEEP3D", "SPINMC_SWEEP3D_Z", "SPINMC_SWEEP3D_PASS", "SPINMC_SWEEP3D_NT",
                             "SPINMC_SWEEP3D_PACK"})
        if (getenv(name)) return true;
    return false;
}

bool use_pairs3d(const smc_desc *d, int64_t n_sweeps) {
    const char *env = getenv("SPINMC_PAIRS3D");
    if ((env && env[0] == '0') || d->L <= 0 || (d->model != SMC_ISING && d->model != SMC_EA) ||
        !pairs3d_supported(d->dim, d->L) || !pairs3d_launchable(d->L, d->n_rep))
        return false;
    if (env && env[0] == '1') return true;
    if (n_sweeps < 8 && n_sweeps * d->n_rep * sites(3, d->L) < (int64_t)1 << (d->L % 16 ? 20 : 22)) return false;
    if (d->L % 16) return n_sweeps >= 2;
    if (sweep3d_asked_for()) return false;
    if (d->model == SMC_ISING && pass3d_enabled(d)) return n_sweeps >= 6 && d->L < 1024;
    return n_sweeps >= 3 && d->L >= 32;
}

// Tempering of a uniform 2D Ising batch on the one-pass colour-split sweep:
// L a power of two in [1024, 16384], aligned spins, thresholds of every
// temperature with 16-bit high halves; SPINMC_PT_SPLIT2D=0 sends such
// batches to the generic kernels (same results).
bool use_pt_split2d(const smc_desc *d, const void *spins, const std::vector<ThrRow> &rows) {
    const char *env = getenv("SPINMC_PT_SPLIT2D");
    if (env && env[0] == '0') return false;
    return use_lattice2d(d, spins, rows);
}

// --------------------------------------------------------------- validation --

int64_t sites(int dim, int L) { return dim == 3 ? (int64_t)L * L * L : (int64_t)L * L; }

// The coupling samples of a uniform EA batch: sample q at q * d * N.
void fill_uniform_samples(const smc_desc *d, Plan &plan) {
    if (d->L <= 0 || d->model != SMC_EA || !plan.samples.empty()) return;
    plan.samples.resize((size_t)plan.n_samples);
    for (int64_t q = 0; q < plan.n_samples; ++q) {
        smc_inst &g = plan.samples[(size_t)q];
        g.L = d->L;
        g.sample = (int32_t)q;
        g.spin_off = 0;
        g.coup_off = q * d->dim * plan.b.N;
    }
}

// A piece of 16 sites spans at most two rows when every edge is at least 16.  Where rows end inside
// pieces a thread takes half as long again as where they do not, which counts once the
// chip is full: below 2^18 (2D) or 2^19 (3D) sites in the batch a thread per pair of sites is
// faster (per half-sweep with one and with the other, 2D EA: one 50^2 lattice 4.4 and 3.9 us, 16
// of 100^2 5.2 and 4.6, 64 of 100^2 5.6 and 6.0; 3D EA: one 18^3 6.2 and 4.3, one 50^3 6.2
// and 4.7, four 6.5 and 6.1, eight 6.8 and 8.2; Ising 26^3 5.3 and 4.9, 64 of them 6.1 and 8.3).
PieceUse piece_use(int dim, int min_L, bool ragged, int64_t all_sites) {
    if (min_L < 16) return kNoPieces;
    return !ragged || all_sites >= (int64_t)1 << (dim == 3 ? 19 : 18) ? kPieces : kFewPieces;
}

int validate(const smc_desc *d, bool need_coup, Plan &plan) {
    if (!d) return fail(SMC_EINVAL, "desc is NULL");
    if (d->model < SMC_ISING || d->model > SMC_HEISENBERG) return fail(SMC_EINVAL, "unknown model %d", d->model);
    if (d->dim != 2 && d->dim != 3) return fail(SMC_EINVAL, "dim must be 2 or 3 (got %d)", d->dim);
    if (d->n_rep < 1) return fail(SMC_EINVAL, "n_rep must be >= 1 (got %d)", d->n_rep);
    if (d->spins_len <= 0) return fail(SMC_EINVAL, "spins_len must be > 0");
    if (d->model == SMC_HEISENBERG && d->renorm_every < 0) return fail(SMC_EINVAL, "renorm_every must be >= 0");
    const bool ea = d->model == SMC_EA;
    const int per_site = d->model == SMC_HEISENBERG ? 3 : 1;
    Batch &b = plan.b;
    b.dim = d->dim;
    b.model = d->model;
    b.n_rep = d->n_rep;
    b.L = d->L;
    b.rep_per_sample = 1;
    b.inst = nullptr;
    b.N = 0;
    plan.samples.clear();
    if (d->L > 0) {
        if (d->inst) return fail(SMC_EINVAL, "inst must be NULL for a uniform batch (L > 0)");
        if (d->L % 2 || d->L < 4) return fail(SMC_EINVAL, "L must be even and >= 4 (got %d)", d->L);
        if (d->L > (d->dim == 3 ? 1024 : 65536)) return fail(SMC_EINVAL, "L too large (got %d)", d->L);
        b.N = sites(d->dim, d->L);
        if (b.N / 2 > 0xFFFFFFFFll) return fail(SMC_EINVAL, "lattice too large for 32-bit site counters");
        plan.max_L = d->L;
        plan.pieces = piece_use(d->dim, d->L, d->L % 16 != 0, (int64_t)d->n_rep * b.N);
        if ((int64_t)d->n_rep * b.N * per_site > d->spins_len)
            return fail(SMC_EINVAL, "spin buffer too small: need %lld elements, have %lld",
                        (long long)((int64_t)d->n_rep * b.N * per_site), (long long)d->spins_len);
        if (ea) {
            if (d->rep_per_sample < 1) return fail(SMC_EINVAL, "rep_per_sample must be >= 1 for EA");
            b.rep_per_sample = d->rep_per_sample;
            plan.n_samples = (d->n_rep + d->rep_per_sample - 1) / d->rep_per_sample;
            // the sample table is built only where a path needs it (fill_uniform_samples)
            if (need_coup) {
                if (d->coup_len <= 0) return fail(SMC_EINVAL, "coup_len must be > 0 for EA");
                if (plan.n_samples * d->dim * b.N > d->coup_len)
                    return fail(SMC_EINVAL, "couplings of sample %lld lie outside the coupling buffer",
                                (long long)(d->coup_len / (d->dim * b.N)));
            }
        }
    } else {
        if (!d->inst) return fail(SMC_EINVAL, "inst is required when L == 0");
        std::map<int32_t, smc_inst> seen;
        int min_L = 0;
        bool ragged = false;
        int64_t all = 0;
        for (int r = 0; r < d->n_rep; ++r) {
            const smc_inst &g = d->inst[r];
            if (g.L % 2 || g.L < 4 || g.L > (d->dim == 3 ? 1024 : 65536))
                return fail(SMC_EINVAL, "inst[%d].L must be even and in [4, limit] (got %d)", r, g.L);
            const int64_t N = sites(d->dim, g.L);
            if (g.spin_off < 0 || g.spin_off > d->spins_len / per_site - N)
                return fail(SMC_EINVAL, "inst[%d] spins lie outside the spin buffer", r);
            if (ea) {
                if (g.sample < 0) return fail(SMC_EINVAL, "inst[%d].sample must be >= 0", r);
                auto it = seen.find(g.sample);
                if (it == seen.end()) {
                    seen[g.sample] = g;
                } else if (it->second.L != g.L || it->second.coup_off != g.coup_off) {
                    return fail(SMC_EINVAL, "inst[%d]: sample %d used with two geometries", r, g.sample);
                }
            }
            if (g.L > plan.max_L) plan.max_L = g.L;
            if (r == 0 || g.L < min_L) min_L = g.L;
            ragged |= g.L % 16 != 0;
            all += N;
        }
        plan.pieces = piece_use(d->dim, min_L, ragged, all);
        for (auto &kv : seen) plan.samples.push_back(kv.second);
        plan.n_samples = (int64_t)plan.samples.size();
    }
    if (ea && need_coup && d->L == 0) {
        if (d->coup_len <= 0) return fail(SMC_EINVAL, "coup_len must be > 0 for EA");
        for (const smc_inst &g : plan.samples) {
            const int64_t need = (int64_t)d->dim * sites(d->dim, g.L);
            if (g.coup_off < 0 || g.coup_off > d->coup_len - need)
                return fail(SMC_EINVAL, "couplings of sample %d lie outside the coupling buffer", g.sample);
        }
    }
    return SMC_OK;
}

int upload_inst(StreamCtx &c, hipStream_t s, const smc_desc *d, Plan &plan) {
    if (d->L > 0) return SMC_OK;
    void *p = nullptr;
    int rc = upload(c, s, kInst, d->inst, sizeof(smc_inst) * (size_t)d->n_rep, &p);
    plan.b.inst = (const smc_inst *)p;
    return rc;
}

}  // namespace smc
