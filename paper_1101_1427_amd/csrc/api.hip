// C-ABI layer of libspinmc.so: argument validation, acceptance tables,
// per-stream scratch, and dispatch to the sweep / exchange kernels.
#include <math.h>
#include <stdarg.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <algorithm>
#include <functional>
#include <map>
#include <mutex>
#include <string>
#include <tuple>
#include <utility>
#include <vector>

#include "bands2d.hpp"
#include "bins2d.hpp"
#include "internal.hpp"
#include "pairs3d.hpp"
#include "runtime.hpp"
#include "small3d.hpp"

namespace smc {
namespace {

// ------------------------------------------------ uneven 2D tempering ----
// Tempering of 2D batches with edges in {16, 32, ..., 256}, uniform or uneven,
// goes to the bins of replicas.
bool use_uneven2d(const smc_desc *d, const void *spins, const int8_t *coup, const std::vector<ThrRow> &rows) {
    if (d->dim != 2 || (d->model != SMC_ISING && d->model != SMC_EA)) return false;
    const char *env = getenv("SPINMC_UNEVEN2D");
    if (env && env[0] == '0') return false;
    if (((uintptr_t)spins & 15u) != 0) return false;
    if (d->model == SMC_EA && ((uintptr_t)coup & 15u) != 0) return false;
    for (const ThrRow &r : rows)
        if (r.m[1].x > 0xFFFFu || r.m[2].x > 0xFFFFu) return false;
    if (d->L > 0) return uneven2d_edge_supported(d->L);
    for (int r = 0; r < d->n_rep; ++r) {
        const smc_inst &g = d->inst[r];
        if (!uneven2d_edge_supported(g.L) || g.spin_off % 16) return false;
        if (d->model == SMC_EA && g.coup_off % 16) return false;
    }
    return true;
}

std::vector<smc_inst> inst_rows(const smc_desc *d) {
    std::vector<smc_inst> rows(d->n_rep);
    const int64_t N = (int64_t)d->L * d->L;
    for (int r = 0; r < d->n_rep; ++r) {
        if (d->L > 0) {
            rows[r].L = d->L;
            rows[r].sample = d->model == SMC_EA ? r / d->rep_per_sample : 0;
            rows[r].spin_off = (int64_t)r * N;
            rows[r].coup_off = (int64_t)rows[r].sample * 2 * N;
        } else {
            rows[r] = d->inst[r];
        }
    }
    return rows;
}

int run_uneven2d(StreamCtx &c, hipStream_t s, const smc_desc *desc, void *spins, const int8_t *couplings,
                 SwapArgs &sw, const ThrRow *thr, double *energy, uint64_t step0, int32_t n_steps, int m) {
    int rc;
    const std::vector<smc_inst> rows = inst_rows(desc);
    std::vector<Bin2d> bins;
    std::vector<int32_t> work;
    const size_t lds = make_bins2d(rows, &bins, &work);
    void *ip = nullptr, *bp = nullptr, *wp = nullptr, *pp = nullptr;
    if ((rc = upload(c, s, kInst, rows.data(), sizeof(smc_inst) * rows.size(), &ip))) return rc;
    if ((rc = upload(c, s, kBins2d, bins.data(), sizeof(Bin2d) * bins.size(), &bp))) return rc;
    if ((rc = upload(c, s, kWork, work.data(), sizeof(int32_t) * work.size(), &wp))) return rc;
    // Between the steps of a call the replicas stay in a packed copy; without
    // room for it every step reads and writes the caller's arrays.
    const Bin2d &end = bins.back();
    if (n_steps > 1 && ensure_spare(c, (size_t)(end.packed + (int64_t)end.count * end.L * end.L / 2), &pp)) {
        last_error().clear();
        pp = nullptr;
    }
    Bins2dArgs a;
    a.spins = (int8_t *)spins;
    a.coup = desc->model == SMC_EA ? couplings : nullptr;
    a.packed = (uint8_t *)pp;
    a.inst = (const smc_inst *)ip;
    a.bins = (const Bin2d *)bp;
    a.work = (const int32_t *)wp;
    a.thr = thr;
    a.n_temps = sw.n_temps;
    a.beta_per_chain = sw.beta_per_chain;
    a.beta = sw.beta;
    a.acc = sw.acc;
    a.key = make_key(desc->seed);
    a.sweeps = m;
    // the chains' state twice: a launch reads one and writes the other
    const size_t n_rep = (size_t)desc->n_rep;
    void *ep = nullptr, *rp = nullptr;
    if ((rc = ensure(c, kEnergy64, 2 * sizeof(int64_t) * n_rep, &ep))) return rc;
    if ((rc = ensure(c, kRows, 3 * sizeof(int32_t) * n_rep, &rp))) return rc;
    int32_t *const caller = sw.slot_of_temp;
    int64_t *E[2] = {(int64_t *)ep, (int64_t *)ep + n_rep};
    int32_t *row[2] = {(int32_t *)rp, (int32_t *)rp + n_rep}, *slot[2] = {caller, (int32_t *)rp + 2 * n_rep};
    int e = 0, p = 0;  // the current ones
    const bool fused = bins.size() <= kBinsAtOnce;  // exchange rounds at the start of the next step's launch
    auto round = [&](uint32_t t) {
        sw.E = E[e];
        sw.row_of_rep = row[p];
        sw.slot_of_temp = slot[p];
        sw.t = t;
        return launch_pt_swap(sw, s);
    };
    sw.E = E[0];
    sw.row_of_rep = row[0];
    SMC_HIP(launch_pt_prepare(sw, energy, s));
    for (int32_t k = 0; k < n_steps; ++k) {
        const uint32_t t = (uint32_t)(step0 + (uint64_t)k);
        a.t = t * (uint32_t)m;
        a.swap = fused && k > 0 ? 1 : 0;
        a.swap_t = t - 1u;
        a.row_in = row[p];
        a.slot_in = slot[p];
        a.row_out = row[1 - p];
        a.slot_out = slot[1 - p];
        a.E_in = E[e];
        a.E_out = E[1 - e];
        SMC_HIP(launch_bins2d(a, (int)bins.size(), lds, !pp || k == 0, !pp || k == n_steps - 1, s));
        e = 1 - e;
        if (a.swap) p = 1 - p;
        if (!fused || k == n_steps - 1) SMC_HIP(round(t));
    }
    SMC_HIP(launch_pt_finish(sw, energy, s, p ? caller : nullptr));
    return SMC_OK;
}

// Event pairs around the sweep kernels of each call (profiling aid).
struct TimedCall {
    hipEvent_t start, stop;
    int64_t launches;
};
std::mutex g_timing_mutex;
bool g_timing_on = false;
std::vector<TimedCall> g_timed;

void forget_timed() {
    for (TimedCall &c : g_timed) {
        (void)hipEventDestroy(c.start);
        (void)hipEventDestroy(c.stop);
    }
    g_timed.clear();
}

// Records the start event on construction and the stop event on finish().
struct SweepTimer {
    hipStream_t s;
    TimedCall call{nullptr, nullptr, 0};
    bool on = false;
    SweepTimer(hipStream_t stream, int64_t launches) : s(stream) {
        std::lock_guard<std::mutex> lk(g_timing_mutex);
        if (!g_timing_on) return;
        call.launches = launches;
        if (hipEventCreate(&call.start) != hipSuccess) return;
        if (hipEventCreate(&call.stop) != hipSuccess) {
            (void)hipEventDestroy(call.start);
            return;
        }
        on = hipEventRecord(call.start, s) == hipSuccess;
        if (!on) {
            (void)hipEventDestroy(call.start);
            (void)hipEventDestroy(call.stop);
        }
    }
    void finish() {
        if (!on) return;
        on = false;
        std::lock_guard<std::mutex> lk(g_timing_mutex);
        if (hipEventRecord(call.stop, s) == hipSuccess && g_timing_on) {
            g_timed.push_back(call);
        } else {
            (void)hipEventDestroy(call.start);
            (void)hipEventDestroy(call.stop);
        }
    }
    ~SweepTimer() { finish(); }
};

// Small uniform 2D batches of edge 16 .. 128 (a multiple of 16), and of edge
// 256 with at least 2^19 sites, whose path has its own name in the plans and
// its own switch: SPINMC_SWEEP_LDS2D=0 sends them to the half-sweeps.
bool small2d_shape(const smc_desc *d) {
    if (d->dim != 2 || d->L <= 0 || (d->model != SMC_ISING && d->model != SMC_EA) || !uneven2d_edge_supported(d->L))
        return false;
    return d->L <= 128 || (int64_t)d->n_rep * d->L * d->L >= (int64_t)1 << 19;
}

bool small2d_enabled() {
    const char *env = getenv("SPINMC_SWEEP_LDS2D");
    return !(env && env[0] == '0');
}

// The per-replica sums of one sweep call.  With fewer than 16 workgroups per
// replica and launch, or at most 32 in all, or 256 over the launches, they add to the
// caller's total directly (the collecting launch takes 2 to 4 us: one 48^3 Ising lattice, 27
// workgroups, one sweep 12.1 -> 8.3 us, ten 76.9 -> 74.9; one sweep of two lattices of 64 workgroups
// 12.7 -> 10.4, of four of 35 11.8 and 11.5, three of them 28.7 and 32.3); otherwise each keeps
// a slot, collected once by finish() (four lattices of 64 workgroups each, ten sweeps: 142 us
// without slots, 104 with them, 64 of 32 each 257 and 161).
bool few_groups(int groups, int n_rep, int64_t launches) {
    const int64_t all = (int64_t)groups * n_rep;
    return groups < 16 || all <= 32 || all * launches <= 256;
}

struct CallTally {
    Tally t{nullptr, nullptr, 0};
    int n_rep = 0, groups = 0;

    int begin(StreamCtx &c, int reps, int groups_per_rep, int64_t launches, int64_t *total) {
        n_rep = reps;
        groups = groups_per_rep;
        t.total = total;
        t.first = 1;
        if (!total || few_groups(groups, reps, launches)) return SMC_OK;
        void *p = nullptr;
        if (int rc = ensure(c, kTallySlots, sizeof(int64_t) * (size_t)n_rep * (size_t)groups, &p)) return rc;
        t.slots = (int64_t *)p;
        return SMC_OK;
    }
    // The tally of the next launch.
    Tally next() {
        const Tally now = t;
        t.first = 0;
        return now;
    }
    int finish(hipStream_t s) {
        if (t.slots) SMC_HIP(launch_collect(t.slots, t.total, n_rep, groups, false, s));
        return SMC_OK;
    }
};

// Uniform 2D batches run several sweeps per launch on bands of rows in LDS
// where the estimate says that it is faster than two half-sweep launches per
// sweep (measured: about 3.5 us and 1.2 ps per site each).  Edges that are
// multiples of 16 are cut along their rows too; others in bands of whole rows of half
// a byte per site, of which large edges have too few in LDS, so they keep the
// half-sweeps.  So does a call of one sweep unless the lattice fits in LDS as a whole.
// SPINMC_BANDS2D=0 keeps the half-sweeps (same results), and so does
// SPINMC_PT_SPLIT2D=0 in tempering (even is false there).
bool use_bands2d(const smc_desc *d, int32_t n_sweeps, bool even, BandShape *sh) {
    const char *env = getenv("SPINMC_BANDS2D");
    if ((env && env[0] == '0') || d->dim != 2 || d->L <= 0 || d->model == SMC_HEISENBERG) return false;
    const bool forced = env && env[0] == '1';
    if (!forced && small2d_shape(d) && !small2d_enabled()) return false;
    const char *split = getenv("SPINMC_PT_SPLIT2D");
    if (!forced && !even && split && split[0] == '0') return false;
    if (!bands2d_shape(d->L, d->n_rep, d->model == SMC_EA, n_sweeps, even, sh)) return false;
    return forced || sh->ns_per_sweep < 2.0 * (3500.0 + 1.2e-3 * (double)d->n_rep * (double)sites(2, d->L));
}

// Sweeps on bands, from a.spins to `other` and back, launch by launch.
struct BandRun {
    Bands2dArgs ba;
    BandShape sh;
    int8_t *lattice[2];
    int at = 0;  // the lattice that holds the spins

    BandRun(const SweepArgs &a, const BandShape &shape, void *other) : sh(shape) {
        lattice[0] = (int8_t *)a.spins;
        lattice[1] = shape.whole ? (int8_t *)a.spins : (int8_t *)other;
        ba.coup = a.coup;
        ba.rep_per_sample = a.b.rep_per_sample;
        ba.thr = a.thr;
        ba.row_of_rep = a.row_of_rep;
        ba.key = a.key;
        ba.rng_shift = a.rng_shift;
        ba.n_rep = a.b.n_rep;
        ba.L = a.b.L;
    }
    int sweeps(hipStream_t s, uint64_t sweep0, int32_t n_sweeps, int launches, CallTally &tally) {
        int32_t done = 0;
        for (int k = 0; k < launches; ++k) {
            const int32_t n = (n_sweeps - done + launches - k - 1) / (launches - k);
            ba.src = lattice[at];
            ba.dst = lattice[1 - at];
            ba.t = (uint32_t)(sweep0 + (uint64_t)done);
            SMC_HIP(launch_bands2d(ba, sh, n, tally.next(), s));
            done += n;
            at = 1 - at;
        }
        return SMC_OK;
    }
};

int run_bands2d(StreamCtx &c, hipStream_t s, const SweepArgs &a, const BandShape &sh, void *other, uint64_t sweep0,
                int32_t n_sweeps, int64_t *dE) {
    CallTally tally;
    const int launches = bands2d_launches(sh, n_sweeps, true);
    int rc = tally.begin(c, a.b.n_rep, bands2d_groups(a.b.L, sh), launches, dE);
    if (rc) return rc;
    BandRun run(a, sh, other);
    SweepTimer timer(s, launches);
    if ((rc = run.sweeps(s, sweep0, n_sweeps, launches, tally))) return rc;
    timer.finish();
    return tally.finish(s);
}

// Tempering on the bands: m sweeps, then the exchange round, per step.
int run_pt_bands2d(StreamCtx &c, hipStream_t s, const SweepArgs &a, const BandShape &sh, void *other, SwapArgs &sw,
                   double *energy, uint64_t step0, int32_t n_steps, int m) {
    int rc;
    SMC_HIP(launch_pt_prepare(sw, energy, s));
    BandRun run(a, sh, other);
    const int launches = bands2d_launches(sh, m, false);
    for (int32_t k = 0; k < n_steps; ++k) {
        sw.t = (uint32_t)(step0 + (uint64_t)k);
        CallTally tally;
        if ((rc = tally.begin(c, a.b.n_rep, bands2d_groups(a.b.L, sh), launches, sw.E))) return rc;
        if ((rc = run.sweeps(s, (uint64_t)sw.t * (uint64_t)m, m, launches, tally))) return rc;
        if ((rc = tally.finish(s))) return rc;
        SMC_HIP(launch_pt_swap(sw, s));
    }
    if (!sh.whole && run.at)
        SMC_HIP(hipMemcpyAsync(a.spins, other, (size_t)a.b.n_rep * (size_t)a.b.N, hipMemcpyDeviceToDevice, s));
    SMC_HIP(launch_pt_finish(sw, energy, s));
    return SMC_OK;
}

// Sweeps of small 3D replicas in LDS, up to kSmall3dSweeps per launch (so
// that one launch stays short).  A workgroup takes enough replicas to fill a
// wavefront, and more only once there are four workgroups per compute unit.
constexpr int kSmall3dSweeps = 4096;

int run_small3d(hipStream_t s, const SweepArgs &a, uint64_t sweep0, int32_t n_sweeps, int64_t *dE) {
    Small3dArgs sa;
    memset(&sa, 0, sizeof sa);
    sa.spins = (int8_t *)a.spins;
    sa.coup = a.coup;
    sa.rep_per_sample = a.b.rep_per_sample;
    sa.L = a.b.L;
    sa.n_rep = a.b.n_rep;
    const int blocks = (int)((a.b.N / 2 + 7) / 8);  // Philox blocks, one lane each
    const int fill = (63 + blocks) / blocks, spread = (a.b.n_rep + 1023) / 1024;
    sa.n = fill > spread ? fill : spread;
    const int most = small3d_max_reps(a.b.L);
    if (sa.n > most) sa.n = most;
    sa.thr = a.thr;
    sa.key = a.key;
    sa.n_steps = 1;
    sa.rng_shift = a.rng_shift;
    sa.dE = dE;
    SweepTimer timer(s, (n_sweeps + kSmall3dSweeps - 1) / kSmall3dSweeps);
    for (int32_t done = 0; done < n_sweeps; done += sa.m) {
        sa.m = n_sweeps - done < kSmall3dSweeps ? n_sweeps - done : kSmall3dSweeps;
        sa.t0 = (uint32_t)(sweep0 + (uint64_t)done);
        SMC_HIP(launch_small3d(sa, s));
    }
    timer.finish();
    return SMC_OK;
}

// The packed copy of a call; SMC_ENOMEM (the caller's bytes serve then) if
// there is no room for it.
int pairs3d_args(StreamCtx &c, const SweepArgs &a, Pairs3dArgs *p) {
    void *q = nullptr;
    const size_t bytes = pairs3d_bytes(a.b.L, a.b.n_rep);
    if (int rc = ensure_spare(c, bytes, &q)) return rc;
    p->packed = (uint32_t *)q;
    p->rep_per_sample = a.b.rep_per_sample;
    p->thr = a.thr;
    p->row_of_rep = a.row_of_rep;
    p->key = a.key;
    p->t = 0;
    p->rng_shift = a.rng_shift;
    p->n_rep = a.b.n_rep;
    p->L = a.b.L;
    return SMC_OK;
}

int run_pairs3d(StreamCtx &c, hipStream_t s, const SweepArgs &a, Pairs3dArgs &p, uint64_t sweep0, int32_t n_sweeps,
                int64_t *dE) {
    const int planes = pairs3d_planes(p.L, p.n_rep);
    CallTally tally;
    int rc = tally.begin(c, p.n_rep, pairs3d_groups(p.L, planes), 2 * (int64_t)n_sweeps, dE);
    if (rc) return rc;
    SMC_HIP(launch_pairs3d_pack((const int8_t *)a.spins, a.coup, p, s));
    SweepTimer timer(s, 2 * (int64_t)n_sweeps);
    for (int32_t k = 0; k < n_sweeps; ++k) {
        p.t = (uint32_t)(sweep0 + (uint64_t)k);
        for (int col = 0; col < 2; ++col)
            SMC_HIP(launch_pairs3d_half(p, a.coup != nullptr, col, planes, tally.next(), s));
    }
    timer.finish();
    SMC_HIP(launch_pairs3d_unpack((int8_t *)a.spins, p, s));
    return tally.finish(s);
}

int run_pt_pairs3d(StreamCtx &c, hipStream_t s, const SweepArgs &a, Pairs3dArgs &p, SwapArgs &sw, double *energy,
                   uint64_t step0, int32_t n_steps, int m) {
    int rc;
    const int planes = pairs3d_planes(p.L, p.n_rep);
    SMC_HIP(launch_pt_prepare(sw, energy, s));
    SMC_HIP(launch_pairs3d_pack((const int8_t *)a.spins, a.coup, p, s));
    for (int32_t k = 0; k < n_steps; ++k) {
        sw.t = (uint32_t)(step0 + (uint64_t)k);
        CallTally tally;
        if ((rc = tally.begin(c, p.n_rep, pairs3d_groups(p.L, planes), 2 * (int64_t)m, sw.E))) return rc;
        for (int j = 0; j < m; ++j) {
            p.t = sw.t * (uint32_t)m + (uint32_t)j;
            for (int col = 0; col < 2; ++col)
                SMC_HIP(launch_pairs3d_half(p, a.coup != nullptr, col, planes, tally.next(), s));
        }
        if ((rc = tally.finish(s))) return rc;
        SMC_HIP(launch_pt_swap(sw, s));
    }
    SMC_HIP(launch_pairs3d_unpack((int8_t *)a.spins, p, s));
    SMC_HIP(launch_pt_finish(sw, energy, s));
    return SMC_OK;
}

// Where the steps of a tempering call run.  The packed copy and the bands give way to the
// half-sweeps where there is no room for their scratch.
enum PtRoute { kPtSmall3d, kPtSplit2d, kPtBins2d, kPtPairs3d, kPtBands2d, kPtHalves };

PtRoute pt_route(const smc_desc *d, const void *spins, const int8_t *coup, const std::vector<ThrRow> &rows, int n_temps,
                 int n_chains, int32_t n_steps, int m, BandShape *sh) {
    if (use_small3d_pt(d, n_temps, n_chains)) return kPtSmall3d;
    const bool bands = use_bands2d(d, m, false, sh);
    if (use_pt_split2d(d, spins, rows) && !(bands && bands_before_lattice2d(d, m, true))) return kPtSplit2d;
    // (few replicas: bands of their rows give more workgroups than a bin each)
    if (use_uneven2d(d, spins, coup, rows) &&
        !(bands && sh->ns_per_sweep * m < bins2d_ns(d->L, d->n_rep) * m + 3500.0))
        return kPtBins2d;
    if (use_pairs3d(d, (int64_t)n_steps * m)) return kPtPairs3d;
    return bands ? kPtBands2d : kPtHalves;
}

// The most launches of a tempering call of n_steps steps of m sweeps on a route.
int64_t pt_launches(PtRoute route, const Batch &b, const SweepArgs &a, const BandShape &sh, int64_t n_steps, int64_t m) {
    // per step: the sweeps, the sums of 16 and more workgroups collected, the exchange round
    auto steps = [&](int64_t sweeps, int groups) {
        return n_steps * (sweeps + (few_groups(groups, b.n_rep, sweeps) ? 0 : 1) + 1);
    };
    const int64_t halves = 2 + steps(2 * m, half_sweep_groups(a));  // prepare, finish
    switch (route) {
        case kPtSmall3d: return 1;
        // prepare, zero, to split; per step: thresholds, m sweeps, collect, add, exchange; from split, copy, finish
        case kPtSplit2d: return 6 + n_steps * (m + 4);
        // prepare, finish; per step the launches of every edge's bins and, of many bins, the exchange round
        case kPtBins2d: return 2 + n_steps * (bins2d_launches(b.n_rep) + 1);
        // prepare, pack, unpack, finish
        case kPtPairs3d:
            return std::max(halves, 4 + steps(2 * m, pairs3d_groups(b.L, pairs3d_planes(b.L, b.n_rep))));
        // prepare, a copy back, finish
        case kPtBands2d:
            return std::max(halves, 3 + steps(bands2d_launches(sh, (int)m, false), bands2d_groups(b.L, sh)));
        default: return halves;
    }
}

// The sweeps of a call on the general path.
// bands: the shape of the bands, where the caller has asked for it.
int run_generic(StreamCtx &c, hipStream_t s, const smc_desc *desc, SweepArgs &a, uint64_t sweep0, int32_t n_sweeps,
                int64_t *dE, const BandShape *bands = nullptr) {
    if (use_small3d(desc) && !(desc->L % 16 == 0 && sweep3d_asked_for()))
        return run_small3d(s, a, sweep0, n_sweeps, dE);
    if (use_pairs3d(desc, n_sweeps)) {
        Pairs3dArgs p;
        if (pairs3d_args(c, a, &p) == SMC_OK) return run_pairs3d(c, s, a, p, sweep0, n_sweeps, dE);
        last_error().clear();
    }
    BandShape sh;
    if (bands) sh = *bands;
    if (bands || use_bands2d(desc, n_sweeps, true, &sh)) {
        void *other = nullptr;
        if (sh.whole || ensure_spare(c, (size_t)a.b.n_rep * (size_t)a.b.N, &other) == SMC_OK)
            return run_bands2d(c, s, a, sh, other, sweep0, n_sweeps, dE);
        last_error().clear();  // no room for a second lattice: the half-sweeps need none
    }
    CallTally tally;
    int rc = tally.begin(c, a.b.n_rep, half_sweep_groups(a), 2 * (int64_t)n_sweeps, dE);
    if (rc) return rc;
    SweepTimer timer(s, 2 * (int64_t)n_sweeps);
    for (int32_t k = 0; k < n_sweeps; ++k) {
        a.t = (uint32_t)(sweep0 + (uint64_t)k);
        for (int col = 0; col < 2; ++col) {
            a.tally = tally.next();
            SMC_HIP(launch_half_sweep_generic(a, col, s));
        }
    }
    timer.finish();
    return tally.finish(s);
}

}  // namespace
}  // namespace smc

using namespace smc;

extern "C" {

const char *smc_strerror(int status) {
    switch (status) {
        case SMC_OK: return "success";
        case SMC_EINVAL: return "invalid argument";
        case SMC_EUNSUPPORTED: return "unsupported combination of arguments";
        case SMC_EHIP: return "HIP runtime error";
        case SMC_ENOMEM: return "out of device memory for scratch";
        default: return "unknown status";
    }
}

const char *smc_last_error(void) { return last_error().c_str(); }

int smc_kernel_timing_enable(int enable) {
    std::lock_guard<std::mutex> lk(g_timing_mutex);
    g_timing_on = enable != 0;
    if (!g_timing_on) forget_timed();
    return SMC_OK;
}

int smc_philox_bench(uint64_t seed, uint32_t t, uint32_t r, uint32_t tag, int32_t n_threads, int32_t per_thread,
                     uint32_t *out, void *stream) {
    last_error().clear();
    if (!out) return fail(SMC_EINVAL, "out is NULL");
    if (n_threads <= 0 || per_thread <= 0) return fail(SMC_EINVAL, "n_threads and per_thread must be positive");
    if ((int64_t)n_threads * per_thread > (int64_t)1 << 32)
        return fail(SMC_EINVAL, "n_threads * per_thread exceeds 2^32");
    SMC_HIP(launch_philox_bench(make_key(seed), t, r, tag, (uint32_t)n_threads, per_thread, out,
                                (hipStream_t)stream));
    return SMC_OK;
}

int smc_kernel_timing_read(double *elapsed_ms, int64_t *launches) {
    last_error().clear();
    if (!elapsed_ms || !launches) return fail(SMC_EINVAL, "output pointers are required");
    std::lock_guard<std::mutex> lk(g_timing_mutex);
    double ms = 0.0;
    int64_t n = 0;
    int rc = SMC_OK;
    for (TimedCall &c : g_timed) {
        float part = 0.0f;
        hipError_t e = hipEventSynchronize(c.stop);
        if (e == hipSuccess) e = hipEventElapsedTime(&part, c.start, c.stop);
        if (e != hipSuccess) {
            rc = fail(SMC_EHIP, "%s", hipGetErrorString(e));
            break;
        }
        ms += part;
        n += c.launches;
    }
    forget_timed();
    *elapsed_ms = ms;
    *launches = n;
    return rc;
}

int smc_sweep_plan(const smc_desc *desc, int32_t *launches_per_sweep, const char **kernel_name) {
    last_error().clear();
    Plan plan;
    int rc = validate(desc, false, plan);
    if (rc) return rc;
    if (!launches_per_sweep || !kernel_name) return fail(SMC_EINVAL, "output pointers are required");
    if (desc->model == SMC_HEISENBERG) {
        *launches_per_sweep = 2;
        if (use_heis3d_tiled(desc, 2)) {
            *launches_per_sweep = 1;
            *kernel_name = "k_heis3d_tiled";
        } else {
            *kernel_name = use_heis3d(desc) ? "k_heis3d_half" : "k_heis_half_sweep_generic";
        }
    } else if (desc->model == SMC_ISING && desc->dim == 2 && desc->L > 0 && lattice2d_supported(desc->L)) {
        *launches_per_sweep = 1;
        *kernel_name = "k_ising2d_split";
    } else if (sweep3d_shape(desc)) {
        const bool pass = pass3d_enabled(desc);
        *launches_per_sweep = pass ? 1 : 2;
        *kernel_name = pass ? "k_ising3d_pass" : "k_ising3d_half";
    } else if (small2d_shape(desc) && small2d_enabled() &&
               !(getenv("SPINMC_UNEVEN2D") && getenv("SPINMC_UNEVEN2D")[0] == '0')) {
        *launches_per_sweep = 1;  // at most: up to 256 sweeps per launch
        *kernel_name = "k_uneven2d_sweep";
    } else {
        *launches_per_sweep = 2;
        *kernel_name = "k_half_sweep_generic";
    }
    return SMC_OK;
}

int smc_pt_plan(const smc_desc *desc, const smc_pt_desc *pt, int32_t n_steps, int32_t *launches,
                const char **kernel_name) {
    last_error().clear();
    Plan plan;
    int rc = validate(desc, false, plan);
    if (rc) return rc;
    if (!pt || !launches || !kernel_name) return fail(SMC_EINVAL, "pt desc and output pointers are required");
    if (n_steps < 0) return fail(SMC_EINVAL, "n_steps must be >= 0");
    if (pt->n_temps < 2 || !pt->beta) return fail(SMC_EINVAL, "need n_temps >= 2 and beta");
    if (pt->sweeps_per_step < 0) return fail(SMC_EINVAL, "sweeps_per_step must be >= 0");
    const int m = pt->sweeps_per_step > 0 ? pt->sweeps_per_step : 1;
    const int rows_n = pt->beta_per_chain ? pt->n_chains : 1;
    std::vector<ThrRow> all_rows((size_t)rows_n * pt->n_temps);
    for (size_t k = 0; k < all_rows.size(); ++k) all_rows[k] = threshold_row(pt->beta[k], desc->dim);
    SweepArgs a;
    memset(&a, 0, sizeof a);
    a.b = plan.b;
    a.pieces = plan.pieces;
    a.max_L = plan.max_L;
    BandShape sh;
    const PtRoute route = pt_route(desc, nullptr, nullptr, all_rows, pt->n_temps,
                                   std::max(1, desc->n_rep / pt->n_temps), n_steps, m, &sh);
    const int64_t most = n_steps > 0 ? pt_launches(route, plan.b, a, sh, n_steps, m) : 0;
    *launches = (int32_t)std::min<int64_t>(most, INT32_MAX);
    const bool fits = use_pt3d(desc, pt->n_temps);
    bool fits2d = !fits && desc->dim == 2 && (desc->model == SMC_ISING || desc->model == SMC_EA);
    if (fits2d) {
        const char *env = getenv("SPINMC_UNEVEN2D");
        if (env && env[0] == '0') fits2d = false;
        for (int r = 0; fits2d && desc->L == 0 && r < desc->n_rep; ++r)
            fits2d = uneven2d_edge_supported(desc->inst[r].L) && desc->inst[r].spin_off % 16 == 0 &&
                     (desc->model != SMC_EA || desc->inst[r].coup_off % 16 == 0);
        if (desc->L > 0) fits2d = uneven2d_edge_supported(desc->L);
        for (int64_t k = 0; fits2d && k < (int64_t)rows_n * pt->n_temps; ++k) {
            const ThrRow r = threshold_row(pt->beta[k], desc->dim);
            fits2d = r.m[1].x <= 0xFFFFu && r.m[2].x <= 0xFFFFu;
        }
    }
    *kernel_name = fits ? "k_pt3d_chain"
                   : use_pt_split2d(desc, (const void *)nullptr, all_rows) ? "k_ising2d_split"
                   : fits2d ? "k_uneven2d_sweep"
                            : "k_half_sweep_generic";
    return SMC_OK;
}

int smc_spin_init(const smc_desc *desc, void *spins, int8_t *couplings, void *stream) {
    last_error().clear();
    Plan plan;
    const bool want_coup = desc && desc->model == SMC_EA && couplings;
    int rc = validate(desc, want_coup, plan);
    if (rc) return rc;
    if (!spins) return fail(SMC_EINVAL, "spins is NULL");
    hipStream_t s = (hipStream_t)stream;
    if (int rc_cap = refuse_capture(s)) return rc_cap;
    StreamCtx &c = ctx_for(s);
    if ((rc = upload_inst(c, s, desc, plan))) return rc;
    const Key key = make_key(desc->seed);
    if (desc->model == SMC_HEISENBERG) {
        SMC_HIP(launch_init_heis(plan.b, plan.max_L, (float *)spins, key, s));
    } else {
        SMC_HIP(launch_init_spins(plan.b, plan.max_L, (int8_t *)spins, key, s));
    }
    if (want_coup && plan.n_samples > 0) {
        fill_uniform_samples(desc, plan);
        void *p = nullptr;
        if ((rc = upload(c, s, kSamples, plan.samples.data(), sizeof(smc_inst) * plan.samples.size(), &p))) return rc;
        int maxL = 0;
        for (auto &g : plan.samples) maxL = g.L > maxL ? g.L : maxL;
        SMC_HIP(launch_init_couplings(desc->dim, (int)plan.n_samples, (const smc_inst *)p, maxL, couplings, key, s));
    }
    return SMC_OK;
}

// ------------------------------------- asynchronous multi-spin coding ----
// Replicas 32g .. 32g+31 form group g and share its Metropolis draws.
int msc_check(const smc_desc *d, int word_bits) {
    if (d->model != SMC_ISING && d->model != SMC_EA)
        return fail(SMC_EUNSUPPORTED, "multi-spin coding is provided for the Ising and EA models");
    if (word_bits != 32 && word_bits != 64) return fail(SMC_EINVAL, "word_bits must be 32 or 64 (got %d)", word_bits);
    if (d->L <= 0) return fail(SMC_EINVAL, "multi-spin coding needs a uniform batch (L > 0)");
    if (d->n_rep % word_bits != 0)
        return fail(SMC_EINVAL, "n_rep (%d) must be a multiple of %d", d->n_rep, word_bits);
    if (d->model == SMC_EA && d->rep_per_sample != 1)
        return fail(SMC_EINVAL, "multi-spin coding needs one coupling sample per replica (rep_per_sample = 1)");
    return SMC_OK;
}

// The packed kernel serves 2D batches of edge 16, 32 or 64 with 4-byte
// aligned spins and couplings (SPINMC_MSC2D=0 sends them to the generic
// kernels, which give the same results).
bool use_msc2d(const smc_desc *d, const void *spins, const void *coup) {
    const char *env = getenv("SPINMC_MSC2D");
    if (env && env[0] == '0') return false;
    if (((uintptr_t)spins & 3u) || ((uintptr_t)coup & 3u)) return false;
    return msc2d_supported(d->dim, d->L);
}

int smc_metropolis_sweep(const smc_desc *desc, void *spins, const int8_t *couplings, const double *beta,
                         uint64_t sweep0, int32_t n_sweeps, int64_t *dE_accum, void *stream) {
    last_error().clear();
    Plan plan;
    int rc = validate(desc, true, plan);
    if (rc) return rc;
    if (!spins) return fail(SMC_EINVAL, "spins is NULL");
    if (!beta) return fail(SMC_EINVAL, "beta is NULL");
    if (desc->model == SMC_EA && !couplings) return fail(SMC_EINVAL, "couplings are required for EA");
    if (n_sweeps < 0) return fail(SMC_EINVAL, "n_sweeps must be >= 0");
    if (sweep0 + (uint64_t)n_sweeps > (1ull << 32)) return fail(SMC_EINVAL, "sweep index exceeds 32 bits");
    for (int r = 0; r < desc->n_rep; ++r)
        if (!(beta[r] >= 0.0) || !isfinite(beta[r])) return fail(SMC_EINVAL, "beta[%d] must be finite and >= 0", r);
    if (n_sweeps == 0) return SMC_OK;
    hipStream_t s = (hipStream_t)stream;
    if (int rc_cap = refuse_capture(s)) return rc_cap;
    StreamCtx &c = ctx_for(s);
    if ((rc = upload_inst(c, s, desc, plan))) return rc;

    SweepArgs a;
    memset(&a, 0, sizeof a);
    a.b = plan.b;
    a.spins = spins;
    a.coup = desc->model == SMC_EA ? couplings : nullptr;
    a.key = make_key(desc->seed);
    a.pieces = plan.pieces;
    a.max_L = plan.max_L;
    a.row_of_rep = nullptr;
    void *p = nullptr;
    if (desc->model == SMC_HEISENBERG) {
        std::vector<float> bf(desc->n_rep);
        for (int r = 0; r < desc->n_rep; ++r) bf[r] = (float)beta[r];
        if ((rc = upload(c, s, kTables, bf.data(), sizeof(float) * bf.size(), &p))) return rc;
        a.beta_f = (const float *)p;
        if (use_heis_small(desc, n_sweeps)) {
            constexpr int32_t kPerLaunch = 1024;  // sweeps, so that one launch stays short
            SweepTimer timer(s, (n_sweeps + kPerLaunch - 1) / kPerLaunch);
            for (int32_t done = 0; done < n_sweeps; done += kPerLaunch)
                SMC_HIP(launch_heis_small((float *)spins, a.beta_f, dE_accum, desc->n_rep, desc->dim, desc->L, a.key,
                                          (uint32_t)(sweep0 + (uint64_t)done),
                                          n_sweeps - done < kPerLaunch ? n_sweeps - done : kPerLaunch,
                                          desc->renorm_every, s));
            timer.finish();
            return SMC_OK;
        }
        void *pp = nullptr;
        const size_t bytes = (size_t)desc->n_rep * 3 * sizeof(float) * (size_t)plan.b.N;
        bool tiled = use_heis3d_tiled(desc, n_sweeps);
        if (tiled && ensure_spare(c, bytes, &pp)) {
            last_error().clear();  // no room for a second lattice: the half-sweeps need none
            tiled = false;
        }
        if (tiled) {
            // one-pass sweeps, ping-pong between the caller's buffer and a scratch copy
            float *A = (float *)spins, *B = (float *)pp;
            const int planes = heis3d_tiled_planes(desc->L, desc->n_rep);
            CallTally tally;
            if ((rc = tally.begin(c, desc->n_rep, heis3d_tiled_groups(desc->L, planes), n_sweeps, dE_accum))) return rc;
            SweepTimer timer(s, n_sweeps);
            for (int32_t k = 0; k < n_sweeps; ++k) {
                a.t = (uint32_t)(sweep0 + (uint64_t)k);
                float *src = k & 1 ? B : A, *dst = k & 1 ? A : B;
                // the renormalisation is applied as the sweep stores its spins
                const bool renorm =
                    desc->renorm_every > 0 && ((uint64_t)a.t + 1) % (uint64_t)desc->renorm_every == 0;
                SMC_HIP(launch_heis3d_tiled(src, dst, a.beta_f, tally.next(), desc->n_rep, desc->L, a.key, a.t,
                                            renorm, planes, s));
            }
            timer.finish();
            if ((rc = tally.finish(s))) return rc;
            if (n_sweeps & 1) SMC_HIP(hipMemcpyAsync(A, B, bytes, hipMemcpyDeviceToDevice, s));
            return SMC_OK;
        }
        const bool fast = use_heis3d(desc);
        CallTally tally;
        if ((rc = tally.begin(c, desc->n_rep, fast ? heis3d_half_groups(desc->L) : heis_half_sweep_groups(a),
                              2 * (int64_t)n_sweeps, dE_accum)))
            return rc;
        SweepTimer timer(s, 2 * (int64_t)n_sweeps);  // the renormalisations run inside the same pair
        for (int32_t k = 0; k < n_sweeps; ++k) {
            a.t = (uint32_t)(sweep0 + (uint64_t)k);
            for (int col = 0; col < 2; ++col) {
                a.tally = tally.next();
                if (fast)
                    SMC_HIP(launch_heis3d_half((float *)spins, a.beta_f, a.tally, desc->n_rep, desc->L, a.key, a.t,
                                               col, s));
                else
                    SMC_HIP(launch_heis_half_sweep_generic(a, col, s));
            }
            if (desc->renorm_every > 0 && ((uint64_t)a.t + 1) % (uint64_t)desc->renorm_every == 0)
                SMC_HIP(launch_heis_renorm(plan.b, (float *)spins, plan.max_L, s));
        }
        timer.finish();
        return tally.finish(s);
    }
    std::vector<ThrRow> rows(desc->n_rep);
    for (int r = 0; r < desc->n_rep; ++r) rows[r] = threshold_row(beta[r], desc->dim);
    if ((rc = upload(c, s, kTables, rows.data(), sizeof(ThrRow) * rows.size(), &p))) return rc;
    a.thr = (const ThrRow *)p;
    BandShape sh;
    const bool lattice2d = use_lattice2d(desc, spins, rows);
    const bool bands = lattice2d && bands_before_lattice2d(desc, n_sweeps, false) && use_bands2d(desc, n_sweeps, true, &sh);
    if (lattice2d && !bands) {
        // one-pass sweeps on the colour-split layout, ping-pong between two buffers
        const size_t bytes = (size_t)desc->n_rep * lattice2d_split_bytes(desc->L);
        void *pp = nullptr;
        if ((rc = ensure(c, kLattices, 2 * bytes, &pp))) return rc;
        uint8_t *A = (uint8_t *)pp, *B = A + bytes;
        // energy changes: per-wave partial sums over the call, collected once at the end
        int64_t *part = nullptr;
        if (dE_accum) {
            void *q = nullptr;
            const size_t slots = lattice2d_de_slots(desc->L, desc->n_rep);
            if (slots == 0) return fail(SMC_EINVAL, "no band shape for L=%d", desc->L);
            if ((rc = ensure(c, kL2dPart, slots * sizeof(int64_t), &q))) return rc;
            part = (int64_t *)q;
        }
        const char *fuse_env = getenv("SPINMC_L2D_FUSE");
        if (fuse_env && fuse_env[0] == '0') {
            // separate layout conversions around the sweeps (for comparison)
            SMC_HIP(launch_to_split((const int8_t *)spins, A, desc->L, desc->n_rep, s));
            SweepTimer timer(s, n_sweeps);
            for (int32_t k = 0; k < n_sweeps; ++k) {
                const uint32_t t = (uint32_t)(sweep0 + (uint64_t)k);
                SMC_HIP(launch_ising2d_split(k & 1 ? B : A, false, k & 1 ? A : B, false, desc->L, desc->n_rep,
                                             a.thr, part, k == 0, a.key, t, s));
            }
            timer.finish();
            if (part) SMC_HIP(launch_lattice2d_de_collect(part, dE_accum, desc->L, desc->n_rep, s));
            SMC_HIP(launch_from_split(n_sweeps & 1 ? B : A, (int8_t *)spins, desc->L, desc->n_rep, s));
            return SMC_OK;
        }
        // The first sweep reads the caller's lattice, the last one writes it
        // back; the sweeps between ping-pong on the split layout (sweep k
        // leaves its result in A for even k, in B for odd k).  A single sweep
        // ends in A and is converted back.
        SweepTimer timer(s, n_sweeps);
        for (int32_t k = 0; k < n_sweeps; ++k) {
            const uint32_t t = (uint32_t)(sweep0 + (uint64_t)k);
            const bool first = k == 0, last = k == n_sweeps - 1 && n_sweeps > 1;
            const void *src = first ? spins : (k & 1 ? (const void *)A : (const void *)B);
            void *dst = last ? spins : (k & 1 ? (void *)B : (void *)A);
            SMC_HIP(launch_ising2d_split(src, first, dst, last, desc->L, desc->n_rep, a.thr, part, first, a.key, t,
                                         s));
        }
        timer.finish();
        if (part) SMC_HIP(launch_lattice2d_de_collect(part, dE_accum, desc->L, desc->n_rep, s));
        if (n_sweeps == 1) SMC_HIP(launch_from_split(A, (int8_t *)spins, desc->L, desc->n_rep, s));
        return SMC_OK;
    }
    if (desc->dim == 3 && desc->L % 16 == 0 && use_small3d(desc) && !sweep3d_asked_for())
        return run_small3d(s, a, sweep0, n_sweeps, dE_accum);
    if (desc->L % 16 == 0 && use_pairs3d(desc, n_sweeps)) {
        Pairs3dArgs pa;
        if (pairs3d_args(c, a, &pa) == SMC_OK) return run_pairs3d(c, s, a, pa, sweep0, n_sweeps, dE_accum);
        last_error().clear();
    }
    if (use_sweep3d(desc, spins, a.coup, rows)) {
        // EA calls of several sweeps read the bonds bit-packed (one pass to
        // pack them: 3 B per site per sample in, 0.5 B out; the int8 bonds
        // cost 3 B per site and launch); SPINMC_SWEEP3D_PACK=0 keeps the int8 bonds
        const int8_t *coup8 = a.coup;
        const uint2 *packed = nullptr;
        const char *env = getenv("SPINMC_SWEEP3D_PACK");
        const bool pass = pass3d_enabled(desc);
        if (a.coup && (pass || (n_sweeps >= 4 && !(env && env[0] == '0')))) {
            void *q = nullptr;
            if ((rc = ensure(c, kBonds3d, (size_t)plan.n_samples * (size_t)(plan.b.N / 16) * sizeof(uint2), &q)))
                return rc;
            packed = (const uint2 *)q;
            coup8 = nullptr;
            SMC_HIP(launch_pack_bonds3d(a.coup, (uint2 *)q, desc->L, (int)plan.n_samples, s));
        }
        if (pass) {
            // one launch per sweep, ping-pong between the caller's lattice and
            // a second buffer; an odd count ends with one copy back
            const size_t bytes = (size_t)desc->n_rep * (size_t)plan.b.N;
            void *q = nullptr;
            if ((rc = ensure(c, kLattices, bytes, &q))) return rc;
            int8_t *A = (int8_t *)spins, *B = (int8_t *)q;
            Shape shape{{0, 0, 0}};
            if (!pass3d_launch_shape(desc->L, packed != nullptr, desc->n_rep, &shape))
                return fail(SMC_EINVAL, "no strip shape for L=%d", desc->L);
            CallTally tally;
            if ((rc = tally.begin(c, desc->n_rep, pass3d_groups(desc->L, shape), n_sweeps, dE_accum))) return rc;
            SweepTimer timer(s, n_sweeps);
            for (int32_t k = 0; k < n_sweeps; ++k) {
                const uint32_t t = (uint32_t)(sweep0 + (uint64_t)k);
                SMC_HIP(launch_ising3d_pass(k & 1 ? B : A, k & 1 ? A : B, packed, plan.b.rep_per_sample, a.thr,
                                            tally.next(), desc->n_rep, desc->L, a.key, t, shape, s));
            }
            timer.finish();
            if ((rc = tally.finish(s))) return rc;
            if (n_sweeps & 1) SMC_HIP(hipMemcpyAsync(A, B, bytes, hipMemcpyDeviceToDevice, s));
            return SMC_OK;
        }
        const int Z = sweep3d_rows(desc->L, desc->model == SMC_EA, desc->n_rep);
        CallTally tally;
        if ((rc = tally.begin(c, desc->n_rep, sweep3d_groups(desc->L, Z), 2 * (int64_t)n_sweeps, dE_accum))) return rc;
        SweepTimer timer(s, 2 * (int64_t)n_sweeps);
        for (int32_t k = 0; k < n_sweeps; ++k) {
            const uint32_t t = (uint32_t)(sweep0 + (uint64_t)k);
            for (int col = 0; col < 2; ++col)
                SMC_HIP(launch_ising3d_half((int8_t *)spins, coup8, packed, plan.b.rep_per_sample, a.thr,
                                            tally.next(), desc->n_rep, desc->L, a.key, t, col, Z, s));
        }
        timer.finish();
        return tally.finish(s);
    }
    return run_generic(c, s, desc, a, sweep0, n_sweeps, dE_accum, bands ? &sh : nullptr);
}

int smc_msc_sweep(const smc_desc *desc, void *spins, const int8_t *couplings, const double *beta, uint64_t sweep0,
                  int32_t n_sweeps, int32_t word_bits, int64_t *dE_accum, void *stream) {
    last_error().clear();
    Plan plan;
    int rc = validate(desc, true, plan);
    if (rc) return rc;
    if ((rc = msc_check(desc, word_bits))) return rc;
    if (!spins) return fail(SMC_EINVAL, "spins is NULL");
    if (!beta) return fail(SMC_EINVAL, "beta is NULL");
    if (desc->model == SMC_EA && !couplings) return fail(SMC_EINVAL, "couplings are required for EA");
    if (n_sweeps < 0) return fail(SMC_EINVAL, "n_sweeps must be >= 0");
    if (sweep0 + (uint64_t)n_sweeps > (1ull << 32)) return fail(SMC_EINVAL, "sweep index exceeds 32 bits");
    for (int r = 0; r < desc->n_rep; ++r) {
        if (!(beta[r] >= 0.0) || !isfinite(beta[r])) return fail(SMC_EINVAL, "beta[%d] must be finite and >= 0", r);
        if (beta[r] != beta[r - r % word_bits])
            return fail(SMC_EINVAL, "beta[%d] differs from the rest of its group of %d", r, word_bits);
    }
    if (n_sweeps == 0) return SMC_OK;
    hipStream_t s = (hipStream_t)stream;
    if (int rc_cap = refuse_capture(s)) return rc_cap;
    StreamCtx &c = ctx_for(s);
    if ((rc = upload_inst(c, s, desc, plan))) return rc;
    const int G = desc->n_rep / 32;
    const bool ea = desc->model == SMC_EA;
    if (use_msc2d(desc, spins, ea ? couplings : nullptr)) {
        const int64_t N = (int64_t)desc->L * desc->L;
        std::vector<ThrRow> rows(G);
        for (int g = 0; g < G; ++g)
            rows[g] = (g > 0 && beta[32 * g] == beta[32 * (g - 1)]) ? rows[g - 1] : threshold_row(beta[32 * g], desc->dim);
        void *tp = nullptr, *sp = nullptr, *cp = nullptr, *ep = nullptr, *mp = nullptr;
        if ((rc = upload(c, s, kTables, rows.data(), sizeof(ThrRow) * rows.size(), &tp))) return rc;
        if ((rc = ensure(c, kMscSpins, sizeof(uint32_t) * (size_t)(G * N), &sp))) return rc;
        if ((rc = ensure(c, kMscCoup, sizeof(uint32_t) * (size_t)(G * 2 * N), &cp))) return rc;
        void *gp = nullptr;
        if ((rc = ensure(c, kMscGauge, sizeof(uint32_t) * (size_t)(G * N), &gp))) return rc;
        const size_t mbytes = measure_scratch_bytes(plan.b, plan.max_L);
        if (dE_accum) {
            if ((rc = ensure(c, kMscEnergy, 2 * sizeof(double) * (size_t)desc->n_rep, &ep))) return rc;
            if ((rc = ensure(c, kMeasure, mbytes, &mp))) return rc;
            SMC_HIP(launch_measure(plan.b, spins, ea ? couplings : nullptr, plan.max_L, (double *)ep, nullptr, mp,
                                   mbytes, s));
        }
        SMC_HIP(launch_msc_pack((const int8_t *)spins, (uint32_t *)sp, N, G, s));
        SMC_HIP(launch_msc_pack_coup(ea ? couplings : nullptr, (uint32_t *)cp, 2 * N, G, s));
        SMC_HIP(launch_msc_gauge2d((uint32_t *)sp, (uint32_t *)cp, (uint32_t *)gp, desc->L, G, s));
        SweepTimer timer(s, 1);  // all sweeps in one launch
        SMC_HIP(launch_msc2d((uint32_t *)sp, (const uint32_t *)cp, (const ThrRow *)tp, G, desc->L,
                             make_key(desc->seed), (uint32_t)sweep0, n_sweeps, word_bits / 32, s));
        timer.finish();
        SMC_HIP(launch_msc_unpack((const uint32_t *)sp, (const uint32_t *)gp, (int8_t *)spins, N, G, s));
        if (dE_accum) {
            double *E0 = (double *)ep, *E1 = E0 + desc->n_rep;
            SMC_HIP(launch_measure(plan.b, spins, ea ? couplings : nullptr, plan.max_L, E1, nullptr, mp, mbytes, s));
            SMC_HIP(launch_msc_energy_diff(E0, E1, dE_accum, desc->n_rep, s));
        }
        return SMC_OK;
    }
    // generic per-site kernels with the group index in the draws' counters
    std::vector<ThrRow> rows(desc->n_rep);
    for (int r = 0; r < desc->n_rep; ++r) rows[r] = threshold_row(beta[r], desc->dim);
    void *p = nullptr;
    if ((rc = upload(c, s, kTables, rows.data(), sizeof(ThrRow) * rows.size(), &p))) return rc;
    SweepArgs a;
    memset(&a, 0, sizeof a);
    a.b = plan.b;
    a.spins = spins;
    a.coup = ea ? couplings : nullptr;
    a.thr = (const ThrRow *)p;
    a.key = make_key(desc->seed);
    a.pieces = plan.pieces;
    a.max_L = plan.max_L;
    a.row_of_rep = nullptr;
    a.rng_shift = word_bits == 64 ? 6 : 5;  // the draw group r / word_bits
    return run_generic(c, s, desc, a, sweep0, n_sweeps, dE_accum);
}

// The packed double-checkerboard kernel: thresholds with 16-bit high halves,
// 16-byte aligned buffers, a power-of-two tile; SPINMC_DCB_PACKED=0 forces
// the per-site kernel (same results).
static bool use_dcb_packed(const smc_desc *d, const std::vector<ThrRow> &rows, const void *spins,
                           const int8_t *coup, int tile) {
    const char *env = getenv("SPINMC_DCB_PACKED");
    if (env && env[0] == '0') return false;
    if (d->dim != 2 || !dcb2d_packed_supported(d->L, tile)) return false;
    if (((uintptr_t)spins & 15u) || (d->model == SMC_EA && ((uintptr_t)coup & 15u))) return false;
    for (const ThrRow &r : rows)
        if (r.m[1].x > 0xFFFFu || r.m[2].x > 0xFFFFu) return false;
    return true;
}

// Checks shared by smc_dcb_sweep and smc_dcb_plan.
static int dcb_check(const smc_desc *desc, const double *beta, int tile) {
    Plan plan;
    int rc = validate(desc, true, plan);
    if (rc) return rc;
    if (desc->model != SMC_ISING && desc->model != SMC_EA)
        return fail(SMC_EUNSUPPORTED, "the double checkerboard is provided for the Ising and EA models");
    if (desc->L <= 0) return fail(SMC_EINVAL, "the double checkerboard needs a uniform batch (L > 0)");
    if (desc->dim == 2 && !dcb2d_supported(desc->L, tile))
        return fail(SMC_EINVAL, "tile %d: need a multiple of 16 in [16, 128] dividing L = %d into an even number "
                                "of tiles per row (or one)", tile, desc->L);
    if (desc->dim == 3 && !dcb3d_supported(desc->L, tile))
        return fail(SMC_EINVAL, "tile %d: 3D tiles are 16 x 16 x 16, dividing L = %d into an even number of tiles "
                                "per direction (or one)", tile, desc->L);
    if (!beta) return fail(SMC_EINVAL, "beta is NULL");
    for (int r = 0; r < desc->n_rep; ++r)
        if (!(beta[r] >= 0.0) || !isfinite(beta[r])) return fail(SMC_EINVAL, "beta[%d] must be finite and >= 0", r);
    return SMC_OK;
}

static std::vector<ThrRow> dcb_rows(const smc_desc *desc, const double *beta) {
    std::vector<ThrRow> rows(desc->n_rep);
    for (int r = 0; r < desc->n_rep; ++r)
        rows[r] = (r > 0 && beta[r] == beta[r - 1]) ? rows[r - 1] : threshold_row(beta[r], desc->dim);
    return rows;
}

int smc_dcb_plan(const smc_desc *desc, const double *beta, int32_t tile, const char **kernel_name) {
    last_error().clear();
    if (!kernel_name) return fail(SMC_EINVAL, "kernel_name is NULL");
    int rc = dcb_check(desc, beta, tile);
    if (rc) return rc;
    *kernel_name = desc->dim == 3 ? "k_dcb3d"
                   : use_dcb_packed(desc, dcb_rows(desc, beta), nullptr, nullptr, tile) ? "k_dcb2d_packed"
                                                                                        : "k_dcb2d";
    return SMC_OK;
}

int smc_dcb_sweep(const smc_desc *desc, void *spins, const int8_t *couplings, const double *beta, uint64_t sweep0,
                  int32_t n_sweeps, int32_t tile, int32_t hits, int32_t palindromic, int64_t *dE_accum,
                  int64_t *dE_trace, void *stream) {
    last_error().clear();
    int rc = dcb_check(desc, beta, tile);
    if (rc) return rc;
    if (hits < 1) return fail(SMC_EINVAL, "hits must be >= 1");
    if (!spins) return fail(SMC_EINVAL, "spins is NULL");
    if (desc->model == SMC_EA && !couplings) return fail(SMC_EINVAL, "couplings are required for EA");
    if (desc->dim == 3 && (((uintptr_t)spins & 15u) || (desc->model == SMC_EA && ((uintptr_t)couplings & 15u))))
        return fail(SMC_EINVAL, "3D double checkerboard: spins (and EA couplings) must be 16-byte aligned");
    if (n_sweeps < 0) return fail(SMC_EINVAL, "n_sweeps must be >= 0");
    if ((sweep0 + (uint64_t)n_sweeps) * (uint64_t)hits > (1ull << 32))
        return fail(SMC_EINVAL, "(sweep0 + n_sweeps) * hits exceeds 2^32 (the hit index is one 32-bit word)");
    if (n_sweeps == 0) return SMC_OK;
    hipStream_t s = (hipStream_t)stream;
    if (int rc_cap = refuse_capture(s)) return rc_cap;
    StreamCtx &c = ctx_for(s);
    const std::vector<ThrRow> rows = dcb_rows(desc, beta);
    void *tp = nullptr, *sp = nullptr;
    if ((rc = upload(c, s, kTables, rows.data(), sizeof(ThrRow) * rows.size(), &tp))) return rc;
    const int per_rep =
        2 * (desc->dim == 3 ? dcb3d_tiles_per_colour(desc->L, tile) : dcb2d_tiles_per_colour(desc->L, tile));
    if (dE_accum || dE_trace) {
        if ((rc = ensure(c, kDcbSlots, sizeof(int64_t) * (size_t)desc->n_rep * per_rep, &sp))) return rc;
        SMC_HIP(launch_dcb_zero((int64_t *)sp, (int64_t)desc->n_rep * per_rep, s));
    }
    const bool ea = desc->model == SMC_EA;
    const bool packed = use_dcb_packed(desc, rows, spins, ea ? couplings : nullptr, tile);
    SweepTimer timer(s, 2 * (int64_t)n_sweeps);
    for (int32_t m = 0; m < n_sweeps; ++m) {
        const uint64_t t = sweep0 + (uint64_t)m;
        const bool rev = palindromic && (t & 1u);
        for (int ci = 0; ci < 2; ++ci) {
            if (desc->dim == 3)
                SMC_HIP(launch_dcb3d((int8_t *)spins, ea ? couplings : nullptr, ea ? desc->rep_per_sample : 1,
                                     (const ThrRow *)tp, (int64_t *)sp, desc->n_rep, desc->L, tile, hits,
                                     make_key(desc->seed), (uint32_t)t, rev ? 1 - ci : ci, rev, s));
            else
                SMC_HIP(launch_dcb2d((int8_t *)spins, ea ? couplings : nullptr, ea ? desc->rep_per_sample : 1,
                                     (const ThrRow *)tp, (int64_t *)sp, desc->n_rep, desc->L, tile, hits,
                                     make_key(desc->seed), (uint32_t)t, rev ? 1 - ci : ci, rev, packed, s));
        }
        if (dE_trace)
            SMC_HIP(launch_collect((const int64_t *)sp, dE_trace + (int64_t)m * desc->n_rep, desc->n_rep, per_rep,
                                       true, s));
    }
    timer.finish();
    if (dE_accum) SMC_HIP(launch_collect((const int64_t *)sp, dE_accum, desc->n_rep, per_rep, false, s));
    return SMC_OK;
}

int smc_heis_dcb_sweep(const smc_desc *desc, void *spins, const double *beta, uint64_t sweep0, int32_t n_sweeps,
                       int32_t tile, int32_t hits, int32_t precision, int32_t palindromic, double cap,
                       int64_t *accepts, void *stream) {
    last_error().clear();
    Plan plan;
    int rc = validate(desc, false, plan);
    if (rc) return rc;
    if (desc->model != SMC_HEISENBERG)
        return fail(SMC_EUNSUPPORTED, "smc_heis_dcb_sweep is for the Heisenberg model (smc_dcb_sweep: Ising, EA)");
    if (desc->dim != 2) return fail(SMC_EUNSUPPORTED, "the Heisenberg double checkerboard is provided for 2D");
    if (desc->L <= 0) return fail(SMC_EINVAL, "the double checkerboard needs a uniform batch (L > 0)");
    if (precision < SMC_HEIS_FLOAT || precision > SMC_HEIS_DOUBLE)
        return fail(SMC_EINVAL, "unknown precision %d", precision);
    if (!heis_dcb2d_supported(desc->L, tile, precision))
        return fail(SMC_EINVAL, "tile %d: need 16, 32 or (float modes) 64, dividing L = %d into an even number "
                                "of tiles per row (or one)", tile, desc->L);
    if (hits < 1) return fail(SMC_EINVAL, "hits must be >= 1");
    if (!(cap >= 0.0 && cap <= 2.0)) return fail(SMC_EINVAL, "cap must be in [0, 2]");
    if (!spins) return fail(SMC_EINVAL, "spins is NULL");
    if ((uintptr_t)spins & 15u) return fail(SMC_EINVAL, "spins must be 16-byte aligned");
    if (!beta) return fail(SMC_EINVAL, "beta is NULL");
    if (n_sweeps < 0) return fail(SMC_EINVAL, "n_sweeps must be >= 0");
    if ((sweep0 + (uint64_t)n_sweeps) * (uint64_t)hits > (1ull << 32))
        return fail(SMC_EINVAL, "(sweep0 + n_sweeps) * hits exceeds 2^32 (the hit index is one 32-bit word)");
    for (int r = 0; r < desc->n_rep; ++r)
        if (!(beta[r] >= 0.0) || !isfinite(beta[r])) return fail(SMC_EINVAL, "beta[%d] must be finite and >= 0", r);
    if (n_sweeps == 0) return SMC_OK;
    hipStream_t s = (hipStream_t)stream;
    if (int rc_cap = refuse_capture(s)) return rc_cap;
    StreamCtx &c = ctx_for(s);
    void *bp = nullptr, *sp = nullptr;
    if (precision == SMC_HEIS_DOUBLE) {
        if ((rc = upload(c, s, kTables, beta, sizeof(double) * desc->n_rep, &bp))) return rc;
    } else {
        std::vector<float> bf(desc->n_rep);
        for (int r = 0; r < desc->n_rep; ++r) bf[r] = (float)beta[r];
        if ((rc = upload(c, s, kTables, bf.data(), sizeof(float) * bf.size(), &bp))) return rc;
    }
    const int per_rep = 2 * dcb2d_tiles_per_colour(desc->L, tile);
    if (accepts) {
        if ((rc = ensure(c, kDcbSlots, sizeof(int64_t) * (size_t)desc->n_rep * per_rep, &sp))) return rc;
        SMC_HIP(launch_dcb_zero((int64_t *)sp, (int64_t)desc->n_rep * per_rep, s));
    }
    const int64_t n_spins = (int64_t)desc->n_rep * desc->L * desc->L;
    SweepTimer timer(s, 2 * (int64_t)n_sweeps);
    for (int32_t m = 0; m < n_sweeps; ++m) {
        const uint64_t t = sweep0 + (uint64_t)m;
        const bool rev = palindromic && (t & 1u);
        for (int ci = 0; ci < 2; ++ci)
            SMC_HIP(launch_heis_dcb2d(spins, bp, (int64_t *)sp, desc->n_rep, desc->L, tile, hits, precision, cap,
                                      make_key(desc->seed), (uint32_t)t, rev ? 1 - ci : ci, rev, s));
        if (desc->renorm_every > 0 && (t + 1) % (uint64_t)desc->renorm_every == 0)
            SMC_HIP(launch_heis_dcb_renorm(spins, n_spins, precision, s));
    }
    timer.finish();
    if (accepts) SMC_HIP(launch_collect((const int64_t *)sp, accepts, desc->n_rep, per_rep, false, s));
    return SMC_OK;
}

// Checks shared by the random-number study calls; per-replica state bytes.
static int rng_study_check(const smc_desc *desc, int32_t tile, int32_t generator, int64_t *per_rep) {
    if (!desc) return fail(SMC_EINVAL, "desc is NULL");
    if (desc->dim != 2 || desc->L <= 0 || (desc->model != SMC_ISING && desc->model != SMC_EA))
        return fail(SMC_EINVAL, "the random-number study takes uniform 2D Ising or EA batches");
    if (generator < SMC_RNG_LCG32 || generator > SMC_RNG_FIB1279)
        return fail(SMC_EINVAL, "unknown generator %d", generator);
    if (tile != 16 && tile != 32) return fail(SMC_EINVAL, "tile must be 16 or 32 (got %d)", tile);
    int r = 0, s = 0;
    if (rng_study_lags(generator, &r, &s) && tile != 16)
        return fail(SMC_EINVAL, "the lagged Fibonacci generators take tile 16 (a round of T^2/2 numbers must "
                                "not exceed min(s, r - s))");
    if (desc->L % tile || (desc->L / tile) % 2)
        return fail(SMC_EINVAL, "L / tile must be an even integer (L=%d, tile=%d)", desc->L, tile);
    *per_rep = rng_study_state_bytes(generator, desc->L, tile);
    return SMC_OK;
}

int smc_rng_study_state_bytes(const smc_desc *desc, int32_t tile, int32_t generator, int64_t *bytes) {
    last_error().clear();
    int64_t per = 0;
    int rc = rng_study_check(desc, tile, generator, &per);
    if (rc) return rc;
    if (!bytes) return fail(SMC_EINVAL, "bytes is NULL");
    if (desc->n_rep < 1) return fail(SMC_EINVAL, "n_rep must be >= 1");
    *bytes = per * desc->n_rep;
    return SMC_OK;
}

int smc_rng_study_init(const smc_desc *desc, int32_t tile, int32_t generator, void *state, int64_t state_bytes,
                       void *stream) {
    last_error().clear();
    int64_t per = 0;
    int rc = rng_study_check(desc, tile, generator, &per);
    if (rc) return rc;
    if (desc->n_rep < 1) return fail(SMC_EINVAL, "n_rep must be >= 1");
    if (!state || ((uintptr_t)state & 7u)) return fail(SMC_EINVAL, "state must be a non-NULL 8-byte aligned pointer");
    if (state_bytes < per * desc->n_rep)
        return fail(SMC_EINVAL, "state holds %lld bytes, needs %lld", (long long)state_bytes,
                    (long long)(per * desc->n_rep));
    hipStream_t s = (hipStream_t)stream;
    if (int rc_cap = refuse_capture(s)) return rc_cap;
    SMC_HIP(launch_rng_init(generator, desc->L, tile, desc->n_rep, state, make_key(desc->seed), s));
    return SMC_OK;
}

int smc_rng_study_sweep(const smc_desc *desc, void *spins, const int8_t *couplings, const double *beta,
                        int32_t n_sweeps, int32_t tile, int32_t hits, int32_t generator, void *state,
                        int64_t state_bytes, int64_t *dE_accum, void *stream) {
    last_error().clear();
    int64_t per = 0;
    int rc = rng_study_check(desc, tile, generator, &per);
    if (rc) return rc;
    Plan plan;
    if ((rc = validate(desc, desc->model == SMC_EA, plan))) return rc;
    if (!spins) return fail(SMC_EINVAL, "spins is NULL");
    if (desc->model == SMC_EA && !couplings) return fail(SMC_EINVAL, "couplings are required for EA");
    if (!beta) return fail(SMC_EINVAL, "beta is NULL");
    for (int r = 0; r < desc->n_rep; ++r)
        if (!(beta[r] >= 0.0) || !isfinite(beta[r])) return fail(SMC_EINVAL, "beta[%d] must be finite and >= 0", r);
    if (hits < 1) return fail(SMC_EINVAL, "hits must be >= 1");
    if (n_sweeps < 0) return fail(SMC_EINVAL, "n_sweeps must be >= 0");
    if (!state || ((uintptr_t)state & 7u)) return fail(SMC_EINVAL, "state must be a non-NULL 8-byte aligned pointer");
    if (state_bytes < per * desc->n_rep)
        return fail(SMC_EINVAL, "state holds %lld bytes, needs %lld", (long long)state_bytes,
                    (long long)(per * desc->n_rep));
    if (n_sweeps == 0) return SMC_OK;
    hipStream_t s = (hipStream_t)stream;
    if (int rc_cap = refuse_capture(s)) return rc_cap;
    StreamCtx &c = ctx_for(s);
    std::vector<ThrRow> rows((size_t)desc->n_rep);
    for (int r = 0; r < desc->n_rep; ++r) rows[r] = threshold_row(beta[r], 2);
    void *p = nullptr;
    if ((rc = upload(c, s, kTables, rows.data(), sizeof(ThrRow) * rows.size(), &p))) return rc;
    const int rps = desc->model == SMC_EA ? desc->rep_per_sample : 1;
    for (int32_t t = 0; t < n_sweeps; ++t)
        for (int tc = 0; tc < 2; ++tc)
            SMC_HIP(launch_dcb_rng(generator, (int8_t *)spins, desc->model == SMC_EA ? couplings : nullptr, rps,
                                   (const ThrRow *)p, state, dE_accum, desc->n_rep, desc->L, tile, hits, tc, s));
    return SMC_OK;
}

int smc_msc_plan(const smc_desc *desc, int32_t n_sweeps, int32_t word_bits, int32_t *launches,
                 const char **kernel_name) {
    last_error().clear();
    if (!launches || !kernel_name) return fail(SMC_EINVAL, "output pointers are required");
    Plan plan;
    int rc = validate(desc, false, plan);
    if (rc) return rc;
    if ((rc = msc_check(desc, word_bits))) return rc;
    if (n_sweeps < 0) return fail(SMC_EINVAL, "n_sweeps must be >= 0");
    if (use_msc2d(desc, nullptr, nullptr)) {
        *kernel_name = "k_msc2d";
        *launches = n_sweeps > 0 ? 1 : 0;
    } else {
        *kernel_name = "k_half_sweep_generic";
        *launches = 2 * n_sweeps;
    }
    return SMC_OK;
}

int run_pt_split2d(StreamCtx &c, hipStream_t s, const smc_desc *desc, void *spins, SwapArgs &sw,
                   const ThrRow *thr_rows, double *energy, uint64_t step0, int32_t n_steps, int m) {
    int rc;
    const int L = desc->L, n_rep = desc->n_rep;
    const int64_t N = (int64_t)L * L;
    const size_t bytes = (size_t)n_rep * lattice2d_split_bytes(L);
    const size_t slots = lattice2d_de_slots(L, n_rep);
    if (slots == 0) return fail(SMC_EINVAL, "no band shape for L=%d", L);
    void *pp = nullptr, *q = nullptr, *tr = nullptr, *dd = nullptr, *op = nullptr;
    if ((rc = ensure(c, kLattices, 2 * bytes, &pp))) return rc;
    if ((rc = ensure(c, kL2dPart, slots * sizeof(int64_t), &q))) return rc;
    if ((rc = ensure(c, kPtThr, sizeof(ThrRow) * (size_t)n_rep, &tr))) return rc;
    if ((rc = ensure(c, kPtDelta, sizeof(int64_t) * (size_t)n_rep, &dd))) return rc;
    if ((rc = ensure(c, kPtOut, (size_t)N * (size_t)n_rep, &op))) return rc;
    uint8_t *A = (uint8_t *)pp, *B = A + bytes;
    int64_t *part = (int64_t *)q, *d = (int64_t *)dd;
    ThrRow *thr_rep = (ThrRow *)tr;
    const Key key = make_key(desc->seed);
    SMC_HIP(launch_pt_prepare(sw, energy, s));
    SMC_HIP(launch_zero64(d, n_rep, s));
    SMC_HIP(launch_to_split((const int8_t *)spins, A, L, n_rep, s));
    int64_t done = 0;  // sweeps so far (ping-pong parity)
    SweepTimer timer(s, (int64_t)n_steps * m);
    for (int32_t st = 0; st < n_steps; ++st) {
        const uint32_t t = (uint32_t)(step0 + (uint64_t)st);
        sw.t = t;
        SMC_HIP(launch_pt_gather_thr(thr_rows, sw.row_of_rep, thr_rep, n_rep, s));
        for (int j = 0; j < m; ++j, ++done)
            SMC_HIP(launch_ising2d_split(done & 1 ? B : A, false, done & 1 ? A : B, false, L, n_rep, thr_rep, part,
                                         j == 0, key,
                                         t * (uint32_t)m + (uint32_t)j, s));
        SMC_HIP(launch_lattice2d_de_collect(part, d, L, n_rep, s));
        SMC_HIP(launch_pt_add_masked(d, sw.E, sw.row_of_rep, n_rep, s));
        SMC_HIP(launch_pt_swap(sw, s));
    }
    timer.finish();
    // back to lattice order; replicas of chains that are not permutations keep their spins
    SMC_HIP(launch_from_split(done & 1 ? B : A, (int8_t *)op, L, n_rep, s));
    SMC_HIP(launch_copy_valid((const int8_t *)op, (int8_t *)spins, sw.row_of_rep, N, n_rep, s));
    SMC_HIP(launch_pt_finish(sw, energy, s));
    return SMC_OK;
}

int smc_pt_sweep_swap(const smc_desc *desc, const smc_pt_desc *pt, void *spins, const int8_t *couplings,
                      int32_t *slot_of_temp, double *energy, uint64_t step0, int32_t n_steps,
                      uint64_t *swap_accepts, void *stream) {
    last_error().clear();
    Plan plan;
    int rc = validate(desc, true, plan);
    if (rc) return rc;
    if (!pt) return fail(SMC_EINVAL, "pt desc is NULL");
    if (desc->model == SMC_HEISENBERG)
        return fail(SMC_EUNSUPPORTED, "parallel tempering is provided for Ising and EA models");
    if (pt->n_chains < 1 || pt->n_temps < 2) return fail(SMC_EINVAL, "need n_chains >= 1 and n_temps >= 2");
    if ((int64_t)pt->n_chains * pt->n_temps != desc->n_rep)
        return fail(SMC_EINVAL, "n_rep (%d) must equal n_chains * n_temps", desc->n_rep);
    if (!pt->beta) return fail(SMC_EINVAL, "beta is NULL");
    if (!spins || !slot_of_temp || !energy) return fail(SMC_EINVAL, "spins, slot_of_temp and energy are required");
    if (desc->model == SMC_EA && !couplings) return fail(SMC_EINVAL, "couplings are required for EA");
    if (n_steps < 0) return fail(SMC_EINVAL, "n_steps must be >= 0");
    if (pt->sweeps_per_step < 0) return fail(SMC_EINVAL, "sweeps_per_step must be >= 0");
    const int m = pt->sweeps_per_step > 0 ? pt->sweeps_per_step : 1;
    if ((step0 + (uint64_t)n_steps) * (uint64_t)m > (1ull << 32))
        return fail(SMC_EINVAL, "(step0 + n_steps) * sweeps_per_step exceeds 2^32 (the sweep index is 32 bits)");
    const int n = pt->n_temps;
    const int rows_n = pt->beta_per_chain ? pt->n_chains : 1;
    for (int64_t k = 0; k < (int64_t)rows_n * n; ++k)
        if (!(pt->beta[k] >= 0.0) || !isfinite(pt->beta[k])) return fail(SMC_EINVAL, "beta[%lld] invalid", (long long)k);
    if (desc->model == SMC_EA) {
        if (desc->L > 0) {
            if (desc->rep_per_sample % n) return fail(SMC_EINVAL, "rep_per_sample must be a multiple of n_temps");
        } else {
            for (int q = 0; q < pt->n_chains; ++q)
                for (int k = 1; k < n; ++k)
                    if (desc->inst[q * n + k].sample != desc->inst[q * n].sample)
                        return fail(SMC_EINVAL, "chain %d mixes coupling samples", q);
        }
    }
    if (desc->L == 0) {
        for (int q = 0; q < pt->n_chains; ++q)
            for (int k = 1; k < n; ++k)
                if (desc->inst[q * n + k].L != desc->inst[q * n].L)
                    return fail(SMC_EINVAL, "chain %d mixes lattice sizes", q);
    }
    if (n_steps == 0) return SMC_OK;
    hipStream_t s = (hipStream_t)stream;
    if (int rc_cap = refuse_capture(s)) return rc_cap;
    StreamCtx &c = ctx_for(s);
    if ((rc = upload_inst(c, s, desc, plan))) return rc;

    // tables: beta per (row, k) and threshold rows (row * n + k)
    std::vector<ThrRow> rows((size_t)rows_n * n);
    for (size_t k = 0; k < rows.size(); ++k) rows[k] = threshold_row(pt->beta[k], desc->dim);
    void *thr = nullptr, *bdev = nullptr, *E64 = nullptr, *rowrep = nullptr;
    if ((rc = upload(c, s, kTables, rows.data(), sizeof(ThrRow) * rows.size(), &thr))) return rc;
    if ((rc = upload(c, s, kBeta, pt->beta, sizeof(double) * rows.size(), &bdev))) return rc;
    BandShape sh;
    const PtRoute route = pt_route(desc, spins, couplings, rows, n, pt->n_chains, n_steps, m, &sh);
    if (route == kPtSmall3d) {
        // every step of the call in one launch, a workgroup per chain
        Small3dArgs sa;
        memset(&sa, 0, sizeof sa);
        sa.spins = (int8_t *)spins;
        sa.coup = desc->model == SMC_EA ? couplings : nullptr;
        sa.rep_per_sample = plan.b.rep_per_sample;
        sa.L = desc->L;
        sa.n_rep = desc->n_rep;
        sa.n = n;
        sa.thr = (const ThrRow *)thr;
        sa.key = make_key(desc->seed);
        sa.t0 = (uint32_t)step0;
        sa.n_steps = n_steps;
        sa.m = m;
        sa.beta_per_chain = pt->beta_per_chain ? 1 : 0;
        sa.beta = (const double *)bdev;
        sa.slot_of_temp = slot_of_temp;
        sa.energy = energy;
        sa.acc = (unsigned long long *)swap_accepts;
        SMC_HIP(launch_small3d(sa, s));
        return SMC_OK;
    }
    if ((rc = ensure(c, kEnergy64, sizeof(int64_t) * desc->n_rep, &E64))) return rc;
    if ((rc = ensure(c, kRows, sizeof(int32_t) * desc->n_rep, &rowrep))) return rc;

    SwapArgs sw;
    sw.n_chains = pt->n_chains;
    sw.n_temps = n;
    sw.beta_per_chain = pt->beta_per_chain ? 1 : 0;
    sw.beta = (const double *)bdev;
    sw.slot_of_temp = slot_of_temp;
    sw.row_of_rep = (int32_t *)rowrep;
    sw.E = (int64_t *)E64;
    sw.acc = (unsigned long long *)swap_accepts;
    sw.key = make_key(desc->seed);
    sw.t = 0;

    SweepArgs a;
    memset(&a, 0, sizeof a);
    a.b = plan.b;
    a.spins = spins;
    a.coup = desc->model == SMC_EA ? couplings : nullptr;
    a.key = make_key(desc->seed);
    a.pieces = plan.pieces;
    a.max_L = plan.max_L;
    a.thr = (const ThrRow *)thr;
    a.row_of_rep = (const int32_t *)rowrep;

    if (route == kPtSplit2d)
        return run_pt_split2d(c, s, desc, spins, sw, (const ThrRow *)thr, energy, step0, n_steps, m);
    if (route == kPtBins2d)
        return run_uneven2d(c, s, desc, spins, couplings, sw, (const ThrRow *)thr, energy, step0, n_steps, m);
    if (route == kPtPairs3d) {
        Pairs3dArgs pa;
        if (pairs3d_args(c, a, &pa) == SMC_OK)
            return run_pt_pairs3d(c, s, a, pa, sw, energy, step0, n_steps, m);
        last_error().clear();
    }
    if (route == kPtBands2d) {
        void *other = nullptr;
        if (sh.whole || ensure_spare(c, (size_t)desc->n_rep * (size_t)plan.b.N, &other) == SMC_OK)
            return run_pt_bands2d(c, s, a, sh, other, sw, energy, step0, n_steps, m);
        last_error().clear();  // no room for a second lattice: the half-sweeps need none
    }
    SMC_HIP(launch_pt_prepare(sw, energy, s));
    for (int32_t k = 0; k < n_steps; ++k) {
        const uint32_t t = (uint32_t)(step0 + (uint64_t)k);
        sw.t = t;
        CallTally tally;
        if ((rc = tally.begin(c, desc->n_rep, half_sweep_groups(a), 2 * (int64_t)m, sw.E))) return rc;
        for (int j = 0; j < m; ++j) {
            a.t = t * (uint32_t)m + (uint32_t)j;
            for (int col = 0; col < 2; ++col) {
                a.tally = tally.next();
                SMC_HIP(launch_half_sweep_generic(a, col, s));
            }
        }
        if ((rc = tally.finish(s))) return rc;
        SMC_HIP(launch_pt_swap(sw, s));
    }
    SMC_HIP(launch_pt_finish(sw, energy, s));
    return SMC_OK;
}

int smc_measure_energy_magnetisation(const smc_desc *desc, const void *spins, const int8_t *couplings,
                                     double *energy, double *magnetisation, void *stream) {
    last_error().clear();
    Plan plan;
    int rc = validate(desc, true, plan);
    if (rc) return rc;
    if (!spins || !energy) return fail(SMC_EINVAL, "spins and energy are required");
    if (desc->model == SMC_EA && !couplings) return fail(SMC_EINVAL, "couplings are required for EA");
    hipStream_t s = (hipStream_t)stream;
    if (int rc_cap = refuse_capture(s)) return rc_cap;
    StreamCtx &c = ctx_for(s);
    if ((rc = upload_inst(c, s, desc, plan))) return rc;
    const size_t bytes = measure_scratch_bytes(plan.b, plan.max_L);
    void *p = nullptr;
    if ((rc = ensure(c, kMeasure, bytes, &p))) return rc;
    SMC_HIP(launch_measure(plan.b, spins, desc->model == SMC_EA ? couplings : nullptr, plan.max_L, energy,
                           magnetisation, p, bytes, s));
    return SMC_OK;
}

}  // extern "C"

// ------------------------------------------------------ allocation-free call --
// smc_measure_energy_magnetisation_noalloc keeps its partial sums in this
// fixed array instead of the per-stream scratch.  Host code never passes the
// array's name to a kernel (on the host it is only a stand-in for the device
// symbol): the device address of each GPU's copy is looked up once per device
// with hipGetSymbolAddress and that address is what the kernels receive.
namespace smc {
constexpr size_t kNoAllocScratchBytes = 16u << 20;
static __device__ __align__(256) unsigned char scratch[kNoAllocScratchBytes];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_noalloc_mutex;
void *g_noalloc_ptr[kMaxDevices] = {};

int noalloc_scratch(void **out) {
    int dev = 0;
    SMC_HIP(hipGetDevice(&dev));
    if (dev < 0 || dev >= kMaxDevices) return fail(SMC_EUNSUPPORTED, "device index %d out of range", dev);
    std::lock_guard<std::mutex> lk(g_noalloc_mutex);
    if (!g_noalloc_ptr[dev]) {
        void *ptr = nullptr;
        SMC_HIP(hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)));
        if (!ptr) return fail(SMC_EHIP, "hipGetSymbolAddress returned no address for the scratch array");
        g_noalloc_ptr[dev] = ptr;
    }
    *out = g_noalloc_ptr[dev];
    return SMC_OK;
}
}  // namespace
}  // namespace smc

extern "C" {

int smc_measure_energy_magnetisation_noalloc(const smc_desc *desc, const void *spins, const int8_t *couplings,
                                             double *energy, double *magnetisation, void *stream) {
    using namespace smc;
    last_error().clear();
    Plan plan;
    int rc = validate(desc, true, plan);
    if (rc) return rc;
    if (desc->L <= 0) return fail(SMC_EUNSUPPORTED, "the allocation-free measurement takes uniform batches only");
    if (!spins || !energy) return fail(SMC_EINVAL, "spins and energy are required");
    if (desc->model == SMC_EA && !couplings) return fail(SMC_EINVAL, "couplings are required for EA");
    const size_t bytes = measure_scratch_bytes(plan.b, plan.max_L);
    if (bytes > kNoAllocScratchBytes)
        return fail(SMC_EINVAL, "batch needs %zu bytes of partial sums; the allocation-free call holds at most %zu",
                    bytes, kNoAllocScratchBytes);
    void *p = nullptr;
    if ((rc = noalloc_scratch(&p))) return rc;
    SMC_HIP(launch_measure(plan.b, spins, desc->model == SMC_EA ? couplings : nullptr, plan.max_L, energy,
                           magnetisation, p, bytes, (hipStream_t)stream));
    return SMC_OK;
}

}  // extern "C"
