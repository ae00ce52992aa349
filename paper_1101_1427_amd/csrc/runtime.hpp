// The host runtime of the C-ABI layer: error text, per-stream device
// scratch and pinned staging, acceptance tables, argument validation and
// the predicates that choose an execution path.  Used by the entry points
// (api.hip) and the autotuner (tune.hip); defined in runtime.hip.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include <string>
#include <vector>

#include "internal.hpp"

namespace smc {

// The calling thread's text of the last error (smc_last_error).
std::string &last_error();
// Records the message and returns code.
int fail(int code, const char *fmt, ...);

#define SMC_HIP(call)                                                                                    \
    do {                                                                                                 \
        hipError_t e_ = (call);                                                                          \
        if (e_ != hipSuccess) {                                                                          \
            const std::string why_ = take_launch_rejection();                                            \
            return fail(SMC_EHIP, "%s: %s%s%s", #call, hipGetErrorString(e_), why_.empty() ? "" : ": ", \
                        why_.c_str());                                                                   \
        }                                                                                                \
    } while (0)

// ------------------------------------------------------------------ scratch --
// Device scratch and a pinned staging area, one set per (device, stream):
// calls on one stream are ordered, so reusing the set between them is safe;
// calls on different streams never share a set.
struct Buffer {
    void *p = nullptr;
    size_t bytes = 0;
    // uploaded slots: pinned staging, the event of its last copy, and the
    // bytes last uploaded (an identical upload is skipped)
    void *pinned = nullptr;
    size_t pinned_bytes = 0;
    hipEvent_t staged = nullptr;
    bool staged_pending = false;
    std::vector<unsigned char> last;
};

enum Slot {
    kTables = 0,
    kInst,
    kSamples,
    kMeasure,
    kEnergy64,
    kRows,
    kBeta,
    kWork,
    kTuneSpins,
    kL2dPart,
    kMscSpins,
    kMscCoup,
    kMscEnergy,
    kMscGauge,
    kDcbSlots,
    kLattices,   // second lattices or packed copies: a call has one kind of them at most
    kBins2d,     // bins of the 2D tempering batches
    kTallySlots, // per-workgroup sums of a sweep call
    kPtThr,
    kPtDelta,
    kPtOut,
    kBonds3d,    // bit-packed 3D EA bonds of the segment sweep
    kTuneA,      // scratch lattices of the launch-shape tuner
    kTuneB,
    kNumSlots
};

struct StreamCtx {
    hipStream_t stream = nullptr;  // the stream whose calls use this set
    Buffer dev[kNumSlots];
};

StreamCtx &ctx_for(hipStream_t s);
// Device buffer of at least `bytes` in a slot of the set.
int ensure(StreamCtx &c, Slot slot, size_t bytes, void **out);
// kLattices for a path that another stands in for where there is no room (SMC_ENOMEM): it is
// not grown to more than half of the memory that is free, so that a caller who fills
// the card with lattices keeps the rest.
int ensure_spare(StreamCtx &c, size_t bytes, void **out);
bool spare_fits(size_t bytes, size_t held, size_t free_bytes);
// Frees a slot's device buffer once the set's stream has finished with it.
int release(StreamCtx &c, Slot slot);
// Host bytes into a slot through its pinned staging area.
int upload(StreamCtx &c, hipStream_t s, Slot slot, const void *src, size_t bytes, void **dev_out);
// SMC_EINVAL (nothing issued) if s is capturing a graph.
int refuse_capture(hipStream_t s);

// ----------------------------------------------------------------- tables ----
ThrRow threshold_row(double beta, int dim);

// ------------------------------------------------------------------ paths ----
bool use_heis3d(const smc_desc *d);
bool use_heis3d_tiled(const smc_desc *d, int64_t n_sweeps);
bool use_heis_small(const smc_desc *d, int64_t n_sweeps);
// Small 3D edges with whole replicas on chip (SPINMC_SMALL3D=0: never).
bool use_small3d(const smc_desc *d);
// 3D tempering of edge 16 and at most 32 temperatures, which always runs there
// (the "k_pt3d_chain" path; SPINMC_PT3D=0: never), and of the other small edges.
bool use_pt3d(const smc_desc *d, int n_temps);
bool use_small3d_pt(const smc_desc *d, int n_temps, int n_chains);
bool use_lattice2d(const smc_desc *d, const void *spins, const std::vector<ThrRow> &rows);
// Whether 2D tiles come before the one-pass kernel on an edge that both serve.
bool bands_before_lattice2d(const smc_desc *d, int32_t n_sweeps, bool tempering);
bool sweep3d_shape(const smc_desc *d);
bool pass3d_enabled(const smc_desc *d);
bool use_sweep3d(const smc_desc *d, const void *spins, const int8_t *coup, const std::vector<ThrRow> &rows);
// The packed copy of 3D lattices for a call of n_sweeps sweeps; a launch shape of the 3D
// kernels on the caller's bytes asked for in the environment.
bool use_pairs3d(const smc_desc *d, int64_t n_sweeps);
bool sweep3d_asked_for();
bool use_pt_split2d(const smc_desc *d, const void *spins, const std::vector<ThrRow> &rows);

// --------------------------------------------------------------- validation --
struct Plan {
    Batch b;
    int max_L = 0;
    PieceUse pieces = kNoPieces;
    int64_t n_samples = 0;
    std::vector<smc_inst> samples;  // distinct samples (EA): L, sample, -, coup_off
};

int64_t sites(int dim, int L);
// The coupling samples of a uniform EA batch: sample q at q * d * N.
void fill_uniform_samples(const smc_desc *d, Plan &plan);
int validate(const smc_desc *d, bool need_coup, Plan &plan);
// The instance table of an uneven batch into its scratch slot (plan.b.inst).
int upload_inst(StreamCtx &c, hipStream_t s, const smc_desc *d, Plan &plan);

}  // namespace smc
