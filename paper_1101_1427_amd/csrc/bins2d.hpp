// Tempering sweeps of 2D batches with edges in {16, 32, ..., 256}, uniform or
// uneven: bins of replicas in LDS, one launch per step (bins2d.hip).
#pragma once
#include <vector>

#include "internal.hpp"

namespace smc {

// Edges that the bins serve.
inline bool uneven2d_edge_supported(int L) { return L >= 16 && L <= 256 && L % 16 == 0; }

// Bins that are resident at once (four workgroups per compute unit).
constexpr int kBinsAtOnce = 1024;

// Up to kBinReps replicas of one edge that a workgroup sweeps together.
constexpr int kBinReps = 64;
struct Bin2d {
    int64_t packed;  // first byte of the bin in the packed copy
    int32_t first;   // first entry of the work list (replica indices)
    int32_t count;
    int32_t L;
    int32_t pad;
};

struct Bins2dArgs {
    int8_t *spins;             // caller's spins (row-major int8 +-1 per replica)
    const int8_t *coup;        // EA, else nullptr
    uint8_t *packed;           // the replicas in LDS layout between steps, or nullptr
    const smc_inst *inst;      // device [n_rep]
    const Bin2d *bins;
    const int32_t *work;
    const ThrRow *thr;
    // The state of the chains before the launch and after it: threshold row per replica (-1
    // leaves the chain unchanged), slot per temperature, tracked energy per replica.  The
    // workgroups read the one and write the other.
    const int32_t *row_in, *slot_in;
    int32_t *row_out, *slot_out;  // with `swap` only
    const int64_t *E_in;
    int64_t *E_out;
    // With `swap` the exchange round of step swap_t comes before the sweeps.
    int swap;
    uint32_t swap_t;
    int n_temps, beta_per_chain;
    const double *beta;
    unsigned long long *acc;      // [n_chains][n_temps - 1] or nullptr
    Key key;
    uint32_t t;                // first sweep
    int sweeps;
};

// The bins of a batch (rows: edge and offsets of every replica), largest
// edges first; returns the dynamic LDS of a launch.
size_t make_bins2d(const std::vector<smc_inst> &rows, std::vector<Bin2d> *bins, std::vector<int32_t> *work);
// Estimate of a sweep's time (ns) for a uniform batch.
double bins2d_ns(int L, int n_rep);
// Launches for so many bins (of fewer than 2^32 work-items each).
int bins2d_launches(int n_bins);
// raw_in: from the caller's spins and couplings (else from the packed copy);
// raw_out: to the caller's spins.
hipError_t launch_bins2d(const Bins2dArgs &a, int n_bins, size_t lds, bool raw_in, bool raw_out, hipStream_t s);

}  // namespace smc
