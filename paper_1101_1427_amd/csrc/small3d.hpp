// Small 3D Ising / +-J EA lattices with whole replicas in LDS (small3d.hip).
#pragma once
#include "internal.hpp"

namespace smc {

constexpr int kSmall3dMaxReps = 64;  // replicas per workgroup at most

struct Small3dArgs {
    int8_t *spins;            // [n_rep][L^3]
    const int8_t *coup;       // EA: [sample][3][L^3], else nullptr
    int rep_per_sample;
    int L, n_rep, n;          // n replicas per workgroup (tempering: the chain's temperatures)
    const ThrRow *thr;        // by replica (sweeps); by temperature, [chain][n] with beta_per_chain (tempering)
    Key key;
    uint32_t t0;              // first sweep (sweeps) or step (tempering)
    int n_steps, m;           // tempering: steps and sweeps per step; sweeps: 1 and the number of sweeps
    int rng_shift;
    int64_t *dE;              // sweeps: [n_rep] energy changes, or nullptr
    // tempering (slot_of_temp != nullptr)
    int beta_per_chain;
    const double *beta;
    int32_t *slot_of_temp;
    double *energy;
    unsigned long long *acc;  // [n_chains][n - 1] or nullptr
};

bool small3d_supported(int dim, int L);
int small3d_max_reps(int L);
// Whether tempering of n_chains chains of n replicas is faster with a chain per
// workgroup than with its replicas spread over the chip.
bool small3d_tempers(int L, int n, int n_chains);
// Words before and after the staged replicas: reads at the distances that a
// word does not need (its masks drop them) stay inside.
inline __host__ __device__ int small3d_pad(int L) { return L % 16 ? (L * L * L / 2 + 7) / 8 + 4 : 0; }
hipError_t launch_small3d(const Small3dArgs &a, hipStream_t s);

}  // namespace smc
