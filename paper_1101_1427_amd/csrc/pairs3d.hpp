// Sweeps of uniform 3D Ising / +-J EA batches (any even edge from 16) on a
// packed copy of half a byte per site (pairs3d.hip).
#pragma once
#include "internal.hpp"

namespace smc {

struct Pairs3dArgs {
    uint32_t *packed;          // pairs3d_bytes(L, n_rep)
    int rep_per_sample;        // of the couplings (packing)
    const ThrRow *thr;
    const int32_t *row_of_rep; // threshold row per replica (-1: left unchanged), or nullptr
    Key key;
    uint32_t t;
    int rng_shift;
    int n_rep, L;
};

bool pairs3d_supported(int dim, int L);
// Whether the launches for a batch stay below 2^32 work-items (a thread per 16 sites;
// the kernels on the caller's bytes have up to 16 times fewer threads).
bool pairs3d_launchable(int L, int n_rep);
// Bytes of the packed copy.
size_t pairs3d_bytes(int L, int n_rep);
hipError_t launch_pairs3d_pack(const int8_t *spins, const int8_t *coup, const Pairs3dArgs &a, hipStream_t s);
hipError_t launch_pairs3d_unpack(int8_t *spins, const Pairs3dArgs &a, hipStream_t s);
int pairs3d_planes(int L, int n_rep);         // planes per thread for a batch
int pairs3d_groups(int L, int planes);        // workgroups per replica of a half-sweep
hipError_t launch_pairs3d_half(const Pairs3dArgs &a, bool ea, int c, int planes, const Tally &tally, hipStream_t s);

}  // namespace smc
