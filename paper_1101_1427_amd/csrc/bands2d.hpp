// Sweeps of uniform 2D Ising / +-J EA batches of any even edge with bands of
// rows, or tiles, in LDS and several sweeps per launch (tiles2d.hip).
#pragma once
#include "internal.hpp"

namespace smc {

// How a batch is cut: `rows` rows per workgroup and, of edges that are
// multiples of 16, `words` pieces of 16 sites of them (the whole
// lattice when whole), `sweeps` sweeps per launch, `threads` per workgroup.
struct BandShape {
    int rows = 0, words = 0, sweeps = 0, threads = 0;
    bool whole = false;
    double ns_per_sweep = 0.0;  // the model's estimate for the batch
};

// The shape for a batch of n_rep lattices and n_sweeps sweeps; false if none
// fits in LDS.  even: see bands2d_launches.
bool bands2d_shape(int L, int n_rep, bool ea, int n_sweeps, bool even, BandShape *out);
// The shape that holds whole lattices, of workgroups of at most most_threads.
bool bands2d_whole(int L, int n_rep, bool ea, int n_sweeps, int most_threads, BandShape *out);
int bands2d_groups(int L, const BandShape &sh);  // workgroups per replica
int bands2d_pieces(int L);                       // pieces per staged row
size_t bands2d_lds(int cells);                   // bytes for so many staged pieces
// Launches for n_sweeps sweeps; with even, an even number unless the shape is
// whole, so that the result ends where it began (more than n_sweeps: the shape
// does not serve the call).
int bands2d_launches(const BandShape &sh, int n_sweeps, bool even);

struct Bands2dArgs {
    const int8_t *src;         // [n_rep][L * L]
    int8_t *dst;               // may be src when the shape is whole
    const int8_t *coup;        // EA: [sample][2][L * L], else nullptr
    int rep_per_sample;
    const ThrRow *thr;
    const int32_t *row_of_rep; // threshold row per replica (-1: copied unchanged), or nullptr
    Key key;
    uint32_t t;                // first sweep of the launch
    int rng_shift;
    int n_rep, L;
};
hipError_t launch_bands2d(const Bands2dArgs &a, const BandShape &sh, int sweeps, const Tally &tally, hipStream_t s);

}  // namespace smc
