// Per-replica sums (energy changes, accepted moves) of the sweep kernels: a
// workgroup's sum goes into a slot of its own, added up over the launches of
// a call, and one small kernel at the call's end adds the slots of each
// replica to the caller's total.  Workgroups that add to the total itself
// are served one after the other by the memory side: of the 1024 workgroups
// of a 256^3 EA half-sweep each waited for the others: 20 us per launch
// instead of 11.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace smc {

struct Tally {
    int64_t *slots;  // [n_rep][workgroups per replica], or nullptr: add to total
    int64_t *total;  // [n_rep], or nullptr: no sums wanted
    int first;       // the call's first launch writes its slots, the others add to them
};

__device__ __forceinline__ bool tally_wanted(const Tally &t) { return t.slots || t.total; }

// One thread of the workgroup with index `group` of the grid (replica r).
__device__ __forceinline__ void tally_put(const Tally &t, int64_t group, int r, long long sum) {
    if (t.slots)
        t.slots[group] = t.first ? sum : t.slots[group] + sum;
    else if (sum != 0)
        atomicAdd((unsigned long long *)&t.total[r], (unsigned long long)sum);
}

// dE[r] = (assign) or += (otherwise) the sum of replica r's slots.
hipError_t launch_collect(const int64_t *slots, int64_t *dE, int n_rep, int per_rep, bool assign, hipStream_t s);

}  // namespace smc
