#include "tally.hpp"

#include "internal.hpp"

namespace smc {
namespace {

// One workgroup per replica.  Bound by the latency of its loads, so eight
// per thread are in flight.
__global__ __launch_bounds__(1024) void k_collect(const int64_t *slots, int64_t *dE, int per_rep, int assign) {
    __shared__ long long red[16];
    const int64_t *p = slots + (int64_t)blockIdx.x * per_rep;
    long long v = 0;
    if (per_rep <= (int)blockDim.x) {
        if ((int)threadIdx.x < per_rep) v = p[threadIdx.x];
    } else {
#pragma unroll 8
        for (int i = (int)threadIdx.x; i < per_rep; i += (int)blockDim.x) v += p[i];
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    if (threadIdx.x == 0) {
        long long sum = 0;
        for (int w = 0; w < (int)(blockDim.x >> 6); ++w) sum += red[w];
        // (calls on other streams may add to the same total)
        if (assign)
            dE[blockIdx.x] = sum;
        else
            atomicAdd((unsigned long long *)&dE[blockIdx.x], (unsigned long long)sum);
    }
}

}  // namespace

hipError_t launch_collect(const int64_t *slots, int64_t *dE, int n_rep, int per_rep, bool assign, hipStream_t s) {
    const int threads = per_rep <= 64 ? 64 : per_rep <= 512 ? 256 : 1024;
    SMC_LAUNCH(k_collect, dim3((unsigned)n_rep), dim3(threads), 0, s, slots, dE, per_rep, assign ? 1 : 0);
    return hipGetLastError();
}

}  // namespace smc
