// Sweeps of small uniform Heisenberg lattices, 2D and 3D (Sec. 4), with a whole
// replica in LDS for every sweep and renormalisation of a call, in place.
//
// A workgroup holds a replica as three arrays of components, row-major.  A thread
// takes pairs of sites (2h, 2h + 1), one of either colour; the draw of a move is keyed by
// the pair, as in the other kernels, and the arithmetic is theirs.
//
// Bound: VALU and the latency of a half-sweep on the compute unit that holds the
// replica; the two launches per sweep, and every site read and written through
// memory by each, are gone.
// Per sweep, against two half-sweep launches: one 8^3 lattice 1.5 us (5.6), one 16^3 4.7
// (9.1), 50 of 22^3 11.3 (17.9), 256 of them 11.6 (50), 1024 of 16^3 20 (41), 64 of 64^2 4.1
// (10.9), 256 of 114^2 12.5 (39).
#include <algorithm>

#include "heis_math.hpp"
#include "internal.hpp"

namespace smc {
namespace {

constexpr int kMaxThreads = 1024;

struct KArgs {
    float *spins;       // [n_rep][N][3]
    const float *beta;  // per replica
    int64_t *acc;       // += accepted moves per replica, or nullptr
    Key key;
    uint32_t t;
    int sweeps, renorm_every;
    int L, N;
};

// Where a thread's next pair lies: pair k of row (y, z), advanced without divisions.
struct Walk {
    int k, y, z, h;
    __device__ __forceinline__ void next(int dk, int dy, int dz, int step, int Lh, int L) {
        h += step;
        k += dk;
        y += dy;
        z += dz;
        if (k >= Lh) {
            k -= Lh;
            ++y;
        }
        if (y >= L) {
            y -= L;
            ++z;
        }
    }
};

template <int DIM>
__global__ __launch_bounds__(kMaxThreads) void k_heis_small(KArgs a) {
    extern __shared__ __align__(16) float lds[];  // [3][N]
    __shared__ int red[kMaxThreads / 64];
    const int L = a.L, Lh = L / 2, N = a.N, P = L * L, tid = (int)threadIdx.x, nt = (int)blockDim.x;
    const int r = (int)blockIdx.x;
    float *S = a.spins + (size_t)r * 3 * (size_t)N;
    float *X = lds, *Y = lds + N, *Z = lds + 2 * N;
    for (int i = tid; i < N; i += nt) {
        X[i] = S[3 * i];
        Y[i] = S[3 * i + 1];
        Z[i] = S[3 * i + 2];
    }
    const float beta = a.beta[r];
    const int drow = nt / Lh, dk = nt - drow * Lh, dz = drow / L, dy = drow - dz * L;
    Walk first;
    first.h = tid;
    const int row = tid / Lh;
    first.k = tid - row * Lh;
    first.z = row / L;
    first.y = row - first.z * L;
    int n_acc = 0;
    __syncthreads();
    for (int sw = 0; sw < a.sweeps; ++sw) {
        const uint32_t t = a.t + (uint32_t)sw;
        for (uint32_t c = 0; c < 2; ++c) {
            for (Walk w = first; w.h < N / 2; w.next(dk, dy, dz, nt, Lh, L)) {
                const int x = 2 * w.k + (int)(((uint32_t)(w.y + w.z) ^ c) & 1u);
                const int i = (w.z * L + w.y) * L + x;
                float3 hf = make_float3(0.f, 0.f, 0.f);
                auto add = [&](int j) {
                    hf.x += X[j];
                    hf.y += Y[j];
                    hf.z += Z[j];
                };
                add(i + (x == L - 1 ? 1 - L : 1));
                add(i - (x == 0 ? 1 - L : 1));
                add(i + (w.y == L - 1 ? L - P : L));
                add(i - (w.y == 0 ? L - P : L));
                if constexpr (DIM == 3) {
                    add(i + (w.z == L - 1 ? P - N : P));
                    add(i - (w.z == 0 ? P - N : P));
                }
                const uint4 u =
                    philox4x32_10_wide(make_uint4((uint32_t)w.h, t, (uint32_t)r, 2 * kTagHeis + c), a.key);
                const float3 sp = heis_proposal(unit23f(u.x), unit23f(u.y));
                const float3 so = make_float3(X[i], Y[i], Z[i]);
                const float dE = -((sp.x - so.x) * hf.x + (sp.y - so.y) * hf.y + (sp.z - so.z) * hf.z);
                if (dE <= 0.0f || unit23f(u.z) < heis_boltzmann(beta, dE)) {
                    X[i] = sp.x;
                    Y[i] = sp.y;
                    Z[i] = sp.z;
                    ++n_acc;
                }
            }
            __syncthreads();
        }
        if (a.renorm_every > 0 && ((uint64_t)t + 1) % (uint64_t)a.renorm_every == 0) {
            for (int i = tid; i < N; i += nt) {
                const float3 u = heis_unit(X[i], Y[i], Z[i]);
                X[i] = u.x;
                Y[i] = u.y;
                Z[i] = u.z;
            }
            __syncthreads();
        }
    }
    for (int i = tid; i < N; i += nt) {
        S[3 * i] = X[i];
        S[3 * i + 1] = Y[i];
        S[3 * i + 2] = Z[i];
    }
    if (a.acc) {
        int v = n_acc;
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
        if ((tid & 63) == 0) red[tid >> 6] = v;
        __syncthreads();
        if (tid == 0) {
            long long tot = 0;
            for (int w = 0; w < nt >> 6; ++w) tot += red[w];
            atomicAdd((unsigned long long *)&a.acc[r], (unsigned long long)tot);
        }
    }
}

int sites_of(int dim, int L) { return dim == 3 ? L * L * L : L * L; }

}  // namespace

bool heis_small_supported(int dim, int L) {
    return L >= 4 && L % 2 == 0 && L <= (dim == 3 ? 22 : 114) && (dim == 2 || dim == 3);
}

hipError_t launch_heis_small(float *spins, const float *beta, int64_t *acc, int n_rep, int dim, int L, Key key,
                             uint32_t t, int sweeps, int renorm_every, hipStream_t s) {
    if (!heis_small_supported(dim, L) || n_rep < 1 || sweeps < 1) return hipErrorInvalidValue;
    KArgs a;
    a.spins = spins;
    a.beta = beta;
    a.acc = acc;
    a.key = key;
    a.t = t;
    a.sweeps = sweeps;
    a.renorm_every = renorm_every;
    a.L = L;
    a.N = sites_of(dim, L);
    const int threads = std::min(kMaxThreads, (a.N / 2 + 63) / 64 * 64);
    const size_t lds = 3 * sizeof(float) * (size_t)a.N;
    void (*kernel)(KArgs) = dim == 3 ? k_heis_small<3> : k_heis_small<2>;
    if (lds > 65536 - 1024)
        if (hipError_t e = hipFuncSetAttribute((const void *)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds))
            return e;
    SMC_LAUNCH(kernel, dim3((unsigned)n_rep), dim3(threads), lds, s, a);
    return hipGetLastError();
}

}  // namespace smc
