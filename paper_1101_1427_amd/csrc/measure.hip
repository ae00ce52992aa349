// Energy and magnetisation of every replica (Eqs. 1, 10, 11; Sec. 3.5,
// Sec. 4): partial sums per workgroup, then one workgroup per replica adds
// them in a fixed order.
//
// Bound: memory.  A thread owns 16 sites of a row (one site: Heisenberg) and
// walks along the slowest axis (y in 2D, z in 3D), so the neighbour row it
// loads is its own row of the next step and a lattice is read about once;
// the remaining neighbours are in lines that its wavefront loads anyway.
// Ising and EA bonds are counted four to a word: (a ^ b) & 2 per byte of two
// +-1 spin bytes (and the bond's byte) and one population count, three
// instructions per word and direction, no multiplication and no division per
// site.  Any even edge: a row's last piece may hold fewer than 16 sites, and
// no access needs more than byte alignment.
//
// Three lattices of 16384^2 (0.805 GB): 160 us = 5.0 TB/s; one byte load per
// neighbour with 64-bit divisions and a serial final sum per replica took 1703.
#include "internal.hpp"
#include "intrin.hpp"
#include "rows.hpp"

namespace smc {

namespace {

constexpr int kBlock = 256;
constexpr int kMaxStrip = 16;  // rows along the slowest axis per thread

struct Partial {
    double e, mx, my, mz;
};

struct MeasureOut {
    Partial *part;   // [n_rep][nblk], used when nblk > 1
    double *energy;  // written directly when nblk == 1
    double *magnet;  // [n_rep] or [n_rep][3], or nullptr
    int nblk;        // workgroups per replica
    int strip;       // rows per thread along the slowest axis
};

__device__ __forceinline__ void put(const MeasureOut &o, bool vec, int r, const Partial &p) {
    o.energy[r] = p.e;
    if (!o.magnet) return;
    if (vec) {
        o.magnet[3 * (int64_t)r] = p.mx;
        o.magnet[3 * (int64_t)r + 1] = p.my;
        o.magnet[3 * (int64_t)r + 2] = p.mz;
    } else {
        o.magnet[r] = p.mx;
    }
}

// Sum over the workgroup of N doubles per thread, in a fixed order; valid in
// thread 0.
template <int N>
__device__ __forceinline__ void block_sum(double (&v)[N], double (*smem)[N]) {
#pragma unroll
    for (int k = 0; k < N; ++k)
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) v[k] += __shfl_xor(v[k], o, 64);
    if ((threadIdx.x & 63) == 0)
#pragma unroll
        for (int k = 0; k < N; ++k) smem[threadIdx.x >> 6][k] = v[k];
    __syncthreads();
    if (threadIdx.x == 0) {
#pragma unroll
        for (int k = 0; k < N; ++k) v[k] = 0.0;
        for (int w = 0; w < (int)(blockDim.x >> 6); ++w)
#pragma unroll
            for (int k = 0; k < N; ++k) v[k] += smem[w][k];
    }
}

__device__ __forceinline__ uint32_t count2(uint32_t a, uint32_t b, uint32_t m, uint32_t acc) {
    return (uint32_t)__popc(__builtin_amdgcn_bitop3_b32(a, b, m, 0x28)) + acc;  // (a ^ b) & m
}

__device__ __forceinline__ uint32_t count_bonds(const uint4 &a, const uint4 &b, const uint4 &m, uint32_t acc) {
    return count2(a.x, b.x, m.x, count2(a.y, b.y, m.y, count2(a.z, b.z, m.z, count2(a.w, b.w, m.w, acc))));
}

__device__ __forceinline__ uint4 xor4(const uint4 &a, const uint4 &b) {
    return make_uint4(a.x ^ b.x, a.y ^ b.y, a.z ^ b.z, a.w ^ b.w);
}

template <int DIM, bool EA>
__global__ __launch_bounds__(kBlock) void k_measure_ising(Batch b, const int8_t *spins, const int8_t *coup,
                                                          MeasureOut out) {
    __shared__ double red[kBlock / 64][2];
    const int r = blockIdx.x / out.nblk, bx = blockIdx.x % out.nblk;
    const smc_inst g = replica_geom(b, r);
    const int L = g.L;
    const int64_t LL = L, P = DIM == 3 ? LL * LL : LL, N = P * LL;
    const int8_t *S = spins + g.spin_off;
    const int8_t *J = EA ? coup + g.coup_off : nullptr;
    const uint32_t pieces = (uint32_t)(L + 15) >> 4;               // per row
    const uint32_t cols = DIM == 3 ? pieces * (uint32_t)L : pieces;  // per plane (3D) or row (2D)
    const uint32_t strips = ((uint32_t)L + out.strip - 1) / out.strip;
    uint32_t unsat = 0, minus = 0;
    for (uint32_t q = bx * kBlock + threadIdx.x; q < cols * strips; q += out.nblk * kBlock) {
        const uint32_t st = q / cols, col = q - st * cols;
        const uint32_t y = DIM == 3 ? col / pieces : 0u;
        const int x0 = (int)(col - y * pieces) << 4;
        const RowEnd end(L - x0);
        const int64_t in_plane = (int64_t)y * L + x0;
        int64_t i = (int64_t)(st * out.strip) * P + in_plane;
        uint4 own = load16(S, i, N);
        const int last = min((int)(st * out.strip) + out.strip, L);
        for (int z = (int)(st * out.strip); z < last; ++z) {
            const int64_t up = z == L - 1 ? in_plane : i + P;
            const uint4 next = load16(S, up, N);
            const uint32_t xr = (uint8_t)S[end.partial ? i - x0 : x0 + 16 == L ? i - x0 : i + 16];
            const uint4 right = end.shifted_down(own, xr);
            if constexpr (EA) {
                unsat = count_bonds(xor4(own, load16(J, i, N)), right, end.m2, unsat);
                if constexpr (DIM == 3) {
                    const int64_t iy = (int)y == L - 1 ? i - (P - LL) : i + LL;
                    unsat = count_bonds(xor4(own, load16(J + N, i, N)), load16(S, iy, N), end.m2, unsat);
                }
                unsat = count_bonds(xor4(own, load16(J + (DIM - 1) * N, i, N)), next, end.m2, unsat);
            } else {
                unsat = count_bonds(own, right, end.m2, unsat);
                if constexpr (DIM == 3) {
                    const int64_t iy = (int)y == L - 1 ? i - (P - LL) : i + LL;
                    unsat = count_bonds(own, load16(S, iy, N), end.m2, unsat);
                }
                unsat = count_bonds(own, next, end.m2, unsat);
            }
            minus = (uint32_t)__popc(own.x & end.m2.x) + (uint32_t)__popc(own.y & end.m2.y) +
                    (uint32_t)__popc(own.z & end.m2.z) + (uint32_t)__popc(own.w & end.m2.w) + minus;
            own = next;
            i = up;
        }
    }
    double v[2] = {(double)unsat, (double)minus};
    block_sum<2>(v, red);
    if (threadIdx.x == 0) {
        // E = (unsatisfied - satisfied bonds), M = (plus - minus spins); the
        // constants enter once per replica (whole numbers below 2^53: exact)
        const double n = bx == 0 ? (double)N : 0.0;
        const Partial p{2.0 * v[0] - DIM * n, n - 2.0 * v[1], 0.0, 0.0};
        if (out.nblk == 1)
            put(out, false, r, p);
        else
            out.part[(int64_t)r * out.nblk + bx] = p;
    }
}

__device__ __forceinline__ float3 ld3(const float *s, int64_t i) {
    return make_float3(s[3 * i], s[3 * i + 1], s[3 * i + 2]);
}

__device__ __forceinline__ double dot3(const float3 &a, const float3 &b) {
    return (double)a.x * b.x + (double)a.y * b.y + (double)a.z * b.z;
}

template <int DIM>
__global__ __launch_bounds__(kBlock) void k_measure_heis(Batch b, const float *spins, MeasureOut out) {
    __shared__ double red[kBlock / 64][4];
    const int r = blockIdx.x / out.nblk, bx = blockIdx.x % out.nblk;
    const smc_inst g = replica_geom(b, r);
    const int L = g.L;
    const int64_t LL = L, P = DIM == 3 ? LL * LL : LL;
    const float *S = spins + 3 * g.spin_off;
    const uint32_t cols = DIM == 3 ? (uint32_t)L * L : (uint32_t)L;
    const uint32_t strips = ((uint32_t)L + out.strip - 1) / out.strip;
    double v[4] = {0.0, 0.0, 0.0, 0.0};
    for (uint64_t q = bx * kBlock + threadIdx.x; q < (uint64_t)cols * strips; q += out.nblk * kBlock) {
        const uint32_t st = (uint32_t)(q / cols), col = (uint32_t)(q - (uint64_t)st * cols);
        const int y = DIM == 3 ? (int)(col / (uint32_t)L) : 0, x = DIM == 3 ? (int)(col % (uint32_t)L) : (int)col;
        int64_t i = (int64_t)(st * out.strip) * P + col;
        float3 own = ld3(S, i);
        const int last = min((int)(st * out.strip) + out.strip, L);
        for (int z = (int)(st * out.strip); z < last; ++z) {
            const int64_t up = z == L - 1 ? (int64_t)col : i + P;
            const float3 next = ld3(S, up);
            double e = dot3(own, ld3(S, x == L - 1 ? i - (LL - 1) : i + 1)) + dot3(own, next);
            if constexpr (DIM == 3) e += dot3(own, ld3(S, y == L - 1 ? i - (P - LL) : i + LL));
            v[0] -= e;
            v[1] += own.x;
            v[2] += own.y;
            v[3] += own.z;
            own = next;
            i = up;
        }
    }
    block_sum<4>(v, red);
    if (threadIdx.x == 0) {
        const Partial p{v[0], v[1], v[2], v[3]};
        if (out.nblk == 1)
            put(out, true, r, p);
        else
            out.part[(int64_t)r * out.nblk + bx] = p;
    }
}

// One workgroup per replica: its partial sums in a fixed order.
__global__ __launch_bounds__(kBlock) void k_measure_final(bool vec, MeasureOut out) {
    __shared__ double red[kBlock / 64][4];
    const Partial *part = out.part + (int64_t)blockIdx.x * out.nblk;
    double v[4] = {0.0, 0.0, 0.0, 0.0};
    for (int k = threadIdx.x; k < out.nblk; k += kBlock) {
        const Partial p = part[k];
        v[0] += p.e;
        v[1] += p.mx;
        v[2] += p.my;
        v[3] += p.mz;
    }
    block_sum<4>(v, red);
    if (threadIdx.x == 0) put(out, vec, (int)blockIdx.x, Partial{v[0], v[1], v[2], v[3]});
}

int64_t sites_of(int dim, int L) { return dim == 3 ? (int64_t)L * L * L : (int64_t)L * L; }

// Most workgroups per replica (the scratch array holds one partial sum each).
int measure_blocks(const Batch &b, int max_L) {
    int64_t nb = (sites_of(b.dim, max_L) + 4095) / 4096;
    if (nb < 1) nb = 1;
    if (nb > 2048) nb = 2048;
    return (int)nb;
}

}  // namespace

size_t measure_scratch_bytes(const Batch &b, int max_L) {
    return (size_t)measure_blocks(b, max_L) * (size_t)b.n_rep * sizeof(Partial);
}

hipError_t launch_measure(const Batch &b, const void *spins, const int8_t *coup, int max_L, double *energy,
                          double *magnet, void *scratch, size_t scratch_bytes, hipStream_t s) {
    if (scratch_bytes < measure_scratch_bytes(b, max_L)) return hipErrorInvalidValue;
    const bool heis = b.model == SMC_HEISENBERG;
    // Threads of a replica at `strip` rows each.  Long strips read fewer
    // neighbour rows twice, short ones give more threads: the longest that
    // still gives a workgroup per replica and 2^18 threads in all (four
    // wavefronts on every SIMD), one row at the least.
    const int64_t cols = (b.dim == 3 ? max_L : 1) * (int64_t)(heis ? max_L : (max_L + 15) / 16);
    int strip = kMaxStrip;
    auto threads = [&]() { return cols * ((max_L + strip - 1) / strip); };
    while (strip > 1 && (threads() < kBlock || threads() * b.n_rep < (1 << 18))) strip >>= 1;
    MeasureOut out;
    out.part = (Partial *)scratch;
    out.energy = energy;
    out.magnet = magnet;
    out.strip = strip;
    const int64_t want = (threads() + kBlock - 1) / kBlock;
    const int most = measure_blocks(b, max_L);
    out.nblk = want < most ? (int)want : most;
    const dim3 grid((unsigned)(out.nblk * b.n_rep));
    if (heis) {
        if (b.dim == 3)
            SMC_LAUNCH(k_measure_heis<3>, grid, dim3(kBlock), 0, s, b, (const float *)spins, out);
        else
            SMC_LAUNCH(k_measure_heis<2>, grid, dim3(kBlock), 0, s, b, (const float *)spins, out);
    } else if (b.dim == 3) {
        if (coup)
            SMC_LAUNCH((k_measure_ising<3, true>), grid, dim3(kBlock), 0, s, b, (const int8_t *)spins, coup, out);
        else
            SMC_LAUNCH((k_measure_ising<3, false>), grid, dim3(kBlock), 0, s, b, (const int8_t *)spins, coup, out);
    } else {
        if (coup)
            SMC_LAUNCH((k_measure_ising<2, true>), grid, dim3(kBlock), 0, s, b, (const int8_t *)spins, coup, out);
        else
            SMC_LAUNCH((k_measure_ising<2, false>), grid, dim3(kBlock), 0, s, b, (const int8_t *)spins, coup, out);
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || out.nblk == 1) return e;
    SMC_LAUNCH(k_measure_final, dim3((unsigned)b.n_rep), dim3(kBlock), 0, s, heis, out);
    return hipGetLastError();
}

}  // namespace smc
