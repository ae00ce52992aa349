// Half-sweeps of any Ising / +-J EA batch with edges of at least 16, in place
// on row-major int8 spins (Eq. 2 on the square or cubic lattice): the general
// path beside the kernels that need an edge of a certain form.
//
// One thread owns 16 consecutive sites i0 = 16 g .. i0 + 15 of a replica.
// They are eight pairs (2h, 2h + 1) and each pair holds one site of either
// colour, so the piece's colour-c sites are the in-colour indices 8 g .. 8 g + 7
// and their 16-bit heads are the eight halves of one Philox block (g, t, r,
// 2*HEAD + c).  With an edge that is no multiple of 16 a piece may hold the end
// of one row and the start of the next.  A row holds at least 16 sites, so there
// is at most one such border in a piece, and it lies between two pairs: pairs
// below it belong to the first row, the others to the second.  What differs
// between the two rows (the parity of the own sites, wrapped neighbours) is
// merged with byte masks.
//
// Bound: launches and VALU.  Per eight updates one Philox block, 2d + 1 piece
// loads and byte-parallel counting, where a thread per site draws a block and
// computes 64-bit indices per update.
// 512^2 Ising, per half-sweep: 9.4 -> 4.2 us; 64 x 200^2 EA: 23 -> 7.5 us;
// 4 x 100^3 Ising: 96 -> 18 us.
#include "internal.hpp"
#include "rows.hpp"
#include "segment3d.hpp"

namespace smc {
namespace {

using namespace seg3d;

constexpr int kThreads = 256;

// Eight bytes, one per pair of the piece.
typedef uint64_t b8;
__device__ __forceinline__ b8 to_b8(uint2 v) { return ((uint64_t)v.y << 32) | v.x; }
__device__ __forceinline__ uint2 to_u2(b8 v) { return make_uint2((uint32_t)v, (uint32_t)(v >> 32)); }
__device__ __forceinline__ b8 merge(b8 m, b8 one, b8 zero) { return (one & m) | (zero & ~m); }
__device__ __forceinline__ b8 even8(const uint4 &w) { return to_b8(half_of(w, 0x06040200u)); }
__device__ __forceinline__ b8 odd8(const uint4 &w) { return to_b8(half_of(w, 0x07050301u)); }
// Mask of the pairs k .. 7 (0 <= k <= 8).
__device__ __forceinline__ b8 from_pair(uint32_t k) { return k >= 8 ? 0ull : ~0ull << (8 * k); }
__device__ __forceinline__ b8 put_byte(b8 v, uint32_t k, uint32_t byte) {
    const b8 m = 0xFFull << (8 * k);
    return (v & ~m) | ((b8)byte << (8 * k));
}

template <int DIM, bool EA>
__global__ __launch_bounds__(kThreads) void k_half_sweep_pieces(SweepArgs a, int c, int bpr, uint32_t one2) {
    __shared__ long long red[kThreads / 64];
    const int r = blockIdx.x / bpr;
    const smc_inst g = replica_geom(a.b, r);
    const int L = g.L;
    const int64_t LL = L, P = DIM == 3 ? LL * LL : LL, N = P * LL;  // P: sites per plane (3D) or row (2D)
    const uint32_t piece = (uint32_t)(blockIdx.x % bpr) * kThreads + threadIdx.x;
    const int64_t i0 = (int64_t)piece * 16;
    const int row = a.row_of_rep ? a.row_of_rep[r] : r;
    long long dE = 0;
    if (i0 < N && row >= 0) {
        int8_t *S = (int8_t *)a.spins + g.spin_off;
        const int8_t *J = EA ? a.coup + g.coup_off : nullptr;
        const int n = (int)min((int64_t)16, N - i0);  // sites of the piece (a multiple of 4)
        // first row of the piece, the row after it, and the first pair of the latter
        const uint32_t q = (uint32_t)i0 / (uint32_t)L;
        const int x0 = (int)((uint32_t)i0 - q * (uint32_t)L), left = L - x0;
        const uint32_t b = left >= 16 ? 8u : (uint32_t)left >> 1;
        const int z1 = DIM == 3 ? (int)(q / (uint32_t)L) : (int)q, y1 = DIM == 3 ? (int)(q - (uint32_t)z1 * L) : 0;
        int y2 = y1, z2 = z1;
        if (b < 8) {
            y2 = DIM == 3 ? (y1 == L - 1 ? 0 : y1 + 1) : 0;
            z2 = DIM == 3 ? (y1 == L - 1 ? z1 + 1 : z1) : z1 + 1;
        }
        const bool A1 = (((y1 + z1) & 1) ^ c) != 0, A2 = (((y2 + z2) & 1) ^ c) != 0;  // own sites odd in x
        const b8 second = from_pair(b);
        const b8 odd_own = (A1 ? ~second : 0ull) | (A2 ? second : 0ull);

        const uint4 w = load16(S, i0, N);
        const b8 E = even8(w), O = odd8(w);
        const b8 own = merge(odd_own, O, E), oth = merge(odd_own, E, O);
        // x neighbours in the next pair (own sites odd) or the one before (even)
        const uint32_t eL = (uint8_t)S[x0 == 0 ? i0 + L - 1 : i0 - 1];
        const uint32_t eR = (uint8_t)S[left == 16 ? i0 + 16 - L : i0 + 16 < N ? i0 + 16 : i0];
        b8 up = (O << 8) | eL, down = (E >> 8) | ((b8)eR << 56);
        const int64_t s2 = i0 + left, e2 = s2 + L - 1;  // ends of the second row
        const bool border = left < 16 && n > left;      // the piece holds sites of two rows
        if (left < 16) down = put_byte(down, b - 1, (uint8_t)S[s2 - L]);
        if (border) up = put_byte(up, b, (uint8_t)S[e2]);
        const b8 sh = merge(odd_own, down, up);

        // the neighbour sites (or their bonds) at offset d1 for the first row, d2 for the second
        auto beside = [&](const int8_t *p, int64_t d1, int64_t d2) {
            const uint4 v = load16(p, i0 + d1, N);
            b8 s = merge(odd_own, odd8(v), even8(v));
            if (border && d2 != d1) {
                const uint4 v2 = load16(p, i0 + d2, N);
                s = merge(second, merge(odd_own, odd8(v2), even8(v2)), s);
            }
            return s;
        };
        const int64_t zp1 = z1 == L - 1 ? P - N : P, zp2 = z2 == L - 1 ? P - N : P;
        const int64_t zm1 = z1 == 0 ? N - P : -P, zm2 = z2 == 0 ? N - P : -P;
        const int64_t yp1 = y1 == L - 1 ? LL - P : LL, yp2 = y2 == L - 1 ? LL - P : LL;
        const int64_t ym1 = y1 == 0 ? P - LL : -LL, ym2 = y2 == 0 ? P - LL : -LL;
        uint32_t n0 = 0, n1 = 0;  // twice the unsatisfied bonds of each own site
        auto count = [&](b8 nb, b8 bond) {
            const uint2 s = to_u2(own ^ bond), v = to_u2(nb);
            n0 += unsat(s.x, v.x, 0x02020202u);
            n1 += unsat(s.y, v.y, 0x02020202u);
        };
        if constexpr (EA) {
            const uint4 jw = load16(J, i0, N);
            const b8 jE = even8(jw), jO = odd8(jw);
            b8 jup = (jO << 8) | (uint8_t)J[x0 == 0 ? i0 + L - 1 : i0 - 1];
            if (border) jup = put_byte(jup, b, (uint8_t)J[e2]);
            count(oth, jE);
            count(sh, merge(odd_own, jO, jup));
            const int8_t *Jz = J + (DIM - 1) * N;
            count(beside(S, zp1, zp2), beside(Jz, 0, 0));
            count(beside(S, zm1, zm2), beside(Jz, zm1, zm2));
            if constexpr (DIM == 3) {
                count(beside(S, yp1, yp2), beside(J + N, 0, 0));
                count(beside(S, ym1, ym2), beside(J + N, ym1, ym2));
            }
        } else {
            count(oth, 0ull);
            count(sh, 0ull);
            count(beside(S, zp1, zp2), 0ull);
            count(beside(S, zm1, zm2), 0ull);
            if constexpr (DIM == 3) {
                count(beside(S, yp1, yp2), 0ull);
                count(beside(S, ym1, ym2), 0ull);
            }
        }

        // Table by the count of unsatisfied bonds: Delta E = 4 (DIM - count).
        // In 2D the entries move up by one: count 2 reads a threshold of 2^32.
        ThrRow th = a.thr[row];
        if constexpr (DIM == 2) {
            th.m[3] = th.m[2];
            th.m[2] = th.m[1];
            th.m[1] = make_uint2(65536u, 0u);
        }
        const Lut3 K = lut_of(th);
        const uint32_t rr = (uint32_t)r >> a.rng_shift;
        const uint4 rnd = philox4x32_10(make_uint4(piece, a.t, rr, 2 * kTagHead + c), a.key);
        RowOut o;
        o.n0 = n0 >> 1;
        o.n1 = n1 >> 1;
        uint32_t eq = 0xFFFFFFFFu;
        o.F0 = decide4(o.n0, rnd.x, rnd.y, K, one2, eq);
        o.F1 = decide4(o.n1, rnd.z, rnd.w, K, one2, eq);
        if (__builtin_expect(__any(has_tie(eq)), 0))
            exact_decisions(o, rnd, th, K, piece * 8u, (uint32_t)c, a.t, rr, a.key, has_tie(eq));
        const uint2 in = to_u2(~from_pair((uint32_t)n >> 1));  // pairs inside the replica
        o.F0 &= in.x;
        o.F1 &= in.y;
        if (o.F0 | o.F1) {
            const b8 flip = to_b8(make_uint2(bytes_fe(o.F0), bytes_fe(o.F1)));
            const uint2 fo = to_u2(flip & odd_own), fe = to_u2(flip & ~odd_own);
            const uint4 out = make_uint4(w.x ^ perm(fo.x, fe.x, 0x05010400u), w.y ^ perm(fo.x, fe.x, 0x07030602u),
                                         w.z ^ perm(fo.y, fe.y, 0x05010400u), w.w ^ perm(fo.y, fe.y, 0x07030602u));
            if (n == 16) {
                __builtin_memcpy(S + i0, &out, 16);
            } else {
                __builtin_memcpy(S + i0, &out.x, 4);
                if (n > 4) __builtin_memcpy(S + i0 + 4, &out.y, 4);
                if (n > 8) __builtin_memcpy(S + i0 + 8, &out.z, 4);
            }
            // flip_energy counts 12 - 4 n per flip; in 2D it is 8 - 4 n
            dE = flip_energy(o);
            if constexpr (DIM == 2) dE -= 4 * (__popc(o.F0) + __popc(o.F1));
        }
    }
    if (a.dE) {
#pragma unroll
        for (int k = 32; k > 0; k >>= 1) dE += __shfl_xor(dE, k, 64);
        if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = dE;
        __syncthreads();
        if (threadIdx.x == 0) {
            const long long tot = red[0] + red[1] + red[2] + red[3];
            if (tot != 0) atomicAdd((unsigned long long *)&a.dE[r], (unsigned long long)tot);
        }
    }
}

}  // namespace

hipError_t launch_half_sweep_pieces(const SweepArgs &a, int c, hipStream_t s) {
    const int64_t N = a.b.dim == 3 ? (int64_t)a.max_L * a.max_L * a.max_L : (int64_t)a.max_L * a.max_L;
    const int bpr = (int)((N + 16 * kThreads - 1) / (16 * kThreads));
    const int64_t blocks = (int64_t)bpr * a.b.n_rep;
    if (const char *why = launch_config_error((uint64_t)blocks, kThreads, 0))
        return reject_launch("k_half_sweep_pieces", (uint64_t)blocks, kThreads, 0, why);
    const dim3 grid((unsigned)blocks);
    const uint32_t one2 = 0x00010001u;
    if (a.b.dim == 3) {
        if (a.coup)
            SMC_LAUNCH((k_half_sweep_pieces<3, true>), grid, dim3(kThreads), 0, s, a, c, bpr, one2);
        else
            SMC_LAUNCH((k_half_sweep_pieces<3, false>), grid, dim3(kThreads), 0, s, a, c, bpr, one2);
    } else {
        if (a.coup)
            SMC_LAUNCH((k_half_sweep_pieces<2, true>), grid, dim3(kThreads), 0, s, a, c, bpr, one2);
        else
            SMC_LAUNCH((k_half_sweep_pieces<2, false>), grid, dim3(kThreads), 0, s, a, c, bpr, one2);
    }
    return hipGetLastError();
}

}  // namespace smc
