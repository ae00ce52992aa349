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
// 512^2 Ising, per half-sweep: 9.4 -> 3.8 us; 64 x 200^2 EA: 23 -> 6.5 us;
// 4 x 100^3 Ising: 96 -> 8 us.
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

// I: int where a replica has at most 2^30 sites, else int64_t.
template <int DIM, bool EA, typename I>
__global__ __launch_bounds__(kThreads) void k_half_sweep_pieces(SweepArgs a, int c, int bpr, uint32_t one2) {
    __shared__ int red[kThreads / 64];
    constexpr int kDir = DIM == 3 ? 4 : 2;  // neighbours outside the row
    const int r = blockIdx.x / bpr;
    const smc_inst g = replica_geom(a.b, r);
    const int L = g.L;
    const I LL = L, P = DIM == 3 ? LL * LL : LL, N = P * LL;  // P: sites per plane (3D) or row (2D)
    const uint32_t piece = (uint32_t)(blockIdx.x % bpr) * kThreads + threadIdx.x;
    const int row = a.row_of_rep ? a.row_of_rep[r] : r;
    int dE = 0;
    if ((int64_t)piece * 16 < (int64_t)N && row >= 0) {
        const I i0 = (I)piece * 16;
        int8_t *S = (int8_t *)a.spins + g.spin_off;
        const int8_t *J = EA ? a.coup + g.coup_off : nullptr;
        const int n = (int)min((I)16, N - i0);  // sites of the piece (a multiple of 4)
        // first row of the piece, the row after it, and the first pair of the latter
        const uint32_t q = (uint32_t)i0 / (uint32_t)L;
        const int x0 = (int)((uint32_t)i0 - q * (uint32_t)L), left = L - x0;
        const uint32_t b = left >= 16 ? 8u : (uint32_t)left >> 1;
        const bool border = left < 16 && n > left;  // the piece holds sites of two rows
        const int z1 = DIM == 3 ? (int)(q / (uint32_t)L) : (int)q, y1 = DIM == 3 ? (int)(q - (uint32_t)z1 * L) : 0;
        int y2 = y1, z2 = z1;
        if (left < 16) {
            y2 = DIM == 3 ? (y1 == L - 1 ? 0 : y1 + 1) : 0;
            z2 = DIM == 3 ? (y1 == L - 1 ? z1 + 1 : z1) : z1 + 1;
        }
        // offsets of the neighbours for the sites of the first and of the second row
        auto off = [&](int k, int y, int z) -> I {
            if (k == 0) return z == L - 1 ? P - N : P;
            if (k == 1) return z == 0 ? N - P : -P;
            if (k == 2) return y == L - 1 ? LL - P : LL;
            return y == 0 ? P - LL : -LL;
        };
        I d1[kDir], d2[kDir];
        bool over = i0 > N - 16, split = false;  // a load beyond the array; two offsets in one piece
#pragma unroll
        for (int k = 0; k < kDir; ++k) {
            d1[k] = off(k, y1, z1);
            d2[k] = off(k, y2, z2);
            over |= i0 + d1[k] < 0 || i0 + d1[k] > N - 16;
            split |= d1[k] != d2[k];
        }
        split &= border;

        // every load of the ordinary case
        uint4 w = load_inside(S, i0, N), nb[kDir], jx, jf[DIM - 1], jb[kDir / 2];
#pragma unroll
        for (int k = 0; k < kDir; ++k) nb[k] = load_inside(S, i0 + d1[k], N);
        const I iL = x0 == 0 ? i0 + L - 1 : i0 - 1, s2 = i0 + left, e2 = s2 + L - 1;
        uint32_t eL = (uint8_t)S[iL], eR = (uint8_t)S[left == 16 ? i0 + 16 - L : i0 + 16 < N ? i0 + 16 : i0];
        uint32_t wR = 0, wL = 0, jeL = 0, jwL = 0;
        if constexpr (EA) {
            jx = load_inside(J, i0, N);
            jeL = (uint8_t)J[iL];
#pragma unroll
            for (int k = 0; k < kDir / 2; ++k) {
                const int8_t *Jm = J + (int64_t)(k == 0 ? DIM - 1 : 1) * N;
                jf[k] = load_inside(Jm, i0, N);                // bonds forward
                jb[k] = load_inside(Jm, i0 + d1[2 * k + 1], N);  // bonds of the neighbours behind
            }
        }
        if (left < 16) {
            wR = (uint8_t)S[s2 - L];  // the first row's periodic end
            if (border) {
                wL = (uint8_t)S[e2];  // the second row's periodic start
                if constexpr (EA) jwL = (uint8_t)J[e2];
            }
        }
        if (__builtin_expect(over, 0)) {
            into_place(w, i0, N);
#pragma unroll
            for (int k = 0; k < kDir; ++k) into_place(nb[k], i0 + d1[k], N);
            if constexpr (EA) {
                into_place(jx, i0, N);
#pragma unroll
                for (int k = 0; k < kDir / 2; ++k) {
                    into_place(jf[k], i0, N);
                    into_place(jb[k], i0 + d1[2 * k + 1], N);
                }
            }
        }
        if (split) {
            // bytes 2b .. 15 of the neighbours come from the second row's offset
            const uint4 ones = make_uint4(~0u, ~0u, ~0u, ~0u), m = bytes_up(ones, 2 * b);
            auto second_from = [&](uint4 &v, const int8_t *p, I i) {
                const uint4 u = load16(p, (int64_t)i, (int64_t)N);
                v = make_uint4((u.x & m.x) | (v.x & ~m.x), (u.y & m.y) | (v.y & ~m.y), (u.z & m.z) | (v.z & ~m.z),
                               (u.w & m.w) | (v.w & ~m.w));
            };
#pragma unroll
            for (int k = 0; k < kDir; ++k)
                if (d1[k] != d2[k]) {
                    second_from(nb[k], S, i0 + d2[k]);
                    if constexpr (EA)
                        if (k & 1) second_from(jb[k >> 1], J + (int64_t)(k == 1 ? DIM - 1 : 1) * N, i0 + d2[k]);
                }
        }

        const bool A1 = (((y1 + z1) & 1) ^ c) != 0, A2 = (((y2 + z2) & 1) ^ c) != 0;  // own sites odd in x
        const b8 second = from_pair(b);
        const b8 odd_own = (A1 ? ~second : 0ull) | (A2 ? second : 0ull);
        const b8 E = even8(w), O = odd8(w);
        const b8 own = merge(odd_own, O, E), oth = merge(odd_own, E, O);
        // x neighbours in the next pair (own sites odd) or the one before (even)
        b8 up = (O << 8) | eL, down = (E >> 8) | ((b8)eR << 56), jup = 0;
        if (left < 16) {
            down = put_byte(down, b - 1, wR);
            if (border) up = put_byte(up, b, wL);
        }
        uint32_t n0 = 0, n1 = 0;  // twice the unsatisfied bonds of each own site
        auto count = [&](b8 v8, b8 bond) {
            const uint2 s = to_u2(own ^ bond), v = to_u2(v8);
            n0 += unsat(s.x, v.x, 0x02020202u);
            n1 += unsat(s.y, v.y, 0x02020202u);
        };
        auto mine = [&](const uint4 &v) { return merge(odd_own, odd8(v), even8(v)); };
        if constexpr (EA) {
            const b8 jE = even8(jx), jO = odd8(jx);
            jup = (jO << 8) | jeL;
            if (border) jup = put_byte(jup, b, jwL);
            count(oth, jE);
            count(merge(odd_own, down, up), merge(odd_own, jO, jup));
#pragma unroll
            for (int k = 0; k < kDir / 2; ++k) {
                count(mine(nb[2 * k]), mine(jf[k]));
                count(mine(nb[2 * k + 1]), mine(jb[k]));
            }
        } else {
            count(oth, 0ull);
            count(merge(odd_own, down, up), 0ull);
#pragma unroll
            for (int k = 0; k < kDir; ++k) count(mine(nb[k]), 0ull);
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
            dE = (int)flip_energy(o);
            if constexpr (DIM == 2) dE -= 4 * (__popc(o.F0) + __popc(o.F1));
        }
    }
    if (tally_wanted(a.tally)) {
#pragma unroll
        for (int k = 32; k > 0; k >>= 1) dE += __shfl_xor(dE, k, 64);
        if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = dE;
        __syncthreads();
        if (threadIdx.x == 0) {
            const long long tot = (long long)red[0] + red[1] + red[2] + red[3];
            tally_put(a.tally, blockIdx.x, r, tot);
        }
    }
}

}  // namespace

int pieces_groups(const SweepArgs &a) {
    const int64_t N = a.b.dim == 3 ? (int64_t)a.max_L * a.max_L * a.max_L : (int64_t)a.max_L * a.max_L;
    return (int)((N + 16 * kThreads - 1) / (16 * kThreads));
}

hipError_t launch_half_sweep_pieces(const SweepArgs &a, int c, hipStream_t s) {
    const int64_t N = a.b.dim == 3 ? (int64_t)a.max_L * a.max_L * a.max_L : (int64_t)a.max_L * a.max_L;
    const int bpr = pieces_groups(a);
    const int64_t blocks = (int64_t)bpr * a.b.n_rep;
    if (const char *why = launch_config_error((uint64_t)blocks, kThreads, 0))
        return reject_launch("k_half_sweep_pieces", (uint64_t)blocks, kThreads, 0, why);
    const dim3 grid((unsigned)blocks);
    const uint32_t one2 = 0x00010001u;
    const bool ea = a.coup != nullptr;
    if (a.b.dim == 3) {
        if (ea)
            SMC_LAUNCH((k_half_sweep_pieces<3, true, int>), grid, dim3(kThreads), 0, s, a, c, bpr, one2);
        else
            SMC_LAUNCH((k_half_sweep_pieces<3, false, int>), grid, dim3(kThreads), 0, s, a, c, bpr, one2);
    } else if (N <= ((int64_t)1 << 30)) {
        if (ea)
            SMC_LAUNCH((k_half_sweep_pieces<2, true, int>), grid, dim3(kThreads), 0, s, a, c, bpr, one2);
        else
            SMC_LAUNCH((k_half_sweep_pieces<2, false, int>), grid, dim3(kThreads), 0, s, a, c, bpr, one2);
    } else {
        if (ea)
            SMC_LAUNCH((k_half_sweep_pieces<2, true, int64_t>), grid, dim3(kThreads), 0, s, a, c, bpr, one2);
        else
            SMC_LAUNCH((k_half_sweep_pieces<2, false, int64_t>), grid, dim3(kThreads), 0, s, a, c, bpr, one2);
    }
    return hipGetLastError();
}

}  // namespace smc
