// ldl_blk.h -- the greedy block system of Algorithm 1, (G + lambda I) y = r_I
// for a greedy set of at most 64 rows, solved on one wave by an LDL^T
// factorisation on 16 x 16 tiles: each diagonal tile is eliminated in
// registers, everything between tiles is FP64 MFMA on registers.  Internal to
// the library; used by the greedy kernels of k_common.hip and k_fwd.hip.
//
// What bounds it: one wave's instruction issue.  A dependent FP64 FMA issues
// every 4.7 cycles, a hardware reciprocal takes 16, an LDS round trip 64, and
// v_mfma_f64_16x16x4f64 occupies the wave's FP64 unit for 64 (it does not
// overlap the wave's other FP64 instructions).  So a pivot step must be few
// instructions with no LDS in its chain: row k of the tile reaches the other
// rows inside the FMA itself (v_fmac_f64 with its first operand broadcast
// from lane k of every 16 lanes, DPP row_newbcast), and the products that link
// the tiles take their operands as the MFMA results leave them.  A 64-row
// system takes 6.5 us (13.5 us in the 16-column panel form that published
// each column through LDS), a 32-row one 2.4 us (5.5 us).
#pragma once

#include <utility>

#include "rorbk_device.h"

namespace rorbk {

constexpr int LB_RS = 65;             // row stride of the work matrix S (64 x 65 doubles)
constexpr int LB_TS = 18;             // row stride of a 16 x 16 tile kept in LDS
constexpr int LB_TILE = 16 * LB_TS;
constexpr int LB_LEN = 64 * LB_RS;    // doubles of S

// Entry f of the packed lower triangle (row-major, j <= i) of the padded
// system written into S: the Gram value g (plus lambda on the diagonal) for
// rows below K, the identity from row K on.  Every f < 64 * 65 / 2 is written
// once by whichever thread holds it, so the workgroup fills S in parallel.
__device__ __forceinline__ void lb_put(double *S, int f, double g, int K, double lambda) {
    // f < 2080: the hardware square root is within a step of the row
    int i = (int)((__builtin_amdgcn_sqrtf(8.0f * (float)f + 1.0f) - 1.0f) * 0.5f);
    i -= (i * (i + 1) / 2 > f) ? 1 : 0;
    i += ((i + 1) * (i + 2) / 2 <= f) ? 1 : 0;
    const int j = f - i * (i + 1) / 2;
    S[i * LB_RS + j] = (i < K) ? ((i == j) ? g + lambda : g) : ((i == j) ? 1.0 : 0.0);
}

// Broadcast of lane J of each 16-lane row to the whole row (DPP row_newbcast).
template <int J>
__device__ __forceinline__ double lb_rowbc(double v) {
    return __builtin_amdgcn_mov_dpp(v, 0x150 + J, 0xf, 0xf, false);
}

// Sum over the four 16-lane rows of the wave, in every row: the halves, then
// the row pairs, exchanged by v_permlane32_swap and v_permlane16_swap (with
// both operands equal, the two results are the two rows to add).
__device__ __forceinline__ double lb_rowsum(double v) {
    uint64_t u = (uint64_t)__double_as_longlong(v);
    const auto l = __builtin_amdgcn_permlane32_swap((uint32_t)u, (uint32_t)u, false, false);
    const auto h = __builtin_amdgcn_permlane32_swap((uint32_t)(u >> 32), (uint32_t)(u >> 32),
                                                    false, false);
    v = __longlong_as_double((long long)(((uint64_t)h[0] << 32) | l[0])) +
        __longlong_as_double((long long)(((uint64_t)h[1] << 32) | l[1]));
    u = (uint64_t)__double_as_longlong(v);
    const auto l2 = __builtin_amdgcn_permlane16_swap((uint32_t)u, (uint32_t)u, false, false);
    const auto h2 = __builtin_amdgcn_permlane16_swap((uint32_t)(u >> 32), (uint32_t)(u >> 32),
                                                     false, false);
    return __longlong_as_double((long long)(((uint64_t)h2[0] << 32) | l2[0])) +
           __longlong_as_double((long long)(((uint64_t)h2[1] << 32) | l2[1]));
}

// Elimination of a 16 x 16 tile A = L D L^T.  Lane li of every 16-lane row
// holds row li of the whole symmetric tile, a[0..15]; the four 16-lane rows
// (lk = 0..3) hold the same a, the columns 4 q + lk (q = 0..3) of the row of
// E = L^{-1} (the identity to begin with) in e[q], and a share of the
// right-hand side in z (the shares add up; every step is linear in z).
//
// Pivot step K (the only VALU work between two pivots): d = a_KK in every
// lane, g its hardware reciprocal; r = 1 / d by g (1 + e + e^2), e = 1 - d g
// (about an ulp; three FMAs); c = -a_iK r for the rows below K, else 0; then
// column K + 1 takes its update first and the next pivot is broadcast and
// sent to the reciprocal unit, whose latency the other updates cover:
// a_ij += c a_Kj for j > K, E_i += c E_K, z_i += c z_K.
//
// The step is one block of instructions because no compiler builtin forms
// v_fmac_f64 with a DPP operand.  A DPP read needs two instructions between
// it and the VALU write of the register it reads: the four leading FMAs stand
// between anything before the block and its first DPP read, two updates
// stand between the one of column K + 1 and its broadcast, and the column
// order keeps every other register's write at least five instructions from
// its read in the next step.  The reciprocal's result is first read in the next step,
// at least one update later.  The last block ends with two wait states,
// after which any instruction may read e.
#define LB_F(r, k)                                                                  \
    "v_fmac_f64_dpp %" #r ", %" #r ", %[c] row_newbcast:" #k " row_mask:0xf bank_mask:0xf\n\t"
#define LB_CHAIN(k, n, f1, f2, f3)                                                  \
    "v_fma_f64 %[c], -%[d], %[g], 1.0\n\t"                                          \
    "v_fma_f64 %[c], %[c], %[c], %[c]\n\t"                                          \
    "v_fma_f64 %[r], %[g], %[c], %[g]\n\t"                                          \
    "v_mul_f64 %[c], -%[m], %[r]\n\t" LB_F(n, k) LB_F(f1, k) LB_F(f2, k)            \
    "v_mov_b64_dpp %[d], %" #n " row_newbcast:" #n " row_mask:0xf bank_mask:0xf\n\t" \
    LB_F(f3, k) "v_rcp_f64 %[g], %[d]\n\t"
#define LB_E(k) LB_F(16, k) LB_F(17, k) LB_F(18, k) LB_F(19, k) LB_F(20, k)
#define LB_15(k) LB_F(15, k) LB_E(k)
#define LB_14(k) LB_F(14, k) LB_15(k)
#define LB_13(k) LB_F(13, k) LB_14(k)
#define LB_12(k) LB_F(12, k) LB_13(k)
#define LB_11(k) LB_F(11, k) LB_12(k)
#define LB_10(k) LB_F(10, k) LB_11(k)
#define LB_9(k) LB_F(9, k) LB_10(k)
#define LB_8(k) LB_F(8, k) LB_9(k)
#define LB_7(k) LB_F(7, k) LB_8(k)
#define LB_6(k) LB_F(6, k) LB_7(k)
#define LB_5(k) LB_F(5, k) LB_6(k)
#define LB_STEP(k, TEXT)                                                                          \
    if constexpr (K == k)                                                                         \
        asm(TEXT                                                                                  \
            : "+v"(a[0]), "+v"(a[1]), "+v"(a[2]), "+v"(a[3]), "+v"(a[4]), "+v"(a[5]), "+v"(a[6]), \
              "+v"(a[7]), "+v"(a[8]), "+v"(a[9]), "+v"(a[10]), "+v"(a[11]), "+v"(a[12]),          \
              "+v"(a[13]), "+v"(a[14]), "+v"(a[15]), "+v"(e[0]), "+v"(e[1]), "+v"(e[2]),          \
              "+v"(e[3]), "+v"(z), [d] "+v"(d), [g] "+v"(g), [c] "=&v"(c), [r] "=&v"(r)           \
            : [m] "v"(m));

template <int K>
__device__ __forceinline__ void lb_pivot(double (&a)[16], double (&e)[4], double &z, double &d,
                                         double &g, double *rd, int li) {
    double c, r;
    const double m = (li > K) ? a[K] : 0.0;
    LB_STEP(0, LB_CHAIN(0, 1, 2, 3, 4) LB_5(0))
    LB_STEP(1, LB_CHAIN(1, 2, 3, 4, 5) LB_6(1))
    LB_STEP(2, LB_CHAIN(2, 3, 4, 5, 6) LB_7(2))
    LB_STEP(3, LB_CHAIN(3, 4, 5, 6, 7) LB_8(3))
    LB_STEP(4, LB_CHAIN(4, 5, 6, 7, 8) LB_9(4))
    LB_STEP(5, LB_CHAIN(5, 6, 7, 8, 9) LB_10(5))
    LB_STEP(6, LB_CHAIN(6, 7, 8, 9, 10) LB_11(6))
    LB_STEP(7, LB_CHAIN(7, 8, 9, 10, 11) LB_12(7))
    LB_STEP(8, LB_CHAIN(8, 9, 10, 11, 12) LB_13(8))
    LB_STEP(9, LB_CHAIN(9, 10, 11, 12, 13) LB_14(9))
    LB_STEP(10, LB_CHAIN(10, 11, 12, 13, 14) LB_15(10))
    LB_STEP(11, LB_CHAIN(11, 12, 13, 14, 15) LB_E(11))
    LB_STEP(12, LB_CHAIN(12, 13, 14, 15, 16) LB_F(17, 12) LB_F(18, 12) LB_F(19, 12) LB_F(20, 12))
    LB_STEP(13, LB_CHAIN(13, 14, 15, 16, 17) LB_F(18, 13) LB_F(19, 13) LB_F(20, 13))
    LB_STEP(14, LB_CHAIN(14, 15, 16, 17, 18) LB_F(19, 14) LB_F(20, 14) "s_nop 1")
    if constexpr (K == 15) {
        const double e0 = __builtin_fma(-d, g, 1.0);
        r = __builtin_fma(g, __builtin_fma(e0, e0, e0), g);
    }
    rd[K] = r;
}

// The sixteen pivot steps; the reciprocal pivots go to rd[0..15] (LDS).
template <int... Ks>
__device__ __forceinline__ void lb_tile(std::integer_sequence<int, Ks...>, double (&a)[16],
                                        double (&e)[4], double &z, double *rd, int li) {
    // the row masks are compared again for every tile (sixteen lane masks kept
    // across the tiles would not fit the scalar registers)
    asm("" : "+v"(li));
    double d = lb_rowbc<0>(a[0]);
    double g = __builtin_amdgcn_rcp(d);
    (lb_pivot<Ks>(a, e, z, d, g, rd, li), ...);
}

// acc + sum_j l[j] y_j, y_j in lane j of each 16-lane row, j in order.  The
// wait states at both ends keep the DPP reads clear of what stands before and
// after the block.
#define LB_D(j, l) \
    "v_fmac_f64_dpp %0, %1, %" #l " row_newbcast:" #j " row_mask:0xf bank_mask:0xf\n\t"
__device__ __forceinline__ double lb_dot(double acc, const double (&l)[16], double y) {
    asm("s_nop 1\n\t" LB_D(0, 2) LB_D(1, 3) LB_D(2, 4) LB_D(3, 5) LB_D(4, 6) LB_D(5, 7)
        LB_D(6, 8) LB_D(7, 9) LB_D(8, 10) LB_D(9, 11) LB_D(10, 12) LB_D(11, 13) LB_D(12, 14)
        LB_D(13, 15) LB_D(14, 16) LB_D(15, 17) "s_nop 1"
        : "+v"(acc)
        : "v"(y), "v"(l[0]), "v"(l[1]), "v"(l[2]), "v"(l[3]), "v"(l[4]), "v"(l[5]), "v"(l[6]),
          "v"(l[7]), "v"(l[8]), "v"(l[9]), "v"(l[10]), "v"(l[11]), "v"(l[12]), "v"(l[13]),
          "v"(l[14]), "v"(l[15]));
    return acc;
}
#undef LB_D
#undef LB_STEP
#undef LB_5
#undef LB_6
#undef LB_7
#undef LB_8
#undef LB_9
#undef LB_10
#undef LB_11
#undef LB_12
#undef LB_13
#undef LB_14
#undef LB_15
#undef LB_E
#undef LB_CHAIN
#undef LB_F

// LDS scratch of the factorisation, laid over S (whose tiles are in registers
// by then): one tile to turn a diagonal tile into rows, E^T of every diagonal
// tile, the tiles of -L below the diagonal, the reciprocal pivots, u = E z.
template <int NP>
struct LbScratch {
    static constexpr int E = LB_TILE;
    static constexpr int L = E + NP * LB_TILE;
    static constexpr int R = L + NP * (NP - 1) / 2 * LB_TILE;
    static constexpr int U = R + 16 * NP;
    static_assert(U + 16 * NP <= LB_LEN, "the scratch fits S");
    // the tile of block row J > p, block column p
    static constexpr int tile(int p, int J) {
        return L + (p * (2 * NP - p - 1) / 2 + J - p - 1) * LB_TILE;
    }
};

// Single-wave solve of the padded (16 NP)^2 system held in S (the 64 x 65 work
// matrix, lower triangle filled by lb_put: the Gram with lambda on the
// diagonal, the identity from row K on; overwritten), right-hand side in zv
// (entries past K zero; overwritten by y).  The identity beyond K leaves the
// leading K x K factor and solution unchanged.
//
// The upper tiles T_IJ (I <= J) live in registers as MFMA results do: entry
// (lk + 4 r, li) in register r.  After the elimination of diagonal tile p,
// W_J = E_p T_pJ (= D L_Jp^T) takes e as its first operand and T_pJ as its
// second without moving either, and T_IJ -= (D^{-1} W_I)^T W_J takes the two
// results the same way.  The right-hand side follows: u_p = E_p z_p from the
// elimination, z_J -= L_Jp u_p; and back: y_p = E_p^T (D^{-1} u_p -
// sum_J L_Jp^T y_J) with the tiles' rows read from LDS.  No block barrier
// inside: the workgroup's other waves may be elsewhere.  Returns false if a
// pivot is not positive.
template <int NP>
__device__ __forceinline__ bool ldl_blk(double *S, double *zv) {
    using X = LbScratch<NP>;
    const int lane = threadIdx.x & 63, li = lane & 15, lk = lane >> 4;
    dvec4 T[NP][NP];
    double z[NP];   // shares of the 16-lane rows
#pragma unroll
    for (int I = 0; I < NP; ++I) {
        z[I] = (lk == 0) ? zv[16 * I + li] : 0.0;
#pragma unroll
        for (int J = I; J < NP; ++J)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int i = 16 * I + lk + 4 * r, j = 16 * J + li;
                T[I][J][r] = (J > I || i < j) ? S[j * LB_RS + i] : S[i * LB_RS + j];
            }
    }
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int p = 0; p < NP; ++p) {
        double a[16], e[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) S[(lk + 4 * r) * LB_TS + li] = T[p][p][r];
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int j = 0; j < 16; ++j) a[j] = S[li * LB_TS + j];
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int q = 0; q < 4; ++q) e[q] = (li == 4 * q + lk) ? 1.0 : 0.0;
        lb_tile(std::make_integer_sequence<int, 16>{}, a, e, z[p], S + X::R + 16 * p, li);
        z[p] = lb_rowsum(z[p]);
        if (lk == 0) S[X::U + 16 * p + li] = z[p];
#pragma unroll
        for (int q = 0; q < 4; ++q) S[X::E + p * LB_TILE + (4 * q + lk) * LB_TS + li] = e[q];
        __builtin_amdgcn_wave_barrier();
        double rd[4], u[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            rd[q] = S[X::R + 16 * p + 4 * q + lk];
            u[q] = S[X::U + 16 * p + 4 * q + lk];
        }
        dvec4 W[NP], V[NP];   // W_J and -D^{-1} W_J
#pragma unroll
        for (int J = p + 1; J < NP; ++J) {
            W[J] = dvec4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int q = 0; q < 4; ++q)
                W[J] = __builtin_amdgcn_mfma_f64_16x16x4f64(e[q], T[p][J][q], W[J], 0, 0, 0);
        }
#pragma unroll
        for (int J = p + 1; J < NP; ++J)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                V[J][q] = -W[J][q] * rd[q];
                S[X::tile(p, J) + (lk + 4 * q) * LB_TS + li] = V[J][q];
                z[J] = __builtin_fma(V[J][q], u[q], z[J]);
            }
#pragma unroll
        for (int I = p + 1; I < NP; ++I)
#pragma unroll
            for (int J = I; J < NP; ++J)
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    T[I][J] = __builtin_amdgcn_mfma_f64_16x16x4f64(V[I][q], W[J][q], T[I][J], 0, 0, 0);
    }
    __builtin_amdgcn_wave_barrier();
    double y[NP], rv[NP];
    bool ok = true;
#pragma unroll
    for (int p = 0; p < NP; ++p) {
        rv[p] = S[X::R + 16 * p + li];
        ok = ok && rv[p] > 0.0 && rv[p] < __builtin_inf();
    }
    if (__ballot(ok) != ~0ull) return false;
#pragma unroll
    for (int p = NP - 1; p >= 0; --p) {
        double t = z[p] * rv[p];
#pragma unroll
        for (int J = p + 1; J < NP; ++J) {
            double l[16];
#pragma unroll
            for (int j = 0; j < 16; ++j) l[j] = S[X::tile(p, J) + li * LB_TS + j];
            t = lb_dot(t, l, y[J]);
        }
        double l[16];
#pragma unroll
        for (int j = 0; j < 16; ++j) l[j] = S[X::E + p * LB_TILE + li * LB_TS + j];
        y[p] = lb_dot(0.0, l, t);
        if (lk == 0) zv[16 * p + li] = y[p];
    }
    __builtin_amdgcn_wave_barrier();
    return true;
}

// K <= 64 on one wave: the smallest padded size that holds the system.
__device__ __forceinline__ bool ldl_blk64(double *S, double *z, int K) {
    if (K <= 16) return ldl_blk<1>(S, z);
    if (K <= 32) return ldl_blk<2>(S, z);
    if (K <= 48) return ldl_blk<3>(S, z);
    return ldl_blk<4>(S, z);
}

}  // namespace rorbk
