// ldl_wg.h -- LDL^T of a symmetric positive definite system of up to 176 rows
// in one workgroup's LDS, for greedy sets of 65 to 161 rows (Algorithm 1's
// greedy step) and for the stored inverses of fixed blocks of at most 161 rows
// (Section 3.1).  Internal to the library.
//
// The matrix is kept as the upper 16 x 16 tiles T_pJ (p <= J) of its padded
// size 16 P in LDS, entry (r, c) of a tile at 16 r + (c xor r), so that rows and
// columns are both read without bank conflicts.  Tile row p: wave 0 eliminates the diagonal
// tile in registers (lb_tile, ldl_blk.h) and leaves E_p^T in its place; the
// waves form W_J = E_p T_pJ; then T_IJ -= W_I^T D_p^{-1} W_J on FP64 MFMA, wave
// 0 taking the next diagonal tile and going on to eliminate it while the
// others update the rest.  The sixteen terms of a product are summed by themselves
// and added to T_IJ once: with T_IJ as the accumulator each of the four MFMAs
// rounds at its size, which showed where rows nearly repeat and a pivot is a
// small difference (160 rows in pairs 1e-4 apart: x 1.5 to 1.7 times further from
// the exact one).  All operands are read as rows, the layout the MFMA
// results are written in, so nothing is transposed; only the backward pass
// reads columns.  What bounds it is the chain of eliminations, 1.9 us per tile
// row with its two barriers; the products fit beside it.
#pragma once

#include "ldl_blk.h"

namespace rorbk {

constexpr int WT = 256;                                    // doubles of a tile
constexpr int WL_MAXP = (MAXB + 15) / 16;                  // 11: blocks of 161 rows
constexpr int wl_tiles(int P) { return P * (P + 1) / 2; }
__device__ __forceinline__ int wl_at(int r, int c) { return r * 16 + (c ^ r); }
__device__ __forceinline__ int wl_tile(int P, int p, int J) {
    return (p * P - p * (p - 1) / 2 + J - p) * WT;
}

// The packed lower triangle (the sum of nch chunks of K (K + 1) / 2 doubles, in
// chunk order) into the tiles, lambda on the diagonal and the identity from
// row K on, by NW waves: a wave a row, its columns over the lanes, so that an
// entry costs a load and two or three address operations (the row from a
// packed index takes a square root: 2 us for 128 rows).  (i, j), j <= i, goes to
// (j, i) of the upper triangle, in a diagonal tile to both.
template <int P, int NW>
__device__ __forceinline__ void wl_load(double *T, const double *__restrict__ G, int nch, int K,
                                        double lambda) {
    constexpr int RW = (16 * P + NW - 1) / NW, JG = (16 * P + 63) / 64, RB = 4;
    const int lane = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int KP = K * (K + 1) / 2;
    int at[JG], jx[JG];   // of row j in tile row j / 16, tile column 0; j mod 16
#pragma unroll
    for (int g = 0; g < JG; ++g) {
        const int j = lane + 64 * g, t = j >> 4;
        at[g] = (t * P - t * (t - 1) / 2 - t) * WT + (j & 15) * 16;
        jx[g] = j & 15;
    }
#pragma unroll 1
    for (int r0 = 0; r0 < RW; r0 += RB) {
        double v[RB][JG];
#pragma unroll
        for (int r = 0; r < RB; ++r)
#pragma unroll
            for (int g = 0; g < JG; ++g) v[r][g] = 0.0;
        for (int c = 0; c < nch; ++c) {
            double w[RB][JG];
#pragma unroll
            for (int r = 0; r < RB; ++r) {
                const int i = wv + NW * (r0 + r), ii = i < K ? i : K - 1;   // scalar
                const double *gi = G + (int64_t)c * KP + ii * (ii + 1) / 2;
#pragma unroll
                for (int g = 0; g < JG; ++g) w[r][g] = gi[lane + 64 * g < ii ? lane + 64 * g : ii];
            }
#pragma unroll
            for (int r = 0; r < RB; ++r)
#pragma unroll
                for (int g = 0; g < JG; ++g) v[r][g] += w[r][g];
        }
#pragma unroll
        for (int r = 0; r < RB; ++r) {
            const int i = wv + NW * (r0 + r);
            if (i < 16 * P) {   // scalar
#pragma unroll
                for (int g = 0; g < JG; ++g) {
                    const int j = lane + 64 * g;
                    if (j <= i) {
                        const double x = (i < K) ? ((i == j) ? v[r][g] + lambda : v[r][g])
                                                 : ((i == j) ? 1.0 : 0.0);
                        T[at[g] + (i >> 4) * WT + ((i & 15) ^ jx[g])] = x;
                        if ((j >> 4) == (i >> 4))
                            T[wl_tile(P, j >> 4, j >> 4) + wl_at(i & 15, jx[g])] = x;
                    }
                }
            }
        }
    }
}

// Factorisation of the tiles by NW waves; rd (16 P doubles) takes the
// reciprocal pivots, and with RHS z (16 P doubles) is overwritten by
// L^{-1} z.  On return tile (p, p) holds E_p^T = L_pp^{-T} and tile (p, J) holds
// W_J = D_p L_Jp^T.  Starts and ends with a barrier; false (in every thread)
// if a pivot is not positive.
template <int P, int NW, bool RHS>
__device__ __forceinline__ bool wl_factor(double *T, double *rd, double *z) {
    const int lane = threadIdx.x & 63, li = lane & 15, lk = lane >> 4;
    const int wv = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    int at[4];   // entry (4 q + lk, li) of a tile
#pragma unroll
    for (int q = 0; q < 4; ++q) at[q] = wl_at(4 * q + lk, li);
    __syncthreads();
#pragma unroll 1
    for (int p = 0; p < P; ++p) {
        double *Tp = T + wl_tile(P, p, p);
        if (wv == 0) {
            double a[16], e[4];
#pragma unroll
            for (int j = 0; j < 16; ++j) a[j] = Tp[wl_at(j, li)];
#pragma unroll
            for (int q = 0; q < 4; ++q) e[q] = (li == 4 * q + lk) ? 1.0 : 0.0;
            double zz = RHS ? z[16 * p + li] : 0.0;
            lb_tile(std::make_integer_sequence<int, 16>{}, a, e, zz, rd + 16 * p, li);
            if (RHS && lk == 0) z[16 * p + li] = zz;
#pragma unroll
            for (int q = 0; q < 4; ++q) Tp[at[q]] = e[q];
        }
        __syncthreads();
        if (p + 1 == P) break;   // uniform
        double e[4], r[4], u[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            e[q] = Tp[at[q]];
            r[q] = rd[16 * p + 4 * q + lk];
            u[q] = RHS ? z[16 * p + 4 * q + lk] : 0.0;
        }
        for (int J = p + 1 + wv; J < P; J += NW) {
            double *t = Tp + (J - p) * WT;
            dvec4 w = {0.0, 0.0, 0.0, 0.0};
            double b[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) b[q] = t[at[q]];
#pragma unroll
            for (int q = 0; q < 4; ++q) w = __builtin_amdgcn_mfma_f64_16x16x4f64(e[q], b[q], w, 0, 0, 0);
#pragma unroll
            for (int q = 0; q < 4; ++q) t[at[q]] = w[q];
            if (RHS) {
                double s = 0.0;
#pragma unroll
                for (int q = 0; q < 4; ++q) s = __builtin_fma(-w[q] * r[q], u[q], s);
                s = lb_rowsum(s);
                if (lk == 0) z[16 * J + li] += s;
            }
        }
        __syncthreads();
        // the next diagonal tile on wave 0, the others dealt to the rest: with
        // more than four waves to those of the other three SIMDs (wave w runs
        // on SIMD w mod 4), whose MFMA does not hold up wave 0
        const int n = P - p - 1;
        constexpr bool APART = NW > 4;
        constexpr int NR = APART ? NW - (NW + 3) / 4 : NW - 1;
        if (APART && wv != 0 && (wv & 3) == 0) continue;
        int I = 0, J = (wv == 0) ? 0 : (APART ? wv - (wv >> 2) : wv);
        while (true) {
            while (I < n && J >= n) { ++I; J -= n - I; }   // tile (I, J) in row order
            if (I >= n) break;
            const double *wi = Tp + (I + 1) * WT, *wj = Tp + (J + 1) * WT;
            double *t = T + wl_tile(P, p + 1 + I, p + 1 + J);
            double av[4], bv[4], tv[4];
            dvec4 acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                av[q] = -wi[at[q]] * r[q];
                bv[q] = wj[at[q]];
                tv[q] = t[at[q]];
            }
#pragma unroll
            for (int q = 0; q < 4; ++q)
                acc = __builtin_amdgcn_mfma_f64_16x16x4f64(av[q], bv[q], acc, 0, 0, 0);
#pragma unroll
            for (int q = 0; q < 4; ++q) t[at[q]] = tv[q] + acc[q];
            if (wv == 0) break;
            J += NR;
        }
    }
    bool ok = true;
    for (int i = threadIdx.x; i < 16 * P; i += blockDim.x)
        ok = ok && rd[i] > 0.0 && rd[i] < __builtin_inf();
    return __syncthreads_and(ok ? 1 : 0) != 0;
}

// y = L^{-T} D^{-1} z after wl_factor with RHS, into z: from the last tile row,
// y_p = E_p^T w_p on wave 0, then w_I -= L_pI^T y_p for the rows above, wave 0
// taking the row that it needs next (so that one barrier a tile row is
// enough), the other waves the rest.  Ends with a barrier.
template <int P, int NW>
__device__ __forceinline__ void wl_back(const double *T, const double *rd, double *z) {
    const int lane = threadIdx.x & 63, li = lane & 15, lk = lane >> 4;
    const int wv = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    // sum over k of tile entry (li, k) and v_k, k = 4 q + lk, in every 16-lane row
    auto row_dot = [&](const double (&t)[4], const double *v) -> double {
        double s = 0.0;
#pragma unroll
        for (int q = 0; q < 4; ++q) s = __builtin_fma(t[q], v[4 * q + lk], s);
        return lb_rowsum(s);
    };
    auto row_load = [&](const double *tile, double (&t)[4]) {
#pragma unroll
        for (int q = 0; q < 4; ++q) t[q] = tile[wl_at(li, 4 * q + lk)];
    };
    for (int i = threadIdx.x; i < 16 * P; i += blockDim.x) z[i] *= rd[i];
    __syncthreads();
    double e[4], w[4];
    if (wv == 0) row_load(T + wl_tile(P, P - 1, P - 1), e);
#pragma unroll 1
    for (int p = P - 1; p >= 0; --p) {
        if (wv == 0) {
            if (p > 0) row_load(T + wl_tile(P, p - 1, p), w);
            const double y = row_dot(e, z + 16 * p);
            if (lk == 0) z[16 * p + li] = y;
            if (p > 0) row_load(T + wl_tile(P, p - 1, p - 1), e);
        }
        __syncthreads();
        if (wv == 0) {
            if (p > 0) {
                const int i = 16 * (p - 1) + li;
                const double s = row_dot(w, z + 16 * p);
                if (lk == 0) z[i] = __builtin_fma(-rd[i], s, z[i]);
                __builtin_amdgcn_wave_barrier();
            }
        } else {
            for (int I = wv - 1; I < p - 1; I += NW - 1) {
                double t[4];
                row_load(T + wl_tile(P, I, p), t);
                const double s = row_dot(t, z + 16 * p);
                if (lk == 0) z[16 * I + li] = __builtin_fma(-rd[16 * I + li], s, z[16 * I + li]);
            }
        }
    }
    __syncthreads();
}

// X = L^{-1} after wl_factor, wave J < P forming tile column J in registers,
// X_IJ = -E_I sum_k L_Ik X_kJ with the X_kJ of the column at hand.
template <int P>
__device__ __forceinline__ void wl_lower_inverse(const double *T, const double *rd, dvec4 (&X)[P]) {
    const int lane = threadIdx.x & 63, li = lane & 15, lk = lane >> 4;
    const int J = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    if (J >= P) return;
    int at[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) at[q] = wl_at(4 * q + lk, li);
#pragma unroll
    for (int I = 0; I < P; ++I) {
        if (I == J) {
            const double *E = T + wl_tile(P, J, J);
#pragma unroll
            for (int r = 0; r < 4; ++r) X[I][r] = E[wl_at(li, 4 * r + lk)];
        } else if (I > J) {
            dvec4 acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int k = 0; k < I; ++k)
                if (k >= J) {
                    const double *w = T + wl_tile(P, k, I);
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        acc = __builtin_amdgcn_mfma_f64_16x16x4f64(
                            -w[at[q]] * rd[16 * k + 4 * q + lk], X[k][q], acc, 0, 0, 0);
                }
            const double *E = T + wl_tile(P, I, I);
            X[I] = dvec4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int q = 0; q < 4; ++q)
                X[I] = __builtin_amdgcn_mfma_f64_16x16x4f64(E[at[q]], acc[q], X[I], 0, 0, 0);
        }
    }
}

// The factored form of (L D L^T)^{-1} after wl_factor, row-major K x K:
// X = L^{-1} below the diagonal, its mirror image above, 1 / d_i on it.
// y = X^T D^{-1} X r from it is as accurate as the two substitutions, which
// the product with the inverse is not: of rows that nearly repeat, r almost
// the same for both, each entry of H r rounds by itself, and A^T y passes the
// rounding on magnified (160 rows, pairs 1e-4 apart: the adjoint's dL/dx0 59
// times further from the exact one).
template <int P, int NW>
__device__ __forceinline__ void wl_put_factor(const double *T, const double *rd, int K,
                                              double *__restrict__ M) {
    static_assert(NW >= P, "a wave per tile column");
    const int lane = threadIdx.x & 63, li = lane & 15, lk = lane >> 4;
    const int J = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    dvec4 X[P];
    wl_lower_inverse<P>(T, rd, X);
    if (J >= P) return;
#pragma unroll
    for (int I = 0; I < P; ++I)
        if (I >= J)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int i = 16 * I + lk + 4 * r, j = 16 * J + li;
                if (i < K && j < i) {
                    M[(int64_t)i * K + j] = X[I][r];
                    M[(int64_t)j * K + i] = X[I][r];
                }
            }
    for (int i = 16 * J + lane; i < 16 * J + 16 && i < K; i += 64) M[(int64_t)i * K + i] = rd[i];
}

// H = (L D L^T)^{-1} after wl_factor, written row-major K x K: X = L^{-1}, its
// columns into the tiles' places, then
// H_IJ = sum_{k >= I} X_kI^T D_k^{-1} X_kJ with the mirrored entries from the
// lower ones, so that H is exactly symmetric.
template <int P, int NW>
__device__ __forceinline__ void wl_inverse(double *T, const double *rd, int K,
                                           double *__restrict__ H) {
    static_assert(NW >= P, "a wave per tile column");
    const int lane = threadIdx.x & 63, li = lane & 15, lk = lane >> 4;
    const int wv = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    int at[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) at[q] = wl_at(4 * q + lk, li);
    dvec4 X[P];
    wl_lower_inverse<P>(T, rd, X);
    __syncthreads();
    if (wv < P) {
        const int J = wv;
#pragma unroll
        for (int I = 0; I < P; ++I)
            if (I >= J) {
                double *t = T + wl_tile(P, J, I);
#pragma unroll
                for (int r = 0; r < 4; ++r) t[at[r]] = X[I][r];
            }
    }
    __syncthreads();
    int J = 0, I = wv;   // tile (I, J) of H, J <= I, dealt to the waves
    while (true) {
        while (J < P && I >= P) { ++J; I -= P - J; }
        if (J >= P) break;
        dvec4 acc = {0.0, 0.0, 0.0, 0.0};
        for (int k = I; k < P; ++k) {
            const double *xi = T + wl_tile(P, I, k), *xj = T + wl_tile(P, J, k);
#pragma unroll
            for (int q = 0; q < 4; ++q)
                acc = __builtin_amdgcn_mfma_f64_16x16x4f64(xi[at[q]] * rd[16 * k + 4 * q + lk],
                                                           xj[at[q]], acc, 0, 0, 0);
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int i = 16 * I + lk + 4 * r, j = 16 * J + li;
            if (i < K && j <= i) {
                H[(int64_t)i * K + j] = acc[r];
                if (j < i) H[(int64_t)j * K + i] = acc[r];
            }
        }
        I += NW;
    }
}

}  // namespace rorbk
