// ldl_wg.h -- LDL^T of a symmetric positive definite system of up to 176 rows
// in one workgroup's LDS, for greedy sets of 65 to 161 rows (Algorithm 1's
// greedy step) and for the stored inverses of fixed blocks of at most 161 rows
// (Section 3.1).  Internal to the library.
//
// The matrix is kept as the upper 16 x 16 tiles T_pJ (p <= J) of its padded
// size 16 P, row-major, in LDS.  Tile row p: wave 0 eliminates the diagonal
// tile in registers (lb_tile, ldl_blk.h) and leaves E_p^T in its place; the
// waves form W_J = E_p T_pJ; then T_IJ -= W_I^T D_p^{-1} W_J on FP64 MFMA, wave
// 0 taking the next diagonal tile and going on to eliminate it while the
// others update the rest.  All operands are read as rows of 16 consecutive
// doubles, the layout the MFMA results are written in, so nothing is
// transposed.  What bounds it is the chain of eliminations, 1.4 us per tile
// row with its two barriers; the products fit beside it.
#pragma once

#include "ldl_blk.h"

namespace rorbk {

constexpr int WT = 256;                                    // doubles of a tile
constexpr int WL_MAXP = (MAXB + 15) / 16;                  // 11: blocks of 161 rows
constexpr int wl_tiles(int P) { return P * (P + 1) / 2; }
__device__ __forceinline__ int wl_tile(int P, int p, int J) {
    return (p * P - p * (p - 1) / 2 + J - p) * WT;
}

// Entry f of the packed lower triangle (value g) into the tiles: (j, i) of the
// upper triangle, both halves of a diagonal tile; lambda on the diagonal.
__device__ __forceinline__ void wl_put(double *T, int P, int f, double g, double lambda) {
    int i = (int)((__builtin_amdgcn_sqrtf(8.0f * (float)f + 1.0f) - 1.0f) * 0.5f);
    i -= (i * (i + 1) / 2 > f) ? 1 : 0;
    i += ((i + 1) * (i + 2) / 2 <= f) ? 1 : 0;
    const int j = f - i * (i + 1) / 2;
    double *t = T + wl_tile(P, j >> 4, i >> 4);
    const double v = (i == j) ? g + lambda : g;
    t[(j & 15) * 16 + (i & 15)] = v;
    if ((j >> 4) == (i >> 4)) t[(i & 15) * 16 + (j & 15)] = v;
}

// The identity in rows K .. 16 P - 1, by the whole workgroup.
__device__ __forceinline__ void wl_pad(double *T, int P, int K) {
    const int pad = 16 * P - K;   // at most 16 rows: the last tile column
    for (int e = threadIdx.x; e < pad * 16 * P; e += blockDim.x) {
        const int i = K + e / (16 * P), j = e % (16 * P);
        if (j > i) continue;
        double *t = T + wl_tile(P, j >> 4, i >> 4);
        const double v = (i == j) ? 1.0 : 0.0;
        t[(j & 15) * 16 + (i & 15)] = v;
        if ((j >> 4) == (i >> 4)) t[(i & 15) * 16 + (j & 15)] = v;
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
    const int at = lk * 16 + li;   // + 64 q: entry (4 q + lk, li) of a tile
    __syncthreads();
#pragma unroll 1
    for (int p = 0; p < P; ++p) {
        double *Tp = T + wl_tile(P, p, p);
        if (wv == 0) {
            double a[16], e[4];
#pragma unroll
            for (int j = 0; j < 16; ++j) a[j] = Tp[j * 16 + li];
#pragma unroll
            for (int q = 0; q < 4; ++q) e[q] = (li == 4 * q + lk) ? 1.0 : 0.0;
            double zz = RHS ? z[16 * p + li] : 0.0;
            lb_tile(std::make_integer_sequence<int, 16>{}, a, e, zz, rd + 16 * p, li);
            if (RHS && lk == 0) z[16 * p + li] = zz;
#pragma unroll
            for (int q = 0; q < 4; ++q) Tp[64 * q + at] = e[q];
        }
        __syncthreads();
        if (p + 1 == P) break;   // uniform
        double e[4], r[4], u[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            e[q] = Tp[64 * q + at];
            r[q] = rd[16 * p + 4 * q + lk];
            u[q] = RHS ? z[16 * p + 4 * q + lk] : 0.0;
        }
        for (int J = p + 1 + wv; J < P; J += NW) {
            double *t = Tp + (J - p) * WT;
            dvec4 w = {0.0, 0.0, 0.0, 0.0};
            double b[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) b[q] = t[64 * q + at];
#pragma unroll
            for (int q = 0; q < 4; ++q) w = __builtin_amdgcn_mfma_f64_16x16x4f64(e[q], b[q], w, 0, 0, 0);
#pragma unroll
            for (int q = 0; q < 4; ++q) t[64 * q + at] = w[q];
            if (RHS) {
                double s = 0.0;
#pragma unroll
                for (int q = 0; q < 4; ++q) s = __builtin_fma(-w[q] * r[q], u[q], s);
                s = lb_rowsum(s);
                if (lk == 0) z[16 * J + li] += s;
            }
        }
        __syncthreads();
        // the next diagonal tile on wave 0, the others dealt to the rest
        const int n = P - p - 1;
        int I = 0, J = (wv == 0) ? 0 : wv;
        while (true) {
            while (I < n && J >= n) { ++I; J -= n - I; }   // tile (I, J) in row order
            if (I >= n) break;
            const double *wi = Tp + (I + 1) * WT, *wj = Tp + (J + 1) * WT;
            double *t = T + wl_tile(P, p + 1 + I, p + 1 + J);
            double av[4], bv[4];
            dvec4 acc;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                av[q] = -wi[64 * q + at] * r[q];
                bv[q] = wj[64 * q + at];
                acc[q] = t[64 * q + at];
            }
#pragma unroll
            for (int q = 0; q < 4; ++q)
                acc = __builtin_amdgcn_mfma_f64_16x16x4f64(av[q], bv[q], acc, 0, 0, 0);
#pragma unroll
            for (int q = 0; q < 4; ++q) t[64 * q + at] = acc[q];
            if (wv == 0) break;
            J += NW - 1;
        }
    }
    bool ok = true;
    for (int i = threadIdx.x; i < 16 * P; i += blockDim.x)
        ok = ok && rd[i] > 0.0 && rd[i] < __builtin_inf();
    return __syncthreads_and(ok ? 1 : 0) != 0;
}

// y = L^{-T} D^{-1} z after wl_factor with RHS, into z: from the last tile row,
// y_p = E_p^T w_p on wave 0, then w_I -= L_pI^T y_p for the rows above, a wave
// each.  Ends with a barrier.
template <int P, int NW>
__device__ __forceinline__ void wl_back(const double *T, const double *rd, double *z) {
    const int lane = threadIdx.x & 63, li = lane & 15, lk = lane >> 4;
    const int wv = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    for (int i = threadIdx.x; i < 16 * P; i += blockDim.x) z[i] *= rd[i];
#pragma unroll 1
    for (int p = P - 1; p >= 0; --p) {
        double l[16];
        if (wv == 0) {
            const double *E = T + wl_tile(P, p, p) + li * 16;
#pragma unroll
            for (int j = 0; j < 16; ++j) l[j] = E[j];
        }
        __syncthreads();
        if (wv == 0) {
            const double y = lb_dot(0.0, l, z[16 * p + li]);
            if (lk == 0) z[16 * p + li] = y;
        }
        __syncthreads();
        for (int I = wv; I < p; I += NW) {
            const double *w = T + wl_tile(P, I, p) + li * 16 + lk;
            double s = 0.0;
#pragma unroll
            for (int q = 0; q < 4; ++q) s = __builtin_fma(w[4 * q], z[16 * p + 4 * q + lk], s);
            s = lb_rowsum(s);
            if (lk == 0) z[16 * I + li] = __builtin_fma(-rd[16 * I + li], s, z[16 * I + li]);
        }
    }
    __syncthreads();
}

// H = (L D L^T)^{-1} after wl_factor, written row-major K x K: X = L^{-1} by
// tile columns, a wave each (X_IJ = -E_I sum_k L_Ik X_kJ with the X_kJ of the
// column in registers), the columns into the tiles' places, then
// H_IJ = sum_{k >= I} X_kI^T D_k^{-1} X_kJ with the mirrored entries from the
// lower ones, so that H is exactly symmetric.
template <int P, int NW>
__device__ __forceinline__ void wl_inverse(double *T, const double *rd, int K,
                                           double *__restrict__ H) {
    static_assert(NW >= P, "a wave per tile column");
    const int lane = threadIdx.x & 63, li = lane & 15, lk = lane >> 4;
    const int wv = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int at = lk * 16 + li;
    dvec4 X[P];
    if (wv < P) {
        const int J = wv;
#pragma unroll
        for (int I = 0; I < P; ++I) {
            if (I == J) {
                const double *E = T + wl_tile(P, J, J) + li * 16 + lk;
#pragma unroll
                for (int r = 0; r < 4; ++r) X[I][r] = E[4 * r];
            } else if (I > J) {
                dvec4 acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
                for (int k = 0; k < I; ++k)
                    if (k >= J) {
                        const double *w = T + wl_tile(P, k, I);
#pragma unroll
                        for (int q = 0; q < 4; ++q)
                            acc = __builtin_amdgcn_mfma_f64_16x16x4f64(
                                -w[64 * q + at] * rd[16 * k + 4 * q + lk], X[k][q], acc, 0, 0, 0);
                    }
                const double *E = T + wl_tile(P, I, I);
                X[I] = dvec4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    X[I] = __builtin_amdgcn_mfma_f64_16x16x4f64(E[64 * q + at], acc[q], X[I], 0, 0, 0);
            }
        }
    }
    __syncthreads();
    if (wv < P) {
        const int J = wv;
#pragma unroll
        for (int I = 0; I < P; ++I)
            if (I >= J) {
                double *t = T + wl_tile(P, J, I);
#pragma unroll
                for (int r = 0; r < 4; ++r) t[64 * r + at] = X[I][r];
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
                acc = __builtin_amdgcn_mfma_f64_16x16x4f64(xi[64 * q + at] * rd[16 * k + 4 * q + lk],
                                                           xj[64 * q + at], acc, 0, 0, 0);
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
