// rorbk_device.h -- device-side building blocks shared by the ROR-BK kernels:
// element types, 16-byte vector loads, FP64 MFMA Gram tiles and deterministic
// reductions.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <utility>

#include "rorbk_internal.h"

namespace rorbk {

constexpr int WAVE = 64;
constexpr int MAXB = RORBK_MAX_BLOCK_ROWS + 1;          // largest block (rows)
constexpr int BIGB = RORBK_MAX_BIG_BLOCK_ROWS;          // largest block, dense large-block path
constexpr int MAXK = BIGB > MAXB ? BIGB : MAXB;         // largest greedy set

typedef uint16_t bf16_t;
typedef double dvec2 __attribute__((ext_vector_type(2)));
typedef float fvec4 __attribute__((ext_vector_type(4)));
typedef uint32_t uvec4 __attribute__((ext_vector_type(4)));
typedef double dvec4 __attribute__((ext_vector_type(4)));

// Closed-form partition (Algorithm 1, first step): block t starts at
// t*q + min(t, rem) and has q or q+1 rows; its stored inverse starts at
// sum_{s<t} b_s (b_s + zc), zc columns of zeros standing behind each.
__device__ __forceinline__ int64_t blk_start(int64_t t, int64_t q, int64_t rem) {
    return t * q + (t < rem ? t : rem);
}
__device__ __forceinline__ int blk_rows(int64_t t, int64_t q, int64_t rem) {
    return (int)(q + (t < rem ? 1 : 0));
}
__device__ __forceinline__ int64_t blk_hoff(int64_t t, int64_t q, int64_t rem, int64_t zc) {
    const int64_t big = t < rem ? t : rem;
    return big * (q + 1) * (q + 1 + zc) + (t - big) * q * (q + zc);
}

// Storage traits: elements per 16-byte load.
template <typename T> struct Tr;
template <> struct Tr<double> { static constexpr int VW = 2; };
template <> struct Tr<float> { static constexpr int VW = 4; };
template <> struct Tr<bf16_t> { static constexpr int VW = 8; };

__device__ __forceinline__ float bf16_to_f32(bf16_t v) {
    return __uint_as_float(((uint32_t)v) << 16);
}

template <typename V> __device__ __forceinline__ V to_v(double a) { return (V)a; }
template <typename V> __device__ __forceinline__ V to_v(float a) { return (V)a; }
template <typename V> __device__ __forceinline__ V to_v(bf16_t a) { return (V)bf16_to_f32(a); }

__device__ __forceinline__ double fmaT(double a, double b, double c) { return __builtin_fma(a, b, c); }
__device__ __forceinline__ float fmaT(float a, float b, float c) { return __builtin_fmaf(a, b, c); }

// Elements of a raw 16-byte vector (VW elements from column c) at or past
// `lim` set to zero, by selects (no branch).
template <typename T>
__device__ __forceinline__ uvec4 mask_raw(uvec4 w, int64_t c, int64_t lim) {
    if constexpr (sizeof(T) == 8) {
        const bool k1 = c + 1 < lim;
        const bool k0 = c < lim;
        w[0] = k0 ? w[0] : 0u;
        w[1] = k0 ? w[1] : 0u;
        w[2] = k1 ? w[2] : 0u;
        w[3] = k1 ? w[3] : 0u;
    } else if constexpr (sizeof(T) == 4) {
#pragma unroll
        for (int e = 0; e < 4; ++e) w[e] = (c + e < lim) ? w[e] : 0u;
    } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const uint32_t lo = (c + 2 * e < lim) ? 0x0000ffffu : 0u;
            const uint32_t hi = (c + 2 * e + 1 < lim) ? 0xffff0000u : 0u;
            w[e] &= (lo | hi);
        }
    }
    return w;
}

// 16 raw bytes (VW elements) of a row at column c (c < lim); elements at or
// past `lim` read as zero.  ALIGNED (row start 16-byte aligned, row stride a
// multiple of VW elements, c a multiple of VW): one 16-byte load, which stays
// inside the row's stride even when it crosses lim (c < lim <= n <= stride),
// and the tail masked by selects, so the code has no branch around the load.
// Otherwise one 16-byte load at the element's own alignment (gfx950 reads any
// byte address; a line that two loads share is read from the cache the second
// time): of the vector at c, or, where that would cross lim, of the last whole
// vector before lim, moved down by tail_shift.  Where no lane of the wave
// crosses lim the shift is skipped by a scalar branch.  Rows of fewer than VW
// elements are read one by one.
typedef uvec4 uvec4_a2 __attribute__((aligned(2)));
typedef uvec4 uvec4_a4 __attribute__((aligned(4)));
typedef uvec4 uvec4_a8 __attribute__((aligned(8)));
template <typename T, bool NT>
__device__ __forceinline__ uvec4 load_any(const T *__restrict__ p) {
    if constexpr (sizeof(T) == 2) {
        const uvec4_a2 *q = reinterpret_cast<const uvec4_a2 *>(p);
        return NT ? __builtin_nontemporal_load(q) : *q;
    } else if constexpr (sizeof(T) == 4) {
        const uvec4_a4 *q = reinterpret_cast<const uvec4_a4 *>(p);
        return NT ? __builtin_nontemporal_load(q) : *q;
    } else {
        const uvec4_a8 *q = reinterpret_cast<const uvec4_a8 *>(p);
        return NT ? __builtin_nontemporal_load(q) : *q;
    }
}

// The vector at c from the one read at min(c, lim - VW): its elements moved
// down by c - (lim - VW) places, zeros at or past lim (all zero for c >= lim).
template <typename T>
__device__ __forceinline__ uvec4 tail_shift(uvec4 w, int64_t c, int64_t lim) {
    constexpr int VW = Tr<T>::VW;
    const int64_t over = c - (lim - VW);
    const uint32_t sh = over <= 0 ? 0u : (over >= VW ? 16u : (uint32_t)over * (uint32_t)sizeof(T));
    if (sh & 8u) w = uvec4{w[2], w[3], 0u, 0u};
    if (sh & 4u) w = uvec4{w[1], w[2], w[3], 0u};
    if constexpr (sizeof(T) == 2) {
        if (sh & 2u)
            w = uvec4{(w[0] >> 16) | (w[1] << 16), (w[1] >> 16) | (w[2] << 16),
                      (w[2] >> 16) | (w[3] << 16), w[3] >> 16};
    }
    return (sh & 16u) ? uvec4{0u, 0u, 0u, 0u} : w;
}

template <typename T, bool ALIGNED, bool NT = false>
__device__ __forceinline__ uvec4 load_raw(const T *__restrict__ row, int64_t c, int64_t lim) {
    constexpr int VW = Tr<T>::VW;
    if constexpr (ALIGNED) {
        const uvec4 *pv = reinterpret_cast<const uvec4 *>(row + c);
        return mask_raw<T>(NT ? __builtin_nontemporal_load(pv) : *pv, c, lim);
    }
    if (lim >= VW) {   // uniform
        const bool full = c + VW <= lim;
        uvec4 w = load_any<T, NT>(row + (full ? c : lim - VW));
        if (__ballot(!full) != 0ull) w = tail_shift<T>(w, c, lim);
        return w;
    }
    uvec4 w = {0u, 0u, 0u, 0u};
    if constexpr (sizeof(T) == 8) {
#pragma unroll
        for (int e = 0; e < 2; ++e)
            if (c + e < lim) {
                const uint64_t u = (uint64_t)__double_as_longlong((double)row[c + e]);
                w[2 * e] = (uint32_t)u;
                w[2 * e + 1] = (uint32_t)(u >> 32);
            }
    } else if constexpr (sizeof(T) == 4) {
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (c + e < lim) w[e] = __float_as_uint((float)row[c + e]);
    } else {
#pragma unroll
        for (int e = 0; e < 8; ++e)
            if (c + e < lim) w[e >> 1] |= ((uint32_t)(uint16_t)row[c + e]) << (16 * (e & 1));
    }
    return w;
}

// load_raw of (row, c) when `ok` and c < lim, else zero, with no branch
// around the load: otherwise the vector at (srow, sc) is read instead (any
// vector known to lie inside the matrix, sc < lim) and dropped by a select.
// (A load behind a lane-dependent branch makes the compiler wait for it to
// land before the other lanes' zero may be written to the same registers,
// which turns loads meant to overlap into a chain of memory round trips.)
template <typename T, bool ALIGNED>
__device__ __forceinline__ uvec4 load_raw_sel(const T *__restrict__ row, int64_t c, int64_t lim,
                                              bool ok, const T *__restrict__ srow, int64_t sc) {
    const bool g = ok && c < lim;
    const uvec4 w = load_raw<T, ALIGNED>(g ? row : srow, g ? c : sc, lim);
    const uvec4 z = {0u, 0u, 0u, 0u};
    return g ? w : z;
}

// load_raw_sel for the Gram kernels, whose steps read many rows: aligned rows
// are masked here by selects; others are left as read, so that the loads of a
// step go out together (behind each load of a row's end would stand a branch
// that waits for it), and the caller clears what was not asked for and moves
// the end of the row with tail_shift.  lim >= VW there.  Lanes that ask for
// nothing read (srow, sc): one address for many lanes costs less than many.
// Block Grams of 31 x 2998 FP32 46 us with a branch at each load, 31 so; 31 x
// 2999 FP64 61 (two 8-byte loads each) and 38; the greedy Grams of one chain
// iteration on those 14 and 11, 21 and 14.
template <typename T, bool ALIGNED>
__device__ __forceinline__ uvec4 load_gram(const T *__restrict__ row, int64_t c, int64_t lim,
                                           bool ok, const T *__restrict__ srow, int64_t sc) {
    constexpr int VW = Tr<T>::VW;
    if constexpr (ALIGNED) {
        return load_raw_sel<T, true>(row, c, lim, ok, srow, sc);
    } else {
        const bool g = ok && c < lim;
        const int64_t ca = c < lim - VW ? c : lim - VW, sa = sc < lim - VW ? sc : lim - VW;
        return load_any<T, false>((g ? row : srow) + (g ? ca : sa));
    }
}

template <typename T, bool ALIGNED>
__device__ __forceinline__ uvec4 load_raw_nt_sel(const T *__restrict__ row, int64_t c, int64_t lim,
                                                 bool ok, const T *__restrict__ srow, int64_t sc) {
    const bool g = ok && c < lim;
    const uvec4 w = load_raw<T, ALIGNED, true>(g ? row : srow, g ? c : sc, lim);
    const uvec4 z = {0u, 0u, 0u, 0u};
    return g ? w : z;
}

template <typename T, typename V>
__device__ __forceinline__ void cvt_raw(const uvec4 &w, V (&out)[Tr<T>::VW]) {
    if constexpr (sizeof(T) == 8) {
        out[0] = (V)__longlong_as_double((long long)(((uint64_t)w[1] << 32) | w[0]));
        out[1] = (V)__longlong_as_double((long long)(((uint64_t)w[3] << 32) | w[2]));
    } else if constexpr (sizeof(T) == 4) {
#pragma unroll
        for (int e = 0; e < 4; ++e) out[e] = (V)__uint_as_float(w[e]);
    } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            out[2 * e] = (V)__uint_as_float(w[e] << 16);
            out[2 * e + 1] = (V)__uint_as_float(w[e] & 0xffff0000u);
        }
    }
}

// FP64 MFMA tile of a Gram product: acc += X_a X_b^T over columns [c0, c1)
// for a 16 x 16 tile, one wave.  Lane l supplies row ra (A side) and rb (B
// side) for tile row/column l % 16 (a negative row reads as zero) and the
// E = 32 / sizeof(T) >= 4 consecutive columns c + g*E .. of lane group
// g = l / 16, which serve as the k index of E v_mfma_f64_16x16x4f64 steps
// (the sum runs over every column once, in a fixed order).  Result layout:
// D[i][j] sits in register i / 4 of lane (i % 4) * 16 + j.  c0 must be a
// multiple of E when ALIGNED.
template <typename T, bool ALIGNED>
__device__ __forceinline__ void mfma_gram_tile(const T *__restrict__ X, int64_t ld, int64_t ra,
                                               int64_t rb, int64_t c0, int64_t c1, dvec4 &acc) {
    constexpr int VW = Tr<T>::VW;
    constexpr int E = (sizeof(T) == 8) ? 4 : VW;   // columns per lane per macro step
    constexpr int NL = E / VW;                      // 16-byte loads per row per step
    constexpr int U = 4;                            // macro steps in flight
    const int g = (threadIdx.x & 63) >> 4;
    const T *pa = X + (ra >= 0 ? ra : 0) * ld;
    const T *pb = X + (rb >= 0 ? rb : 0) * ld;
    const bool same = (ra == rb);
    const bool useb = !same && rb >= 0;
    const bool tiny = !ALIGNED && c1 < VW;   // uniform: no whole vector in the row
    const uvec4 z = {0u, 0u, 0u, 0u};
    for (int64_t c = c0; c < c1; c += 4 * E * U) {
        uvec4 wa[U][NL], wb[U][NL];
        if (tiny) {
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int h = 0; h < NL; ++h) wa[u][h] = wb[u][h] = z;
            if (g == 0) {
                wa[0][0] = load_raw<T, false>(pa, 0, c1);
                wb[0][0] = load_raw<T, false>(pb, 0, c1);
            }
        } else {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int64_t col = c + (int64_t)u * 4 * E + (int64_t)g * E;
#pragma unroll
                for (int h = 0; h < NL; ++h) {
                    wa[u][h] = load_gram<T, ALIGNED>(pa, col + h * VW, c1, ra >= 0, X, c0);
                    wb[u][h] = load_gram<T, ALIGNED>(pb, col + h * VW, c1, useb, X, c0);
                }
            }
        }
        if (!ALIGNED) {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int64_t cu = c + (int64_t)u * 4 * E, col = cu + (int64_t)g * E;
                const bool past = cu >= c1;
                if (!tiny && !past && cu + 4 * E > c1) {
#pragma unroll
                    for (int h = 0; h < NL; ++h) {
                        wa[u][h] = tail_shift<T>(wa[u][h], col + h * VW, c1);
                        wb[u][h] = tail_shift<T>(wb[u][h], col + h * VW, c1);
                    }
                }
#pragma unroll
                for (int h = 0; h < NL; ++h) {
                    wa[u][h] = !past && ra >= 0 ? wa[u][h] : z;
                    wb[u][h] = !past && rb >= 0 ? wb[u][h] : z;
                }
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int h = 0; h < NL; ++h) {
                double av[VW], bv[VW];
                cvt_raw<T, double>(wa[u][h], av);
                if (same) {
#pragma unroll
                    for (int e = 0; e < VW; ++e) bv[e] = av[e];
                } else {
                    cvt_raw<T, double>(wb[u][h], bv);
                }
#pragma unroll
                for (int e = 0; e < VW; ++e)
                    acc = __builtin_amdgcn_mfma_f64_16x16x4f64(av[e], bv[e], acc, 0, 0, 0);
            }
    }
}

// Butterfly sum over the `width` lanes of a lane group (width a power of two
// <= 64).  The combination order is fixed, so the result is reproducible.
template <typename V>
__device__ __forceinline__ V group_sum(V v, int width) {
    for (int off = width >> 1; off > 0; off >>= 1) v += __shfl_xor(v, off, width);
    return v;
}

// Sum over a workgroup of `nthreads` threads in a fixed order: butterfly
// within waves, then wave partials summed in wave order.  `sh` holds at least
// nthreads/64 doubles.  All threads receive the result.
__device__ __forceinline__ double block_sum(double v, double *sh) {
    v = group_sum(v, WAVE);
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    __syncthreads();
    if (lane == 0) sh[w] = v;
    __syncthreads();
    double s = 0.0;
    const int nw = (blockDim.x + 63) >> 6;
    for (int i = 0; i < nw; ++i) s += sh[i];
    __syncthreads();
    return s;
}

__device__ __forceinline__ int pk(int i, int j) { return i * (i + 1) / 2 + j; }  // j <= i

// t-th tile of the lower triangle of an nt x nt tile grid, row-major.
__device__ __forceinline__ void tile_of(int t, int nt, int *bi, int *bj) {
    int i = 0, base = 0;
    while (i < nt && base + i + 1 <= t) { base += i + 1; ++i; }
    if (i >= nt) { *bi = -1; *bj = -1; return; }
    *bi = i;
    *bj = t - base;
}

}  // namespace rorbk
