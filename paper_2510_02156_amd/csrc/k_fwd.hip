// k_fwd.hip -- the forward iteration's block steps for dense row-major
// matrices whose blocks have at most FWD_B rows (row form): the three sampled
// updates of an outer iteration (Algorithm 1, inner loop) in one launch, the
// greedy update fused with the next iteration's products, the cross-Grams
// of the three sampled blocks, and the chain form in which the greedy update
// of iteration it and the sampled updates of iteration it + 1 share one pass.
//
// The three sampled steps x1 = x0 + A1^T y1, x2 = x1 + A2^T y2,
// x3 = x2 + A3^T y3 with y_l = H_l (b_l - A_l x_{l-1}) (Lemma 2's update
// rule, H_l the stored inverse of block l, Section 3.1) need A_2 x1 and
// A_3 x2.  Since A_2 x1 = A_2 x0 + (A_2 A_1^T) y1 and
// A_3 x2 = A_3 x0 + (A_3 A_1^T) y1 + (A_3 A_2^T) y2, the three products
// A_l x0 (one pass, partial sums per column slab) and the cross-Grams
// A_2 A_1^T, A_3 A_1^T, A_3 A_2^T (which do not depend on x and are formed one
// iteration ahead) give y1, y2, y3 in a short chain of small matrix-vector
// products, and x3 = x0 + A_1^T y1 + A_2^T y2 + A_3^T y3 is one more pass.  The
// same iterate results in exact arithmetic; the roundings differ from three
// separate steps.
#include "ldl_blk.h"
#include "rorbk_device.h"
#include "xgram.h"

namespace rorbk {

constexpr int FWD_T = 512;      // threads of the step kernels

// The three blocks drawn at tau[ti .. ti+2]: first row and row count of each
// (named scalars, so that no index into them is computed at run time).
struct Blk3 {
    int64_t s0, s1, s2;
    int c0, c1, c2;
};

__device__ __forceinline__ void blocks3(const int32_t *__restrict__ tau, int64_t ti, int64_t q,
                                        int64_t rem, Blk3 &B) {
    const int64_t t0 = tau[ti], t1 = tau[ti + 1], t2 = tau[ti + 2];
    B.s0 = blk_start(t0, q, rem);
    B.s1 = blk_start(t1, q, rem);
    B.s2 = blk_start(t2, q, rem);
    B.c0 = blk_rows(t0, q, rem);
    B.c1 = blk_rows(t1, q, rem);
    B.c2 = blk_rows(t2, q, rem);
}

// Row qq of the three blocks taken in order: its block l, offset i and row.
__device__ __forceinline__ void split3(const Blk3 &B, int qq, int *l, int *i, int64_t *row) {
    const bool a = qq >= B.c0, b = qq >= B.c0 + B.c1;
    *l = (int)a + (int)b;
    *i = qq - (a ? B.c0 : 0) - (b ? B.c1 : 0);
    // offsets added under two independent selects (a three-way select can be
    // turned into an indexed table in scratch memory)
    *row = B.s0 + (a ? B.s1 - B.s0 : 0) + (b ? B.s2 - B.s1 : 0) + *i;
}

// Columns of one sub-slab: 64 for FP64 storage (16 row groups of 32 lanes
// keep the three-block row set in registers), 128 otherwise.
template <typename T>
__host__ __device__ constexpr int fwd_swc() { return sizeof(T) == 8 ? 64 : 128; }

template <typename T, bool AL, int NW>
__global__ __launch_bounds__(64 * NW) void k_xgram(const T *__restrict__ A, int64_t ld, int64_t n,
                                                   const int32_t *__restrict__ tau, int64_t ti,
                                                   int64_t q, int64_t rem, int bmax,
                                                   double *__restrict__ out,
                                                   const Ctrl *__restrict__ ctrl) {
    if (ctrl->done) return;
    xgram_tile<T, AL, NW>(A, ld, n, tau, ti, q, rem, bmax, blockIdx.x, out);
}

// ------------------------------------------------- Grams of the chain form --
// After the selection of iteration it, with the blocks S' drawn for iteration
// it + 1 at tau[ti .. ti+2]: the greedy Gram A_I A_I^T (packed lower) and
// C = A_{S'} A_I^T (C[j * CHAIN_S + l * FWD_B + i] = <row i of block l, row
// I_j>, so that the consumer's loads over a block's rows are contiguous),
// as partial sums over nch column chunks (chunk ch at G + ch * K(K+1)/2 and
// C + ch * CHAIN_C).  Since A_{S'} (x + A_I^T y) = A_{S'} x + C y, the next
// iteration's z = b_{S'} - A_{S'} x_new = r_{S'} - C y follows from the
// residual r of this iteration (taken at x, before the greedy step) once y is
// known, with no pass over x in between.  One 16 x 16 tile of one chunk per
// workgroup: the GC_W waves take consecutive column ranges (multiples of the
// MFMA step) and are summed in wave order.  (The cross-Grams of S' do not
// depend on I and are formed by spare workgroups of the selection.)
constexpr int GC_W = 8;
constexpr int CHAIN_S = 3 * FWD_B;        // slots of S' rows
constexpr int CHAIN_C = CHAIN_S * 64;     // doubles of one chunk of C

struct GramChainP {
    const void *A;
    int64_t ld, n, q, rem;
    int bmax;
    const int32_t *I;
    int K;
    const int32_t *tau;
    int64_t ti;
    int64_t wc;     // columns per chunk (a multiple of 32)
    double *G;      // [nch][K (K + 1) / 2], packed lower
    double *C;      // [nch][64][3 * FWD_B]
    const Ctrl *ctrl;
};

__host__ __device__ inline int gram_chain_tiles(int K, int bmax) {
    const int nt = (K + 15) / 16, nb = (bmax + 15) / 16;
    return nt * (nt + 1) / 2 + 3 * nb * nt;
}

template <typename T, bool AL>
__global__ __launch_bounds__(64 * GC_W) void k_gram_chain(GramChainP p) {
    // the stop flag is read together with the row indices: one memory
    // latency before the row loads instead of two
    const int stop =
        __hip_atomic_load(&p.ctrl->done, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    constexpr int E = (sizeof(T) == 8) ? 4 : Tr<T>::VW;
    const T *__restrict__ A = (const T *)p.A;
    const int K = p.K;
    const int nt = (K + 15) / 16, ntg = nt * (nt + 1) / 2;
    const int nb = (p.bmax + 15) / 16, nc = 3 * nb * nt;
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63, li = lane & 15;
    const int job = (int)blockIdx.x % (ntg + nc), ch = (int)blockIdx.x / (ntg + nc);
    int kind, bi, bj, l = 0, ca = K;
    int64_t ra, rb;
    if (job < ntg) {                 // greedy Gram, lower tiles
        kind = 0;
        tile_of(job, nt, &bi, &bj);
    } else {                         // C: block l of S' against I
        kind = 1;
        const int c = job - ntg;
        l = c / (nb * nt);
        const int rest = c - l * nb * nt;
        bi = rest / nt;
        bj = rest - bi * nt;
    }
    // the greedy rows of this lane, read with clamped indices (no branch
    // around the loads) before the sampled block's start
    const int ia = bi * 16 + li, ib = bj * 16 + li;
    const int32_t Ia = p.I[ia < K ? ia : K - 1];
    const int32_t Ib = p.I[ib < K ? ib : K - 1];
    rb = (ib < K) ? (int64_t)Ib : -1;
    if (kind == 0) {
        ra = (ia < K) ? (int64_t)Ia : -1;
    } else {
        // tile rows j (greedy rows), tile columns i (the block's rows): a
        // wave's stores then run along the slots
        const int64_t t = p.tau[p.ti + l];
        ca = blk_rows(t, p.q, p.rem);
        if (bi * 16 >= ca) return;   // uniform: a tile past the block
        ra = rb;
        rb = (ia < ca) ? blk_start(t, p.q, p.rem) + ia : -1;
    }
    if (stop) return;
    const int64_t c0 = (int64_t)ch * p.wc;
    const int64_t c1 = (c0 + p.wc < p.n) ? c0 + p.wc : p.n;
    const int64_t stepc = 4 * E;
    const int64_t span = ((c1 - c0 + GC_W * stepc - 1) / (GC_W * stepc)) * stepc;
    const int64_t wa = c0 + (int64_t)w * span;
    const int64_t wb = (wa + span < c1) ? wa + span : c1;
    dvec4 acc = {0.0, 0.0, 0.0, 0.0};
    if (wa < wb) mfma_gram_tile<T, AL>(A, p.ld, ra, rb, wa, wb, acc);
    __shared__ double red[GC_W][64][4];
#pragma unroll
    for (int r = 0; r < 4; ++r) red[w][lane][r] = acc[r];
    __syncthreads();
    if (w != 0) return;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        double s = red[0][lane][r];
#pragma unroll
        for (int v = 1; v < GC_W; ++v) s += red[v][lane][r];
        if (kind == 0) {
            const int ii = bi * 16 + (lane >> 4) + 4 * r, jj = bj * 16 + li;
            if (ii < K && jj <= ii) p.G[(int64_t)ch * (K * (K + 1) / 2) + pk(ii, jj)] = s;
        } else {
            const int jj = bj * 16 + (lane >> 4) + 4 * r, ii = bi * 16 + li;
            if (ii < ca && jj < K) p.C[(int64_t)ch * CHAIN_C + jj * CHAIN_S + l * FWD_B + ii] = s;
        }
    }
}

// ------------------------------------------ greedy update + next products --
// x[cols] += A_I[:, cols]^T y_I (the greedy step, y_I given) over column slabs
// of wu columns per workgroup, then the partial products of the next
// iteration's three sampled blocks on the updated slab:
// Pout[w][l * bmax + i] = A_{S_l}[i, cols] . x[cols].  With I == NULL only the
// products are formed (the first iteration of a run); with tau_next < 0 only
// the update (the last iteration).  Rows are spread over G row groups of NV
// lanes (16 bytes each across a sub-slab of fwd_swc columns): the current rows RC per
// thread, the next rows RN per thread.  Every load of both row sets' first
// sub-slab is issued before the first barrier; with PF the next sub-slab's
// rows load while the current one is reduced.  The last workgroup to finish
// (device-scope acquire-release counter) then forms
// z[l * FWD_B + i] = b_{S_l}[i] - sum_ch Pout[ch][l * bmax + i] (chunk order;
// zero in unused slots), the start of the next three-step chain.
struct FwdGreedyP {
    const void *A;
    int64_t ld, n, q, rem;
    int bmax;
    const int32_t *tau;
    int64_t tau_next;
    const int32_t *I;
    int K;
    const double *y;
    void *x;
    double *Pout;
    int64_t wu;
    const Ctrl *ctrl;
    const void *b;         // right-hand side (vector type)
    double *z3;            // z of the next iteration's blocks, slots l * FWD_B + i
    uint32_t *counter;     // workgroups done (0 between launches)
};

template <typename T, typename V, bool AL, int RC, int RN, bool MS>
__global__ __launch_bounds__(FWD_T) void k_fwd_greedy(FwdGreedyP p) {
    constexpr int VW = Tr<T>::VW;
    constexpr int SWC = fwd_swc<T>();
    constexpr int NV = SWC / VW;
    constexpr int G = FWD_T / NV;
    const T *__restrict__ A = (const T *)p.A;
    V *__restrict__ x = (V *)p.x;
    const int tid = threadIdx.x, g = tid / NV, v = tid % NV;
    Blk3 B = {0, 0, 0, 0, 0, 0};
    if (p.tau_next >= 0) blocks3(p.tau, p.tau_next, p.q, p.rem, B);
    const int ncnt = B.c0 + B.c1 + B.c2;
    const int cnt = p.I ? p.K : 0;
    if (p.ctrl->done) return;
    const int64_t c0 = (int64_t)blockIdx.x * p.wu;
    const int64_t c1 = (c0 + p.wu < p.n) ? c0 + p.wu : p.n;
    const int wcols = (int)(c1 - c0);

    __shared__ V s_x[1024];
    __shared__ V s_red[G][SWC];
    __shared__ double s_y[FWD_B];

    int32_t crow[RC], nrow[RN];
    int nidx[RN];
#pragma unroll
    for (int r = 0; r < RC; ++r) {
        const int qq = g + G * r;
        crow[r] = (qq < cnt) ? p.I[qq] : -1;
    }
#pragma unroll
    for (int r = 0; r < RN; ++r) {
        const int qq = g + G * r;
        nrow[r] = -1;
        nidx[r] = 0;
        if (qq < ncnt) {
            int l, i;
            int64_t row;
            split3(B, qq, &l, &i, &row);
            nrow[r] = (int32_t)row;
            nidx[r] = l * p.bmax + i;
        }
    }
    const uvec4 zero4 = {0u, 0u, 0u, 0u};
    uvec4 ua[RC], un[RN];
    {
        const int64_t col = c0 + (int64_t)v * VW;
#pragma unroll
        for (int r = 0; r < RC; ++r)
            ua[r] = load_raw_sel<T, AL>(A + (int64_t)(crow[r] >= 0 ? crow[r] : 0) * p.ld, col, c1,
                                        crow[r] >= 0, A, c0);
#pragma unroll
        for (int r = 0; r < RN; ++r)
            un[r] = load_raw_sel<T, AL>(A + (int64_t)(nrow[r] >= 0 ? nrow[r] : 0) * p.ld, col, c1,
                                        nrow[r] >= 0, A, c0);
    }
    for (int c = tid; c < wcols; c += FWD_T) s_x[c] = x[c0 + c];
    for (int i = tid; i < cnt; i += FWD_T) s_y[i] = p.y[i];
    __syncthreads();
    V yv[RC];
#pragma unroll
    for (int r = 0; r < RC; ++r) {
        const int qq = g + G * r;
        yv[r] = (qq < cnt) ? (V)s_y[qq] : (V)0;
    }
    V pacc[RN];
#pragma unroll
    for (int r = 0; r < RN; ++r) pacc[r] = (V)0;
    // the next sub-slab's rows in flight too while they fit the registers
    constexpr bool PF = MS && (RC + RN <= 11);
    constexpr int RPc = PF ? RC : 1, RPn = PF ? RN : 1;
    for (int64_t sub = c0; sub < c1; sub += SWC) {
        const int64_t col = sub + (int64_t)v * VW;
        const bool more = sub + SWC < c1;   // uniform
        uvec4 ua2[RPc], un2[RPn];
        if constexpr (PF) {
            if (more) {
                const int64_t coln = col + SWC;
#pragma unroll
                for (int r = 0; r < RC; ++r)
                    ua2[r] = load_raw_sel<T, AL>(A + (int64_t)(crow[r] >= 0 ? crow[r] : 0) * p.ld, coln,
                                                 c1, crow[r] >= 0, A, c0);
#pragma unroll
                for (int r = 0; r < RN; ++r)
                    un2[r] = load_raw_sel<T, AL>(A + (int64_t)(nrow[r] >= 0 ? nrow[r] : 0) * p.ld, coln,
                                                 c1, nrow[r] >= 0, A, c0);
            }
        } else if (sub != c0) {
#pragma unroll
            for (int r = 0; r < RC; ++r)
                ua[r] = load_raw_sel<T, AL>(A + (int64_t)(crow[r] >= 0 ? crow[r] : 0) * p.ld, col, c1,
                                            crow[r] >= 0, A, c0);
#pragma unroll
            for (int r = 0; r < RN; ++r)
                un[r] = load_raw_sel<T, AL>(A + (int64_t)(nrow[r] >= 0 ? nrow[r] : 0) * p.ld, col, c1,
                                            nrow[r] >= 0, A, c0);
        }
        if (cnt > 0) {   // uniform
            V acc[VW];
#pragma unroll
            for (int e = 0; e < VW; ++e) acc[e] = (V)0;
#pragma unroll
            for (int r = 0; r < RC; ++r) {
                V a[VW];
                cvt_raw<T, V>(ua[r], a);
#pragma unroll
                for (int e = 0; e < VW; ++e) acc[e] = fmaT(a[e], yv[r], acc[e]);
            }
#pragma unroll
            for (int e = 0; e < VW; ++e) s_red[g][v * VW + e] = acc[e];
            __syncthreads();
            if (tid < SWC) {
                const int64_t cc = sub + tid;
                if (cc < c1) {
                    V s = (V)0;
                    for (int gg = 0; gg < G; ++gg) s += s_red[gg][tid];
                    s_x[cc - c0] += s;
                }
            }
            __syncthreads();
        }
        if (col < c1) {
#pragma unroll
            for (int r = 0; r < RN; ++r) {
                V a[VW];
                cvt_raw<T, V>(un[r], a);
#pragma unroll
                for (int e = 0; e < VW; ++e)
                    if (col + e < c1) pacc[r] = fmaT(a[e], s_x[col + e - c0], pacc[r]);
            }
        }
        if constexpr (PF) {
            if (more) {
#pragma unroll
                for (int r = 0; r < RC; ++r) ua[r] = ua2[r];
#pragma unroll
                for (int r = 0; r < RN; ++r) un[r] = un2[r];
            }
        }
    }
    if (cnt > 0)
        for (int c = tid; c < wcols; c += FWD_T) x[c0 + c] = s_x[c];
    if (ncnt == 0) return;   // uniform: the last iteration has no next products
    // each row's NV lane sums (consecutive lanes of one wave) by a fixed
    // butterfly
#pragma unroll
    for (int r = 0; r < RN; ++r) {
        const V s = group_sum(pacc[r], NV);
        if (v == 0 && nrow[r] >= 0)
            p.Pout[(int64_t)blockIdx.x * 3 * p.bmax + nidx[r]] = (double)s;
    }
    // count this workgroup done; the last one sums the partials
    __shared__ int s_last;
    __syncthreads();
    if (tid == 0)
        s_last = (__hip_atomic_fetch_add(p.counter, 1u, __ATOMIC_ACQ_REL,
                                         __HIP_MEMORY_SCOPE_AGENT) == gridDim.x - 1) ? 1 : 0;
    __syncthreads();
    if (!s_last) return;
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    if (tid == 0) *p.counter = 0u;   // ready for the next launch
    // two threads per slot, each summing alternate chunks (all loads of a
    // batch in flight), then the pair's sum
    const V *__restrict__ bv = (const V *)p.b;
    const int slot = tid >> 1, h = tid & 1;
    if (slot < 3 * FWD_B) {
        const int l = slot / FWD_B, i = slot - l * FWD_B;
        const int cl = (l == 0) ? B.c0 : ((l == 1) ? B.c1 : B.c2);
        const bool ok = i < cl;
        const int64_t row = (l == 0 ? B.s0 : (l == 1 ? B.s1 : B.s2)) + (ok ? i : 0);
        const V bt = bv[row];
        const double *pp = p.Pout + (ok ? l * p.bmax + i : 0);
        const int64_t st = 3 * (int64_t)p.bmax;
        const int nch = gridDim.x;
        double acc = 0.0;
        int ch = h;
        for (; ch + 14 < nch; ch += 16) {
            const double t0 = pp[(int64_t)ch * st], t1 = pp[(int64_t)(ch + 2) * st];
            const double t2 = pp[(int64_t)(ch + 4) * st], t3 = pp[(int64_t)(ch + 6) * st];
            const double t4 = pp[(int64_t)(ch + 8) * st], t5 = pp[(int64_t)(ch + 10) * st];
            const double t6 = pp[(int64_t)(ch + 12) * st], t7 = pp[(int64_t)(ch + 14) * st];
            acc += t0; acc += t1; acc += t2; acc += t3;
            acc += t4; acc += t5; acc += t6; acc += t7;
        }
        for (; ch < nch; ch += 2) acc += pp[(int64_t)ch * st];
        const double o = __shfl_xor(acc, 1, 2);
        const double tot = h ? (o + acc) : (acc + o);
        if (h == 0) p.z3[slot] = ok ? (double)bt - tot : 0.0;
    }
}

// ---------------------------------------------------- three sampled steps --
// The inner loop of Algorithm 1 for outer iteration it: y1, y2, y3 from
// z = b_S - A_S x0 (formed by the last workgroup of the previous kernel), the
// stored inverses H1, H2, H3 and the cross-Grams xg ([3][bmax][bmax], see
// xgram_tile):
//   z_l = b_l - A_l x0;  y1 = H1 z1;  z2 -= G21 y1;  z3 -= G31 y1;
//   y2 = H2 z2;  z3 -= G32 y2;  y3 = H3 z3;
// every workgroup forms the same y (same order), then updates its column slab
// x[cols] += A_S[:, cols]^T y over the rows of all three blocks.
//
// Memory round trips: the draws, then everything else at once.  Thread range
// k = 0, 1, 2 (two waves each, a pair of threads per row; row 64 of the three
// ranges on one more wave, see chain_rows) reads two of the six matrices into
// registers: H1 and H2, G21 and G32, G31 and H3.  Every thread also loads its entries of x and z, and its rows of
// the update once the first matrix's registers are free.  Each stage of the
// chain is then 16-byte LDS reads of a vector, register FMAs, a pair sum by
// DPP and a barrier.
// Chain form (K > 0): the previous iteration's greedy rows I with their y
// join the update, x += A_I^T y_I + sum_l A_l^T y_l, in the same pass (z then
// already accounts for the greedy step, see k_gram_chain).
struct FwdSamp3P {
    const void *A;
    int64_t ld, n, q, rem;
    int bmax;
    const int32_t *tau;
    int64_t tau_index;
    const double *H;
    const double *xg;
    const double *z3;      // z of the three blocks, slots l * FWD_B + i
    void *x;
    int64_t wu;
    const Ctrl *ctrl;
    const int32_t *I;      // chain form: the greedy rows of the previous iteration
    int K;                 // (0: none) and their y, applied in the same pass
    const double *y;
};

// A pair of threads (h = 0, 1) shares a matrix row of at most FWD_B entries:
// thread h takes the entries hb h + t, t < hb, with hb = mv_half(columns), a
// multiple of MG, so that the vector entries it needs are 16-byte LDS reads
// and no group of MG entries needs a bound of its own.
constexpr int MG = 4;
constexpr int MC = ((FWD_B + 1) / 2 + MG - 1) / MG * MG;   // most entries per thread
// (hb of blocks of bmax rows serves those of bmax - 1 too: 2 hb - (bmax - 1) at most)
static_assert(2 * MG <= RORBK_FWD_ZCOLS, "columns read past a stored inverse are its own zeros");
__device__ __forceinline__ int mv_half(int cols) { return ((cols + 1) / 2 + MG - 1) / MG * MG; }
// LDS slots per block of the vectors mv_dot reads; the slots past the block
// hold zeros, which meet whatever finite entries mv_load read past the matrix
constexpr int ZS = 2 * MC;

// The other lane's value of a pair of lanes (2 u, 2 u + 1).
__device__ __forceinline__ double pair_other(double v) {
    const uint64_t u = (uint64_t)__double_as_longlong(v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)u, 0xb1, 0xf, 0xf, false);
    const uint32_t hi =
        (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)(u >> 32), 0xb1, 0xf, 0xf, false);
    return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}

// Entry (i, hb h + t) of a rows x cols matrix stored at M[i + j * sj] into
// m[t] (rows past it get some other row's entries, whose product is not used).
// Up to eight columns past the matrix are read and multiplied by zero: the
// zeros behind each stored inverse, or finite numbers (the next cross-Grams,
// which are cleared at setup where nothing else writes, and RORBK_FWD_PAD
// doubles behind the last).  So a load is an address addition and no select; clamping
// every address cost 6 us for a thread's two matrices, and a select on the
// loaded value made the compiler wait for every load by itself (12 us).
__device__ __forceinline__ void mv_load(const double *__restrict__ M, uint32_t sj, int i, int h,
                                        int rows, int hb, double (&m)[MC]) {
    const double *pm = M + (uint32_t)(i < rows ? i : 0) + (h ? (uint32_t)hb * sj : 0u);
#pragma unroll
    for (int t0 = 0; t0 < MC; t0 += MG)
        if (t0 < hb) {   // uniform
#pragma unroll
            for (int t = t0; t < t0 + MG; ++t) {
                m[t] = *pm;
                pm += sj;
            }
        }
}

// sum_t m[t] vin[hb h + t] over the pair of threads: four accumulators in a
// fixed order, then the pair's sum.
__device__ __forceinline__ double mv_dot(const double (&m)[MC], const double *vin, int h, int hb) {
    const double *v = vin + h * hb;
    double a[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int t0 = 0; t0 < MC; t0 += MG)
        if (t0 < hb) {
            const dvec2 w0 = *reinterpret_cast<const dvec2 *>(v + t0);
            const dvec2 w1 = *reinterpret_cast<const dvec2 *>(v + t0 + 2);
            a[0] = __builtin_fma(m[t0], w0[0], a[0]);
            a[1] = __builtin_fma(m[t0 + 1], w0[1], a[1]);
            a[2] = __builtin_fma(m[t0 + 2], w1[0], a[2]);
            a[3] = __builtin_fma(m[t0 + 3], w1[1], a[3]);
        }
    const double s = (a[0] + a[1]) + (a[2] + a[3]);
    return s + pair_other(s);
}

// Thread range rg (3: none), row i and half h of thread `lane` of wave w: the
// same range over a whole wave for rows below 64, so that the matrices' bases
// and strides are scalars there.
__device__ __forceinline__ void chain_rows(int w, int lane, int *rg, int *i, int *h) {
    *h = lane & 1;
    if (w < 6) {
        *rg = w >> 1;
        *i = 32 * (w & 1) + (lane >> 1);
    } else {
        *rg = (w == 6 && lane < 6) ? lane >> 1 : 3;
        *i = 64;
    }
}

// The two matrices of thread range rg (see above): m for the first two stages
// of the chain, m2 for the last three; H1, H2, H3 are symmetric, the
// cross-Grams column-major.
__device__ __forceinline__ void chain_mats(const double *__restrict__ H,
                                           const double *__restrict__ xg, int64_t hoff0,
                                           int64_t hoff1, int64_t hoff2, int n0, int n1, int n2,
                                           int bm, int rg, int i, int h, int hb, double (&m)[MC],
                                           double (&m2)[MC]) {
    const double *M = H, *M2 = H;
    uint32_t sj = 1, sj2 = 1;
    int rows = 0, rows2 = 0;
    if (rg == 0) {
        M = H + hoff0; sj = n0; rows = n0;                        // H1
        M2 = H + hoff1; sj2 = n1; rows2 = n1;                     // H2
    } else if (rg == 1) {
        M = xg; sj = bm; rows = n1;                               // G21
        M2 = xg + 2 * (int64_t)bm * bm; sj2 = bm; rows2 = n2;     // G32
    } else if (rg == 2) {
        M = xg + (int64_t)bm * bm; sj = bm; rows = n2;            // G31
        M2 = H + hoff2; sj2 = n2; rows2 = n2;                     // H3
    }
    mv_load(M, sj, i, h, rows, hb, m);
    mv_load(M2, sj2, i, h, rows2, hb, m2);
}

// The same for wave w (scalar; see chain_rows): scalar bases where a wave
// holds one range, and the seventh wave only where blocks have a row 64.
__device__ __forceinline__ void chain_mats_wave(const double *__restrict__ H,
                                                const double *__restrict__ xg, int64_t hoff0,
                                                int64_t hoff1, int64_t hoff2, int n0, int n1,
                                                int n2, int bm, int w, int rg, int i, int h, int hb,
                                                double (&m)[MC], double (&m2)[MC]) {
    if (w < 6)
        chain_mats(H, xg, hoff0, hoff1, hoff2, n0, n1, n2, bm, w >> 1, i, h, hb, m, m2);
    else if (w == 6 && bm > 64)
        chain_mats(H, xg, hoff0, hoff1, hoff2, n0, n1, n2, bm, rg, i, h, hb, m, m2);
}

template <typename T, typename V, bool AL, int RN, bool MS>
__global__ __launch_bounds__(FWD_T) void k_fwd_samp3(FwdSamp3P p) {
    constexpr int VW = Tr<T>::VW;
    constexpr int SWC = fwd_swc<T>();
    constexpr int NV = SWC / VW;
    constexpr int G = FWD_T / NV;
    const T *__restrict__ A = (const T *)p.A;
    V *__restrict__ x = (V *)p.x;
    const int tid = threadIdx.x, g = tid / NV, v = tid % NV;
    Blk3 B;
    blocks3(p.tau, p.tau_index, p.q, p.rem, B);
    const int64_t hoff0 = blk_hoff(p.tau[p.tau_index], p.q, p.rem, RORBK_FWD_ZCOLS);
    const int64_t hoff1 = blk_hoff(p.tau[p.tau_index + 1], p.q, p.rem, RORBK_FWD_ZCOLS);
    const int64_t hoff2 = blk_hoff(p.tau[p.tau_index + 2], p.q, p.rem, RORBK_FWD_ZCOLS);
    const int ncnt = B.c0 + B.c1 + B.c2;
    const int bm = p.bmax;
    const int n0 = B.c0, n1 = B.c1, n2 = B.c2;
    if (p.ctrl->done) return;
    const int64_t c0 = (int64_t)blockIdx.x * p.wu;
    const int64_t c1 = (c0 + p.wu < p.n) ? c0 + p.wu : p.n;
    const int wcols = (int)(c1 - c0);

    __shared__ V s_x[1024];
    __shared__ V s_red[G][SWC];
    __shared__ __align__(16) double s_z[3 * ZS], s_y[3 * ZS + 64];
    static_assert(64 + 3 * FWD_B <= FWD_T, "one row-table entry per thread");
    __shared__ int32_t s_row[64 + 3 * FWD_B], s_slot[64 + 3 * FWD_B];
    const int K = p.K;

    // --- every load of the kernel, in the order the data is needed
    V xv[(1024 + FWD_T - 1) / FWD_T];
#pragma unroll
    for (int u = 0; u < (1024 + FWD_T - 1) / FWD_T; ++u) {
        const int c = tid + u * FWD_T;
        const V t = x[c0 + (c < wcols ? c : 0)];
        xv[u] = (c < wcols) ? t : (V)0;
    }
    const int zl = tid / ZS, zi = tid - zl * ZS;   // slot of z (l, i), padded with zeros
    const bool zok = zl < 3 && zi < FWD_B;
    const double zt = p.z3[zok ? zl * FWD_B + zi : 0];
    const double zv = zok ? zt : 0.0;
    // chain form: the greedy rows and their y (uniform branch)
    int32_t iv = 0;
    double ygv = 0.0;
    if (K > 0) {
        iv = p.I[tid < K ? tid : 0];
        ygv = p.y[tid < K ? tid : 0];
    }
    // two matrices per thread range (H symmetric, read along its rows)
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    int rg, ir, h;
    chain_rows(wv, tid & 63, &rg, &ir, &h);
    const int hb = mv_half(bm);
    double m[MC], m2[MC];
    chain_mats_wave(p.H, p.xg, hoff0, hoff1, hoff2, n0, n1, n2, bm, wv, rg, ir, h, hb, m, m2);
    // row r of this thread's share of the update: its index in A (row 0
    // stands in past the last row) and its slot in s_y, read from the LDS
    // tables each time it is needed (volatile: not held in registers across
    // the chain).  The greedy rows come first.
    const int nrows = K + ncnt;
    auto urow = [&](int r, int64_t *row, int *slot) -> bool {
        const int qq = g + G * r;
        const bool ok = qq < nrows;
        *row = ok ? (int64_t)((volatile int32_t *)s_row)[qq] : 0;
        *slot = ok ? ((volatile int32_t *)s_slot)[qq] : 0;
        return ok;
    };

    // --- z = b_S - A_S x0 (slots l * FWD_B + i; s_y zeroed)
#pragma unroll
    for (int u = 0; u < (1024 + FWD_T - 1) / FWD_T; ++u) {
        const int c = tid + u * FWD_T;
        if (c < wcols) s_x[c] = xv[u];
    }
    if (tid < 3 * ZS) {
        s_z[tid] = zv;
        s_y[tid] = 0.0;
    }
    if (tid < K) s_y[3 * ZS + tid] = ygv;
    // the row tables of the update: entry tid (fewer than FWD_T rows)
    if (tid < nrows) {
        int l, i;
        int64_t r3;
        split3(B, tid >= K ? tid - K : 0, &l, &i, &r3);
        s_row[tid] = (tid < K) ? iv : (int32_t)r3;
        s_slot[tid] = (tid < K) ? 3 * ZS + tid : l * ZS + i;
    }
    __syncthreads();
    // y1 = H1 z1
    if (rg == 0) {
        const double d = mv_dot(m, s_z, h, hb);
        if (h == 0 && ir < n0) s_y[ir] = d;
    }
    __syncthreads();
    // z2 -= G21 y1 and z3 -= G31 y1
    if (rg == 1 || rg == 2) {
        const double d = mv_dot(m, s_y, h, hb);
        const int rows = (rg == 1) ? n1 : n2;
        if (h == 0 && ir < rows) s_z[rg * ZS + ir] -= d;
    }
    // the rows of the update (first sub-slab) load during the rest of the
    // chain, once the registers of the first half are free
    uvec4 ua[RN];
    {
        const int64_t col = c0 + (int64_t)v * VW;
#pragma unroll
        for (int r = 0; r < RN; ++r) {
            int64_t row;
            int slot;
            const bool ok = urow(r, &row, &slot);
            ua[r] = load_raw_sel<T, AL>(A + row * p.ld, col, c1, ok, A, c0);
        }
    }
    __syncthreads();
    // y2 = H2 z2
    if (rg == 0) {
        const double d = mv_dot(m2, s_z + ZS, h, hb);
        if (h == 0 && ir < n1) s_y[ZS + ir] = d;
    }
    __syncthreads();
    // z3 -= G32 y2
    if (rg == 1) {
        const double d = mv_dot(m2, s_y + ZS, h, hb);
        if (h == 0 && ir < n2) s_z[2 * ZS + ir] -= d;
    }
    __syncthreads();
    // y3 = H3 z3
    if (rg == 2) {
        const double d = mv_dot(m2, s_z + 2 * ZS, h, hb);
        if (h == 0 && ir < n2) s_y[2 * ZS + ir] = d;
    }
    __syncthreads();

    // --- x[cols] += A_S[:, cols]^T y
    V yv[RN];
#pragma unroll
    for (int r = 0; r < RN; ++r) {
        int64_t row;
        int slot;
        const bool ok = urow(r, &row, &slot);
        yv[r] = ok ? (V)s_y[slot] : (V)0;
    }
    constexpr bool PF = MS && RN <= 5;
    constexpr int RP = PF ? RN : 1;
    for (int64_t sub = c0; sub < c1; sub += SWC) {
        const int64_t col = sub + (int64_t)v * VW;
        const bool more = sub + SWC < c1;   // uniform
        uvec4 ua2[RP];
        if constexpr (PF) {
            if (more) {
                const int64_t coln = col + SWC;
#pragma unroll
                for (int r = 0; r < RN; ++r) {
                    int64_t row;
                    int slot;
                    const bool ok = urow(r, &row, &slot);
                    ua2[r] = load_raw_sel<T, AL>(A + row * p.ld, coln, c1, ok, A, c0);
                }
            }
        } else if (sub != c0) {
#pragma unroll
            for (int r = 0; r < RN; ++r) {
                int64_t row;
                int slot;
                const bool ok = urow(r, &row, &slot);
                ua[r] = load_raw_sel<T, AL>(A + row * p.ld, col, c1, ok, A, c0);
            }
        }
        V acc[VW];
#pragma unroll
        for (int e = 0; e < VW; ++e) acc[e] = (V)0;
#pragma unroll
        for (int r = 0; r < RN; ++r) {
            V a[VW];
            cvt_raw<T, V>(ua[r], a);
#pragma unroll
            for (int e = 0; e < VW; ++e) acc[e] = fmaT(a[e], yv[r], acc[e]);
        }
#pragma unroll
        for (int e = 0; e < VW; ++e) s_red[g][v * VW + e] = acc[e];
        __syncthreads();
        if (tid < SWC) {
            const int64_t cc = sub + tid;
            if (cc < c1) {
                V s = (V)0;
                for (int gg = 0; gg < G; ++gg) s += s_red[gg][tid];
                s_x[cc - c0] += s;
            }
        }
        __syncthreads();
        if constexpr (PF) {
            if (more) {
#pragma unroll
                for (int r = 0; r < RN; ++r) ua[r] = ua2[r];
            }
        }
    }
    for (int c = tid; c < wcols; c += FWD_T) x[c0 + c] = s_x[c];
}

// ------------------------------------------------------- chain step kernel --
// The rest of iteration it after the chain form's Grams (k_gram_chain), in one
// launch over the column slabs (one sub-slab each): in every workgroup wave 0
// solves the greedy system (G + lambda I) y = r_I (ldl_blk64 on the summed
// Gram chunks; every workgroup forms the same y) while waves 1-7 sum C and
// load the three sampled steps' matrices into registers and LDS, so that
// their memory latency is spent during the factorisation.  Then
// z = r_{S'} - C y (entries of even and odd j summed by the two threads of a
// pair), the chain of k_fwd_samp3 with the same
// arithmetic (the same thread of a row pair, the same sums), and
// x[cols] += A_I[:, cols]^T y + sum_l A_l[:, cols]^T y_l in one pass.  The
// first workgroup writes y and, for a checkpoint, the chain state (I, y, z).
//
// What bounds it: the chain Gram load (2.3 us), factorisation, z, six small
// products, update; and beside the factorisation the loads of waves 1-7, which
// have to end with it (16 workgroups each read the six b x b matrices and C:
// 0.4 MB at b = K = 64 with C in two column chunks).  With the factorisation
// at 6 to 8 us the loads decided, so they are spread as many as the registers
// hold (a select or a clamped address per load cost more than the memory) and
// C comes in at most two chunks (four made the Grams 0.8 us faster and this
// kernel 6 us slower at 2000 columns).  Per launch, kernel trace: 100000 x 2000,
// b = 64: 23.1 us (28.6); 20000 x 1000, b = 50: 18.3 us (26); 2000 x 200, b = 20:
// 11.0 us (20.5).
struct FwdChainP {
    const void *A;
    int64_t ld, n, q, rem;
    int bmax;
    const int32_t *tau;
    int64_t tau_index;     // first draw of iteration it + 1
    const double *H;
    const double *xg;      // cross-Grams of iteration it + 1's blocks
    const double *G;       // [nch][K (K + 1) / 2] packed lower partials
    const double *C;       // [nch][64][3 * FWD_B] partials
    int nch;
    int K;
    double lambda;
    const double *rI;
    const void *r;         // residual of iteration it (vector type)
    const int32_t *I;
    void *x;
    int64_t wu;            // columns per workgroup (one sub-slab)
    double *y;
    double *ckst;          // NULL, or a checkpoint's chain state
    Ctrl *ctrl;
};

constexpr int CHN = 2;                       // most column chunks of G and C
constexpr int FC_T = FWD_T - 64;             // threads of waves 1-7
constexpr int LA = LB_LEN;                   // LDS doubles of region a

template <typename T, typename V, bool AL, int RN>
__global__ __launch_bounds__(FWD_T) void k_fwd_chain(FwdChainP p) {
    constexpr int VW = Tr<T>::VW;
    constexpr int SWC = fwd_swc<T>();
    constexpr int NV = SWC / VW;
    constexpr int G = FWD_T / NV;
    static_assert(1024 + G * SWC * sizeof(V) / 8 <= LA, "phase-2 arrays fit the factorisation's LDS");
    static_assert(2 * CHAIN_S <= FC_T, "two threads per row of C");
    // the update's rows travel as soon as C is summed where the registers hold
    // both, else after z; entries of C's chunks in flight per thread
    constexpr bool EARLY = RN <= 13;
    constexpr int CU = (RN == 13) ? 8 : 16;
    static_assert(3 * ZS <= 256 && 256 + 3 * ZS + 64 <= 1024, "z, y and the row sums side by side");
    const T *__restrict__ A = (const T *)p.A;
    V *__restrict__ x = (V *)p.x;
    const int tid = threadIdx.x;
    const int K = p.K, KP = K * (K + 1) / 2;
    // LDS: region a holds the factorisation (the padded system, then its
    // tiles), then z, y and the update's row sums; s_m2 keeps each thread's
    // entries of its second matrix while C needs the registers
    __shared__ __align__(16) double lds_a[LA];
    __shared__ __align__(16) double s_yk[64];
    __shared__ double s_m2[MC][6 * 64 + 8];
    __shared__ V s_x[SWC];
    __shared__ int32_t s_row[64 + 3 * FWD_B], s_slot[64 + 3 * FWD_B];
    __shared__ int s_ok, s_stop;
    double *Lc = lds_a;
    double *s_z = lds_a, *s_y = lds_a + 256;
    V (*s_red)[SWC] = reinterpret_cast<V (*)[SWC]>(lds_a + 1024);

    // the draws (scalar loads) travel with the first vector loads.  The stop
    // flag takes effect behind the first barrier, as wave 0 read it: another
    // workgroup whose factorisation failed may set it meanwhile, and waves that
    // disagreed would leave the row tables below unwritten for the others.
    // (What is loaded before does not depend on it.)
    const int stop = __hip_atomic_load(&p.ctrl->done, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    Blk3 B;
    blocks3(p.tau, p.tau_index, p.q, p.rem, B);
    const int bm = p.bmax, n0 = B.c0, n1 = B.c1, n2 = B.c2;
    const int ncnt = n0 + n1 + n2, nrows = K + ncnt;
    const int64_t c0 = (int64_t)blockIdx.x * p.wu;
    const int64_t c1 = (c0 + p.wu < p.n) ? c0 + p.wu : p.n;
    const int wcols = (int)(c1 - c0);

    // the Gram chunks and r_I: every thread loads its packed entries, sums
    // them in chunk order and puts them into the padded system (lambda on the
    // diagonal, the identity beyond K)
    constexpr int NU0 = (64 * 65 / 2 + FWD_T - 1) / FWD_T;
    double gt[CHN][NU0];
    double ri;
    auto load_gram = [&]() {
        ri = p.rI[tid < K ? tid : 0];
#pragma unroll
        for (int c = 0; c < CHN; ++c)
            if (c < p.nch) {   // uniform
#pragma unroll
                for (int u = 0; u < NU0; ++u) {
                    const int f = tid + u * FWD_T;
                    gt[c][u] = p.G[c * KP + (f < KP ? f : 0)];
                }
            } else {
#pragma unroll
                for (int u = 0; u < NU0; ++u) gt[c][u] = 0.0;
            }
    };
    auto put_gram = [&]() {
#pragma unroll
        for (int u = 0; u < NU0; ++u) {
            const int f = tid + u * FWD_T;
            double gs = gt[0][u];
#pragma unroll
            for (int c = 1; c < CHN; ++c)
                if (c < p.nch) gs += gt[c][u];
            if (f < 64 * 65 / 2) lb_put(Lc, f, gs, K, p.lambda);
        }
        if (tid < 64) s_yk[tid] = (tid < K) ? ri : 0.0;
    };

    // the update's rows g + G r, r < RN, from the tables: every row index
    // first (LDS), then every load (row 0 stands in past the last row, where
    // y is 0)
    const int g = tid / NV, v = tid % NV;
    uvec4 ua[RN];
    auto load_rows = [&]() {
        const int64_t col = c0 + (int64_t)v * VW;
        int32_t rw[RN];
#pragma unroll
        for (int r = 0; r < RN; ++r) {
            const int qq = g + G * r;
            rw[r] = (qq < nrows) ? s_row[qq] : 0;
        }
        if (AL && c0 + SWC <= p.n) {   // uniform: no column past the matrix
#pragma unroll
            for (int r = 0; r < RN; ++r)
                ua[r] = *reinterpret_cast<const uvec4 *>(A + (int64_t)rw[r] * p.ld + col);
        } else {
#pragma unroll
            for (int r = 0; r < RN; ++r)
                ua[r] = load_raw_sel<T, AL>(A + (int64_t)rw[r] * p.ld, col, c1, true, A, c0);
        }
    };

    // --- phase 1: wave 0 factors while waves 1-7 load everything else (the
    // wave index is made scalar so that both branches are real jumps; each
    // branch meets the same two barriers)
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int t = tid - 64;
    int rg, ir, h;
    chain_rows(wv - 1, tid & 63, &rg, &ir, &h);
    const int hb = mv_half(bm);
    // thread pair cs holds row cs of C, thread ch of it the entries ch kb + u
    const int ts = t < 6 * 64 + 8 ? t : 6 * 64 + 7;   // (threads past it hold no matrix)
    const int cs = t >> 1, ch = t & 1, kb = mv_half(K);
    double m[MC], cv[32];
    double rsv = 0.0;
    bool rok = false;
    if (wv == 0) {
        load_gram();
        put_gram();
        if (tid == 0) s_stop = stop;
        __syncthreads();
        if (s_stop) return;
        // (this wave's chain comes first on its SIMD)
        __builtin_amdgcn_s_setprio(3);
        const bool ok = ldl_blk64(Lc, s_yk, K);
        __builtin_amdgcn_s_setprio(0);
        if (tid == 0) {
            s_ok = ok ? 1 : 0;
            if (!ok) {
                p.ctrl->status = RORBK_ERR_NOT_SPD;
                p.ctrl->done = 1;
            }
        }
        __syncthreads();
    } else {
        load_gram();
        // r at the next blocks' rows, the greedy rows, the slab of x
        V rr = (V)0;
        if (cs < CHAIN_S) {
            const int l = cs / FWD_B, i = cs - l * FWD_B;
            const int cl = (l == 0) ? n0 : ((l == 1) ? n1 : n2);
            const int64_t st = (l == 0) ? B.s0 : ((l == 1) ? B.s1 : B.s2);
            rok = i < cl;
            rr = ((const V *)p.r)[st + (rok ? i : 0)];
        }
        const int32_t iv = p.I[t < K ? t : 0];
        const V xv = x[c0 + (t < wcols ? t : 0)];
        put_gram();
        if (t < nrows) {   // the update's row tables, greedy rows first
            int l, i;
            int64_t r3;
            split3(B, t >= K ? t - K : 0, &l, &i, &r3);
            s_row[t] = (t < K) ? iv : (int32_t)r3;
            s_slot[t] = (t < K) ? 3 * ZS + t : l * ZS + i;
        }
        __syncthreads();
        if (s_stop) return;
        // the sampled steps' matrices (two per thread range, as k_fwd_samp3)
        double m2[MC];
        {
            const int64_t hoff0 = blk_hoff(p.tau[p.tau_index], p.q, p.rem, RORBK_FWD_ZCOLS);
            const int64_t hoff1 = blk_hoff(p.tau[p.tau_index + 1], p.q, p.rem, RORBK_FWD_ZCOLS);
            const int64_t hoff2 = blk_hoff(p.tau[p.tau_index + 2], p.q, p.rem, RORBK_FWD_ZCOLS);
            chain_mats_wave(p.H, p.xg, hoff0, hoff1, hoff2, n0, n1, n2, bm, wv - 1, rg, ir, h, hb,
                            m, m2);
        }
        // C summed over its chunks, CU entries of every chunk in flight
        // (all of them lie inside C, whose rows run to 64 and which was
        // cleared at setup; entries at or past K meet zeros of y); the second
        // matrix goes to LDS while the first of them travel
        const double *pc = p.C + (cs < CHAIN_S ? cs : 0) + ch * kb * CHAIN_S;
#pragma unroll
        for (int u0 = 0; u0 < 32; u0 += CU) {
            if (u0 < kb) {   // uniform
                double ct[CHN][CU];
#pragma unroll
                for (int c = 0; c < CHN; ++c)
                    if (c < p.nch) {
#pragma unroll
                        for (int u = 0; u < CU; ++u) ct[c][u] = pc[c * CHAIN_C + (u0 + u) * CHAIN_S];
                    }
#pragma unroll
                for (int u = 0; u < CU; ++u) {
                    double sum = ct[0][u];
#pragma unroll
                    for (int c = 1; c < CHN; ++c)
                        if (c < p.nch) sum += ct[c][u];
                    cv[u0 + u] = sum;
                }
                if (u0 == 0) {
#pragma unroll
                    for (int e0 = 0; e0 < MC; e0 += MG)
                        if (e0 < hb) {
#pragma unroll
                            for (int e = e0; e < e0 + MG; ++e) s_m2[e][ts] = m2[e];
                        }
                }
            }
        }
        rsv = rok ? (double)rr : 0.0;
        if (t < wcols) s_x[t] = xv;
        if constexpr (EARLY) load_rows();
        __syncthreads();
    }
    if (!s_ok) return;
    if constexpr (EARLY) {
        if (wv == 0) load_rows();
    }

    // --- phase 2: z = r_{S'} - C y, then the chain
    if (wv != 0) {
        const double *yk = s_yk + ch * kb;
        double acc = 0.0;
#pragma unroll
        for (int u0 = 0; u0 < 32; u0 += MG)
            if (u0 < kb) {
                const dvec2 w0 = *reinterpret_cast<const dvec2 *>(yk + u0);
                const dvec2 w1 = *reinterpret_cast<const dvec2 *>(yk + u0 + 2);
                acc = __builtin_fma(cv[u0], w0[0], acc);
                acc = __builtin_fma(cv[u0 + 1], w0[1], acc);
                acc = __builtin_fma(cv[u0 + 2], w1[0], acc);
                acc = __builtin_fma(cv[u0 + 3], w1[1], acc);
            }
        const double o = pair_other(acc);
        if (ch == 0 && cs < CHAIN_S) {
            const double zz = rok ? rsv - (acc + o) : 0.0;
            const int l = cs / FWD_B, i = cs - l * FWD_B;
            s_z[l * ZS + i] = zz;
            s_y[l * ZS + i] = 0.0;
            if (blockIdx.x == 0 && p.ckst) p.ckst[96 + cs] = zz;
        }
    } else if (tid < 3 * (ZS - FWD_B)) {
        // the slots past each block
        const int l = tid / (ZS - FWD_B), i = FWD_B + tid - l * (ZS - FWD_B);
        s_z[l * ZS + i] = 0.0;
        s_y[l * ZS + i] = 0.0;
    }
    if (tid < K) {
        s_y[3 * ZS + tid] = s_yk[tid];
        if (blockIdx.x == 0) {
            p.y[tid] = s_yk[tid];
            if (p.ckst) {
                reinterpret_cast<int32_t *>(p.ckst)[tid] = s_row[tid];
                p.ckst[32 + tid] = s_yk[tid];
            }
        }
    }
    __syncthreads();
    if constexpr (!EARLY) load_rows();
    // this thread's second matrix, once the first is used
    auto second = [&]() {
#pragma unroll
        for (int e0 = 0; e0 < MC; e0 += MG)
            if (e0 < hb) {
#pragma unroll
                for (int e = e0; e < e0 + MG; ++e) m[e] = s_m2[e][ts];
            }
    };
    // y1 = H1 z1
    if (wv != 0 && rg == 0) {
        const double d = mv_dot(m, s_z, h, hb);
        if (h == 0 && ir < n0) s_y[ir] = d;
        second();
    }
    __syncthreads();
    // z2 -= G21 y1 and z3 -= G31 y1
    if (wv != 0 && (rg == 1 || rg == 2)) {
        const double d = mv_dot(m, s_y, h, hb);
        const int rows = (rg == 1) ? n1 : n2;
        if (h == 0 && ir < rows) s_z[rg * ZS + ir] -= d;
        second();
    }
    __syncthreads();
    // y2 = H2 z2
    if (wv != 0 && rg == 0) {
        const double d = mv_dot(m, s_z + ZS, h, hb);
        if (h == 0 && ir < n1) s_y[ZS + ir] = d;
    }
    __syncthreads();
    // z3 -= G32 y2
    if (wv != 0 && rg == 1) {
        const double d = mv_dot(m, s_y + ZS, h, hb);
        if (h == 0 && ir < n2) s_z[2 * ZS + ir] -= d;
    }
    __syncthreads();
    // y3 = H3 z3
    if (wv != 0 && rg == 2) {
        const double d = mv_dot(m, s_z + 2 * ZS, h, hb);
        if (h == 0 && ir < n2) s_y[2 * ZS + ir] = d;
    }
    __syncthreads();

    // --- x[cols] += A_I^T y + sum_l A_l^T y_l (one sub-slab)
    V acc[VW];
#pragma unroll
    for (int e = 0; e < VW; ++e) acc[e] = (V)0;
    {
        // the slots, then their y, then the products (no LDS read waits on
        // another inside the loop)
        int32_t sl[RN];
#pragma unroll
        for (int r = 0; r < RN; ++r) {
            const int qq = g + G * r;
            sl[r] = (qq < nrows) ? s_slot[qq] : -1;
        }
        V yv[RN];
#pragma unroll
        for (int r = 0; r < RN; ++r) yv[r] = (sl[r] >= 0) ? (V)s_y[sl[r] >= 0 ? sl[r] : 0] : (V)0;
#pragma unroll
        for (int r = 0; r < RN; ++r) {
            V av[VW];
            cvt_raw<T, V>(ua[r], av);
#pragma unroll
            for (int e = 0; e < VW; ++e) acc[e] = fmaT(av[e], yv[r], acc[e]);
        }
    }
#pragma unroll
    for (int e = 0; e < VW; ++e) s_red[g][v * VW + e] = acc[e];
    __syncthreads();
    if (tid < wcols) {
        V sx = (V)0;
        for (int gg = 0; gg < G; ++gg) sx += s_red[gg][tid];
        x[c0 + tid] = s_x[tid] + sx;
    }
}

// ------------------------------------------------------------ launchers --
// Size class of the per-thread row counts: rows of one block (RC) and of
// three (RN) per thread for G row groups.
template <typename T>
constexpr int fwd_groups() { return FWD_T / (fwd_swc<T>() / Tr<T>::VW); }

static int fwd_class(int bmax, int G) {
    const int rc = (bmax + G - 1) / G, rn = (3 * bmax + G - 1) / G;
    if (rc <= 2 && rn <= 4) return 0;
    if (rc <= 3 && rn <= 8) return 1;
    return 2;   // rc <= 5, rn <= 13: FWD_B = 65 rows over 16 or 32 row groups
}

template <typename T, typename V, bool AL, bool MS>
static hipError_t greedy_launch_cls(const FwdGreedyP &p, int nblk, int cls, hipStream_t s) {
    switch (cls) {
    case 0: hipLaunchKernelGGL((k_fwd_greedy<T, V, AL, 2, 4, MS>), dim3(nblk), dim3(FWD_T), 0, s, p); break;
    case 1: hipLaunchKernelGGL((k_fwd_greedy<T, V, AL, 3, 8, MS>), dim3(nblk), dim3(FWD_T), 0, s, p); break;
    default: hipLaunchKernelGGL((k_fwd_greedy<T, V, AL, 5, 13, MS>), dim3(nblk), dim3(FWD_T), 0, s, p); break;
    }
    return hipGetLastError();
}

// rows of the update per thread (the three blocks and, in the chain form,
// the greedy rows): 4, 8, 13 or 17
template <typename T, typename V, bool AL, bool MS>
static hipError_t samp3_launch_rn(const FwdSamp3P &p, int nblk, int bmax, hipStream_t s) {
    constexpr int G = fwd_groups<T>();
    const int rn = (3 * bmax + p.K + G - 1) / G;
    if (rn <= 4)
        hipLaunchKernelGGL((k_fwd_samp3<T, V, AL, 4, MS>), dim3(nblk), dim3(FWD_T), 0, s, p);
    else if (rn <= 8)
        hipLaunchKernelGGL((k_fwd_samp3<T, V, AL, 8, MS>), dim3(nblk), dim3(FWD_T), 0, s, p);
    else if (rn <= 13)
        hipLaunchKernelGGL((k_fwd_samp3<T, V, AL, 13, MS>), dim3(nblk), dim3(FWD_T), 0, s, p);
    else
        hipLaunchKernelGGL((k_fwd_samp3<T, V, AL, 17, MS>), dim3(nblk), dim3(FWD_T), 0, s, p);
    return hipGetLastError();
}

template <typename T, typename V>
static hipError_t fwd_greedy_typed(const rorbk_handle_s *h, const FwdArgs &a, hipStream_t s) {
    const Layout &L = h->L;
    FwdGreedyP p;
    p.A = a.A;
    p.ld = L.ld;
    p.n = L.n;
    p.q = L.q;
    p.rem = L.rem;
    p.bmax = (int)L.bmax;
    p.tau = h->d_tau;
    p.tau_next = a.tau_index;
    p.I = a.I;
    p.K = (int)L.K;
    p.y = a.y;
    p.x = a.x;
    p.Pout = h->d_P3;
    p.wu = L.wf;
    p.ctrl = h->d_ctrl;
    p.b = a.b;
    p.z3 = h->d_z3;
    p.counter = h->d_fwdcnt;
    const int cls = fwd_class((int)L.bmax, fwd_groups<T>());
    const bool ms = L.wf > fwd_swc<T>();
    if (a.aligned) {
        if (ms) return greedy_launch_cls<T, V, true, true>(p, L.nch_f, cls, s);
        return greedy_launch_cls<T, V, true, false>(p, L.nch_f, cls, s);
    }
    if (ms) return greedy_launch_cls<T, V, false, true>(p, L.nch_f, cls, s);
    return greedy_launch_cls<T, V, false, false>(p, L.nch_f, cls, s);
}

template <typename T, typename V>
static hipError_t fwd_samp3_typed(const rorbk_handle_s *h, const FwdArgs &a, hipStream_t s) {
    const Layout &L = h->L;
    FwdSamp3P p;
    p.A = a.A;
    p.ld = L.ld;
    p.n = L.n;
    p.q = L.q;
    p.rem = L.rem;
    p.bmax = (int)L.bmax;
    p.tau = h->d_tau;
    p.tau_index = a.tau_index;
    p.H = h->d_H;
    p.xg = a.xg;
    p.z3 = h->d_z3;
    p.x = a.x;
    p.wu = L.wf;
    p.ctrl = h->d_ctrl;
    p.I = a.I;
    p.K = a.I ? (int)L.K : 0;
    p.y = a.y;
    const int bm = (int)L.bmax;
    const bool ms = L.wf > fwd_swc<T>();
    if (a.aligned) {
        if (ms) return samp3_launch_rn<T, V, true, true>(p, L.nch_f, bm, s);
        return samp3_launch_rn<T, V, true, false>(p, L.nch_f, bm, s);
    }
    if (ms) return samp3_launch_rn<T, V, false, true>(p, L.nch_f, bm, s);
    return samp3_launch_rn<T, V, false, false>(p, L.nch_f, bm, s);
}

hipError_t launch_fwd_greedy(const rorbk_handle_s *h, const FwdArgs &a, hipStream_t s) {
    if (a.vec == VEC_F64) return fwd_greedy_typed<double, double>(h, a, s);
    if (a.dt == RORBK_F32) return fwd_greedy_typed<float, float>(h, a, s);
    return fwd_greedy_typed<bf16_t, float>(h, a, s);
}

hipError_t launch_fwd_samp3(const rorbk_handle_s *h, const FwdArgs &a, hipStream_t s) {
    if (a.vec == VEC_F64) return fwd_samp3_typed<double, double>(h, a, s);
    if (a.dt == RORBK_F32) return fwd_samp3_typed<float, float>(h, a, s);
    return fwd_samp3_typed<bf16_t, float>(h, a, s);
}

template <typename T, int NW>
static hipError_t xgram_typed(const rorbk_handle_s *h, const void *A, int aligned, int64_t ti,
                              double *out, hipStream_t s) {
    const Layout &L = h->L;
    const int jobs = xgram_jobs((int)L.bmax);
    if (aligned)
        hipLaunchKernelGGL((k_xgram<T, true, NW>), dim3(jobs), dim3(64 * NW), 0, s, (const T *)A,
                           L.ld, L.n, h->d_tau, ti, L.q, L.rem, (int)L.bmax, out,
                           (const Ctrl *)h->d_ctrl);
    else
        hipLaunchKernelGGL((k_xgram<T, false, NW>), dim3(jobs), dim3(64 * NW), 0, s,
                           (const T *)A, L.ld, L.n, h->d_tau, ti, L.q, L.rem, (int)L.bmax, out,
                           (const Ctrl *)h->d_ctrl);
    return hipGetLastError();
}

// waves: 4 (stand-alone starts, the residual's spare workgroups) or 8 (the
// selection's spare workgroups; the same sums when a chained solve resumes)
hipError_t launch_xgram(const rorbk_handle_s *h, const void *A, int dt, int aligned, int64_t ti,
                        double *out, int waves, hipStream_t s) {
    if (waves == 8) {
        if (dt == RORBK_F64) return xgram_typed<double, 8>(h, A, aligned, ti, out, s);
        if (dt == RORBK_F32) return xgram_typed<float, 8>(h, A, aligned, ti, out, s);
        return xgram_typed<bf16_t, 8>(h, A, aligned, ti, out, s);
    }
    if (dt == RORBK_F64) return xgram_typed<double, 4>(h, A, aligned, ti, out, s);
    if (dt == RORBK_F32) return xgram_typed<float, 4>(h, A, aligned, ti, out, s);
    return xgram_typed<bf16_t, 4>(h, A, aligned, ti, out, s);
}

int fwd_xgram_jobs(int bmax) { return xgram_jobs(bmax); }

template <typename T, typename V, bool AL>
static hipError_t fwd_chain_rn(const FwdChainP &p, int nblk, hipStream_t s) {
    constexpr int G = fwd_groups<T>();
    const int rn = (3 * p.bmax + p.K + G - 1) / G;
    if (rn <= 4)
        hipLaunchKernelGGL((k_fwd_chain<T, V, AL, 4>), dim3(nblk), dim3(FWD_T), 0, s, p);
    else if (rn <= 8)
        hipLaunchKernelGGL((k_fwd_chain<T, V, AL, 8>), dim3(nblk), dim3(FWD_T), 0, s, p);
    else if (rn <= 13)
        hipLaunchKernelGGL((k_fwd_chain<T, V, AL, 13>), dim3(nblk), dim3(FWD_T), 0, s, p);
    else
        hipLaunchKernelGGL((k_fwd_chain<T, V, AL, 17>), dim3(nblk), dim3(FWD_T), 0, s, p);
    return hipGetLastError();
}

template <typename T, typename V>
static hipError_t fwd_chain_typed(const rorbk_handle_s *h, const FwdArgs &a, const void *r,
                                  double *ckst, hipStream_t s) {
    const Layout &L = h->L;
    if (L.wf != fwd_swc<T>() || L.K > 64 || L.bmax > FWD_B || L.nch_c < 1 || L.nch_c > CHN)
        return hipErrorInvalidValue;   // one sub-slab per workgroup, the chain form's sizes
    FwdChainP p;
    p.A = a.A;
    p.ld = L.ld;
    p.n = L.n;
    p.q = L.q;
    p.rem = L.rem;
    p.bmax = (int)L.bmax;
    p.tau = h->d_tau;
    p.tau_index = a.tau_index;
    p.H = h->d_H;
    p.xg = a.xg;
    p.G = h->d_G;
    p.C = h->d_C;
    p.nch = L.nch_c;
    p.K = (int)L.K;
    p.lambda = h->lambda;
    p.rI = h->d_rI;
    p.r = r;
    p.I = a.I;
    p.x = a.x;
    p.wu = L.wf;
    p.y = h->d_y;
    p.ckst = ckst;
    p.ctrl = h->d_ctrl;
    if (a.aligned) return fwd_chain_rn<T, V, true>(p, L.nch_f, s);
    return fwd_chain_rn<T, V, false>(p, L.nch_f, s);
}

hipError_t launch_fwd_chain(const rorbk_handle_s *h, const FwdArgs &a, const void *r,
                            double *ckst, hipStream_t s) {
    if (a.vec == VEC_F64) return fwd_chain_typed<double, double>(h, a, r, ckst, s);
    if (a.dt == RORBK_F32) return fwd_chain_typed<float, float>(h, a, r, ckst, s);
    return fwd_chain_typed<bf16_t, float>(h, a, r, ckst, s);
}

template <typename T>
static hipError_t gram_chain_typed(const rorbk_handle_s *h, const GramChainP &p, int aligned,
                                   hipStream_t s) {
    const int jobs = gram_chain_tiles(p.K, p.bmax) * h->L.nch_c;
    if (aligned)
        hipLaunchKernelGGL((k_gram_chain<T, true>), dim3(jobs), dim3(64 * GC_W), 0, s, p);
    else
        hipLaunchKernelGGL((k_gram_chain<T, false>), dim3(jobs), dim3(64 * GC_W), 0, s, p);
    return hipGetLastError();
}

hipError_t launch_gram_chain(const rorbk_handle_s *h, const void *A, int dt, int aligned,
                             const int32_t *I, int64_t ti, double *G, hipStream_t s) {
    const Layout &L = h->L;
    if (L.K > 64 || L.bmax > FWD_B || !h->d_C) return hipErrorInvalidValue;
    GramChainP p;
    p.A = A;
    p.ld = L.ld;
    p.n = L.n;
    p.q = L.q;
    p.rem = L.rem;
    p.bmax = (int)L.bmax;
    p.I = I;
    p.K = (int)L.K;
    p.tau = h->d_tau;
    p.ti = ti;
    p.wc = L.wc;
    p.G = G;
    p.C = h->d_C;
    p.ctrl = h->d_ctrl;
    if (dt == RORBK_F64) return gram_chain_typed<double>(h, p, aligned, s);
    if (dt == RORBK_F32) return gram_chain_typed<float>(h, p, aligned, s);
    return gram_chain_typed<bf16_t>(h, p, aligned, s);
}

}  // namespace rorbk
