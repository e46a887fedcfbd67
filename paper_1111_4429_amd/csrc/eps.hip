// Dielectric matrix epsilon = 1 - v chi (epsilon section, dielectric-matrix
// equation, asymmetric Coulomb form) and its inverse.
//
// The paper inverts with LU + solve (ZGESV).  Here the inverse is formed by
// blocked Gauss-Jordan elimination with partial pivoting, in place: it uses
// the same pivot sequence as LU with partial pivoting (largest |Re|+|Im| in
// the current column among the rows not yet pivoted, first index on ties),
// costs the same 8 n^3 real flops as getrf+getri, and puts nearly all of
// them into rank-nbo updates (FP64 MFMA GEMMs).
//
// Columns are taken in outer blocks of nbo (64 or 128) columns, each
// factored as panels of nb (16 or 32) columns [ks, ks+nb):
//   k_gje_panel*     the panel's column steps (pivot search, interchange,
//                    elimination of every row: Gauss-Jordan) on its nb
//                    columns; the panel ends up holding its elimination
//                    transform.  One workgroup per matrix, or cooperative:
//                    R workgroups each holding a block of rows, one grid
//                    barrier per column.
//   k_gje_swap_save  applies the panel's row interchanges to the other
//                    columns of the outer block, saves their panel rows and
//                    zeroes them;
//   k_gje_update     A[:, those columns] += P * Rsaved  (complex, FP64 MFMA).
// When the outer block is done its columns hold the transform of all its nbo
// steps (the same numbers an nbo-wide panel would give), and the columns
// outside it take all its interchanges and one rank-nbo update: the matrix
// streams through HBM once per nbo columns instead of once per panel.
// At the end the row interchanges are undone as column interchanges in
// reverse order (k_gje_colperm).
//
// Barrier waits are bounded: a wait that exceeds its spin budget stores
// info = -1000 for that matrix and gives up, so the kernel always terminates.
#include <cfloat>
#include <cstdlib>
#include <cstring>
#include <utility>

#include "common.h"
#include "f64_tile.h"

namespace bgw {

constexpr int kPanelMax = 32;
constexpr int kGjeMaxR = 48;                // workgroups per matrix (n <= 12288, 256 rows each; the narrow
                                            // panel's LDS, 256 x 33 + 64 + 48 x 32 complex, fits 160 KB)
constexpr int kInfoBarrierTimeout = -1000;  // info value when a grid barrier wait gave up

struct GjeScratch {
    double *cand_val;         // [nmat][2][R]
    int *cand_row;            // [nmat][2][R]
    double2 *cand_rows;       // [nmat][2][R][nb]
    double2 *rowbuf;          // [nmat][2][nb]
    unsigned int *bar;        // [nmat] barrier counters (zeroed before the first panel)
};

__global__ void k_eps_build(const double2 *__restrict__ chi, const double *__restrict__ v, int ng, int nw,
                            double2 *__restrict__ eps) {
    const size_t per = (size_t)ng * ng;
    const size_t total = per * nw;
    for (size_t e = blockIdx.x * (size_t)blockDim.x + threadIdx.x; e < total; e += (size_t)gridDim.x * blockDim.x) {
        const size_t r = e % per;
        const int G = (int)(r / ng), H = (int)(r % ng);
        const double2 x = chi[e];
        eps[e] = make_double2((G == H ? 1.0 : 0.0) - v[G] * x.x, -v[G] * x.y);
    }
}

__global__ void k_fill_u32(unsigned int *p, size_t n, unsigned int val) {
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x)
        p[i] = val;
}

__device__ inline double cabs1(double2 a) { return fabs(a.x) + fabs(a.y); }

// x - f p, complex, as four FMAs
__device__ __forceinline__ double2 cfms(double2 x, double2 f, double2 p) {
    return make_double2(fma(-f.x, p.x, fma(f.y, p.y, x.x)), fma(-f.x, p.y, fma(-f.y, p.x, x.y)));
}

__device__ inline double2 cdiv(double2 a, double2 b) {
    // a / b with scaling (Smith's method)
    if (fabs(b.x) >= fabs(b.y)) {
        const double r = b.y / b.x, d = b.x + b.y * r;
        return make_double2((a.x + a.y * r) / d, (a.y - a.x * r) / d);
    }
    const double r = b.x / b.y, d = b.x * r + b.y;
    return make_double2((a.x * r + a.y) / d, (a.y * r - a.x) / d);
}

// grid barrier among the R workgroups of one matrix; `target` = R * (number of
// barriers passed including this one).  One release (the arrival) and one
// acquire fence after the wait: the spin itself uses relaxed loads, since an
// acquire load per iteration would invalidate the XCD's L2 every time.
__device__ inline void matrix_barrier(unsigned int *bar, unsigned int target, int *info) {
    __syncthreads();
    if (threadIdx.x == 0) {
        __hip_atomic_fetch_add(bar, 1u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
        unsigned long long spins = 0;
        while (__hip_atomic_load(bar, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < target) {
            __builtin_amdgcn_s_sleep(1);
            if (++spins > (1ull << 24)) {  // bounded wait: report and give up
                atomicExch(info, kInfoBarrierTimeout);
                break;
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    }
    // the exchanged values are then read with device-scope atomic loads
    __syncthreads();
}

__device__ inline double2 ld_agent(const double2 *p) {
    const double *d = reinterpret_cast<const double *>(p);
    return make_double2(__hip_atomic_load(d, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT),
                        __hip_atomic_load(d + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
}

__device__ inline void st_agent(double2 *p, double2 v) {
    double *d = reinterpret_cast<double *>(p);
    __hip_atomic_store(d, v.x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(d + 1, v.y, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Largest |Re|+|Im| over a wavefront, first row on ties; every lane gets the result.
__device__ inline void wave_argmax(double &v, int &row) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        const double ov = __shfl_xor(v, off);
        const int orow = __shfl_xor(row, off);
        if (ov > v || (ov == v && orow < row)) {
            v = ov;
            row = orow;
        }
    }
}

// A: matrices of a group, [nmat][n][n]; each matrix is factored by R
// consecutive workgroups, workgroup r owning rows [r*rows, min(n, (r+1)*rows))
// (rows <= blockDim.x: one row per thread).  NB: panel width known at compile
// time (0: the runtime nb, for the last, narrower panel).
template <int NB>
__global__ __launch_bounds__(256) void k_gje_panel(double2 *__restrict__ A, int n, int k, int nb_rt, int rows, int R,
                                                   int *__restrict__ ipiv, int *__restrict__ info, GjeScratch sc,
                                                   unsigned int bar_done) {
    extern __shared__ double2 lds[];
    const int nb = NB ? NB : nb_rt;
    const int ps = nb + 1;                       // padded row stride of the panel in LDS
    double2 *P = lds;                            // [rows][ps]
    double2 *prow = P + rows * (kPanelMax + 1);  // scaled pivot row [nb]
    double2 *oldrow = prow + kPanelMax;          // row k+j before the swap [nb]
    double2 *cand = oldrow + kPanelMax;          // candidate rows of all workgroups [R][nb]
    __shared__ double wv[4], cv_s[kGjeMaxR];
    __shared__ int wrow[4], cr_s[kGjeMaxR];

    const int mat = blockIdx.x / R, r = blockIdx.x % R;
    double2 *Am = A + (size_t)mat * n * n;
    int *ip = ipiv + (size_t)mat * n;
    const int row0 = r * rows;
    const int nloc = max(0, min(rows, n - row0));
    double *cval = sc.cand_val + (size_t)mat * 2 * R;
    int *crow = sc.cand_row + (size_t)mat * 2 * R;
    double2 *crows = sc.cand_rows + (size_t)mat * 2 * R * nb;
    double2 *rbuf = sc.rowbuf + (size_t)mat * 2 * nb;
    unsigned int *bar = sc.bar + mat;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int gi = row0 + tid;  // this thread's row
    const bool mine = tid < nloc;
    double2 *pr = P + tid * ps;

    for (int e = tid; e < nloc * nb; e += blockDim.x) {
        const int i = e / nb, c = e % nb;
        P[i * ps + c] = Am[(size_t)(row0 + i) * n + k + c];
    }
    __syncthreads();

    for (int j = 0; j < nb; ++j) {
        const int col = k + j;
        const int slot = j & 1;
        // local pivot candidate among rows >= col
        double best = -1.0;
        int brow = 0x7fffffff;
        if (mine && gi >= col) {
            const double v = cabs1(pr[j]);
            if (v >= 0.0) {  // a NaN entry is never a pivot candidate
                best = v;
                brow = gi;
            }
        }
        wave_argmax(best, brow);
        if (lane == 0) {
            wv[wave] = best;
            wrow[wave] = brow;
        }
        __syncthreads();
        best = wv[0];
        brow = wrow[0];
        for (int w = 1; w < (int)(blockDim.x >> 6); ++w)
            if (wv[w] > best || (wv[w] == best && wrow[w] < brow)) {
                best = wv[w];
                brow = wrow[w];
            }
        // publish the candidate (value, row, row contents) and, from the owner, row col
        if (tid == 0) {
            __hip_atomic_store(&cval[slot * R + r], best, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(&crow[slot * R + r], brow, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        if (tid < nb)
            st_agent(&crows[((size_t)slot * R + r) * nb + tid],
                     best >= 0.0 ? P[(brow - row0) * ps + tid] : make_double2(0.0, 0.0));
        if (col >= row0 && col < row0 + nloc && tid < nb) st_agent(&rbuf[slot * nb + tid], P[(col - row0) * ps + tid]);

        matrix_barrier(bar, (bar_done + j + 1) * (unsigned)R, info + mat);

        // every workgroup fetches all candidates (values, rows, row contents) and row col in one round
        for (int e = tid; e < R * nb; e += blockDim.x) cand[e] = ld_agent(&crows[(size_t)slot * R * nb + e]);
        if (tid < R) {
            cv_s[tid] = __hip_atomic_load(&cval[slot * R + tid], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            cr_s[tid] = __hip_atomic_load(&crow[slot * R + tid], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        if (tid >= 64 && tid < 64 + nb) oldrow[tid - 64] = ld_agent(&rbuf[slot * nb + tid - 64]);
        __syncthreads();
        // global pivot (every thread, same order): largest |Re|+|Im|, first row on ties
        double bv = cv_s[0];
        int p = cr_s[0], win = 0;
        for (int q = 1; q < R; ++q)
            if (cv_s[q] > bv || (cv_s[q] == bv && cr_s[q] < p)) {
                bv = cv_s[q];
                p = cr_s[q];
                win = q;
            }
        if (p >= n) p = col;  // no candidate (a column of NaNs): no interchange; info flags the matrix
        if (tid == 0 && r == 0) {
            if (!(bv > 0.0)) atomicCAS(info + mat, 0, col + 1);
            ip[col] = p;
        }
        const double2 *praw = cand + win * nb;
        if (tid < nb) {
            double2 piv = praw[j];
            if (piv.x == 0.0 && piv.y == 0.0) piv = make_double2(1.0, 0.0);
            const double2 ipv = cdiv(make_double2(1.0, 0.0), piv);
            prow[tid] = tid == j ? ipv : cmul(praw[tid], ipv);
            // row interchange col <-> p inside the panel
            if (p != col && p >= row0 && p < row0 + nloc) P[(p - row0) * ps + tid] = oldrow[tid];
        }
        __syncthreads();
        // eliminate: every row except col; row col becomes the scaled pivot row
        if (mine) {
            if (gi == col) {
#pragma unroll
                for (int c = 0; c < (NB ? NB : kPanelMax); ++c)
                    if (NB || c < nb) pr[c] = prow[c];
            } else {
                const double2 f = pr[j];
                const double2 pj = prow[j];
#pragma unroll
                for (int c = 0; c < (NB ? NB : kPanelMax); ++c)
                    if (NB || c < nb) {
                        const double2 pc = prow[c];
                        const double2 x = pr[c];
                        pr[c] = (c == j) ? make_double2(-(f.x * pj.x - f.y * pj.y), -(f.x * pj.y + f.y * pj.x))
                                         : cfms(x, f, pc);
                    }
            }
        }
        __syncthreads();
    }
    for (int e = tid; e < nloc * nb; e += blockDim.x) {
        const int i = e / nb, c = e % nb;
        Am[(size_t)(row0 + i) * n + k + c] = P[i * ps + c];
    }
}

// Full-width panels (kPanelMax columns): the same column steps as
// k_gje_panel, with each thread's panel row held in registers.  The column
// steps are instantiated per column index, so every row element has a fixed
// register.  Every thread scales by the inverse pivot on the fly:
// row i -= (f / p) * (pivot row) and row col = (pivot row) / p, so the only
// shared data per column are the candidates fetched after the grid barrier.
struct GjeRegCtx {
    double2 *Am;
    int *ip, *info, *crow;
    double *cval;
    double2 *crows, *rbuf, *oldrow, *cand;
    unsigned int *bar;
    double *wv, *cv_s;
    int *wrow, *cr_s;
    int k, R, r, row0, nloc, gi, lane, wave, tid, mat;
    bool mine;
    unsigned int bar_done;
};

template <int J>
__device__ __forceinline__ void gje_reg_column(const GjeRegCtx &x, double2 (&rv)[kPanelMax]) {
    constexpr int nb = kPanelMax;
    const int col = x.k + J;
    constexpr int slot = J & 1;
    const int R = x.R;
    // local pivot candidate among rows >= col
    double best = -1.0;
    int brow = 0x7fffffff;
    if (x.mine && x.gi >= col) {
        const double v = cabs1(rv[J]);
        if (v >= 0.0) {  // a NaN entry is never a pivot candidate
            best = v;
            brow = x.gi;
        }
    }
    wave_argmax(best, brow);
    if (x.lane == 0) {
        x.wv[x.wave] = best;
        x.wrow[x.wave] = brow;
    }
    __syncthreads();
    best = x.wv[0];
    brow = x.wrow[0];
    for (int w = 1; w < (int)(blockDim.x >> 6); ++w)
        if (x.wv[w] > best || (x.wv[w] == best && x.wrow[w] < brow)) {
            best = x.wv[w];
            brow = x.wrow[w];
        }
    // publish the candidate (value, row, row contents) and, from its owner, row col
    if (x.tid == 0) {
        __hip_atomic_store(&x.cval[slot * R + x.r], best, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(&x.crow[slot * R + x.r], brow, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    if (x.mine && x.gi == brow) {
#pragma unroll
        for (int c = 0; c < nb; ++c) st_agent(&x.crows[((size_t)slot * R + x.r) * nb + c], rv[c]);
    }
    if (x.mine && x.gi == col) {
#pragma unroll
        for (int c = 0; c < nb; ++c) st_agent(&x.rbuf[slot * nb + c], rv[c]);
    }

    matrix_barrier(x.bar, (x.bar_done + J + 1) * (unsigned)R, x.info + x.mat);

    // every workgroup fetches all candidates and row col in one round
    for (int e = x.tid; e < R * nb; e += blockDim.x) x.cand[e] = ld_agent(&x.crows[(size_t)slot * R * nb + e]);
    if (x.tid < R) {
        x.cv_s[x.tid] = __hip_atomic_load(&x.cval[slot * R + x.tid], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        x.cr_s[x.tid] = __hip_atomic_load(&x.crow[slot * R + x.tid], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    if (x.tid >= 64 && x.tid < 64 + nb) x.oldrow[x.tid - 64] = ld_agent(&x.rbuf[slot * nb + x.tid - 64]);
    __syncthreads();
    // global pivot (every thread, same order): largest |Re|+|Im|, first row on ties
    double bv = x.cv_s[0];
    int p = x.cr_s[0], win = 0;
    for (int q = 1; q < R; ++q)
        if (x.cv_s[q] > bv || (x.cv_s[q] == bv && x.cr_s[q] < p)) {
            bv = x.cv_s[q];
            p = x.cr_s[q];
            win = q;
        }
    if (p == 0x7fffffff) p = col;  // no candidate (a column of NaNs): no interchange; info flags the matrix
    if (x.tid == 0 && x.r == 0) {
        if (!(bv > 0.0)) atomicCAS(x.info + x.mat, 0, col + 1);
        x.ip[col] = p;
    }
    const double2 *praw = x.cand + win * nb;
    double2 piv = praw[J];
    if (piv.x == 0.0 && piv.y == 0.0) piv = make_double2(1.0, 0.0);
    const double2 ipv = cdiv(make_double2(1.0, 0.0), piv);
    if (x.mine) {
        if (x.gi == col) {
            // row col becomes the scaled pivot row
#pragma unroll
            for (int c = 0; c < nb; ++c) rv[c] = c == J ? ipv : cmul(praw[c], ipv);
        } else {
            if (p != col && x.gi == p) {
#pragma unroll
                for (int c = 0; c < nb; ++c) rv[c] = x.oldrow[c];  // row p receives row col
            }
            const double2 fs = cmul(rv[J], ipv);
#pragma unroll
            for (int c = 0; c < nb; ++c)
                rv[c] = c == J ? make_double2(-fs.x, -fs.y) : cfms(rv[c], fs, praw[c]);
        }
    }
}

template <int J>
struct GjeRegColumns {
    __device__ __forceinline__ static void run(const GjeRegCtx &x, double2 (&rv)[kPanelMax]) {
        gje_reg_column<J>(x, rv);
        GjeRegColumns<J + 1>::run(x, rv);
    }
};
template <>
struct GjeRegColumns<kPanelMax> {
    __device__ __forceinline__ static void run(const GjeRegCtx &, double2 (&)[kPanelMax]) {}
};

__global__ __launch_bounds__(256) void k_gje_panel_reg(double2 *__restrict__ A, int n, int k, int rows, int R,
                                                       int *__restrict__ ipiv, int *__restrict__ info,
                                                       GjeScratch sc, unsigned int bar_done) {
    extern __shared__ double2 lds[];
    __shared__ double wv[4], cv_s[kGjeMaxR];
    __shared__ int wrow[4], cr_s[kGjeMaxR];
    GjeRegCtx x;
    x.mat = blockIdx.x / R;
    x.r = blockIdx.x % R;
    x.Am = A + (size_t)x.mat * n * n;
    x.ip = ipiv + (size_t)x.mat * n;
    x.info = info;
    x.row0 = x.r * rows;
    x.nloc = max(0, min(rows, n - x.row0));
    x.cval = sc.cand_val + (size_t)x.mat * 2 * R;
    x.crow = sc.cand_row + (size_t)x.mat * 2 * R;
    x.crows = sc.cand_rows + (size_t)x.mat * 2 * R * kPanelMax;
    x.rbuf = sc.rowbuf + (size_t)x.mat * 2 * kPanelMax;
    x.bar = sc.bar + x.mat;
    x.oldrow = lds;                  // row k+j before the swap [kPanelMax]
    x.cand = lds + kPanelMax;        // candidate rows of all workgroups [R][kPanelMax]
    x.wv = wv;
    x.cv_s = cv_s;
    x.wrow = wrow;
    x.cr_s = cr_s;
    x.k = k;
    x.R = R;
    x.tid = threadIdx.x;
    x.lane = x.tid & 63;
    x.wave = x.tid >> 6;
    x.gi = x.row0 + x.tid;
    x.mine = x.tid < x.nloc;
    x.bar_done = bar_done;

    double2 rv[kPanelMax];
#pragma unroll
    for (int c = 0; c < kPanelMax; ++c) rv[c] = x.mine ? x.Am[(size_t)x.gi * n + k + c] : make_double2(0.0, 0.0);
    GjeRegColumns<0>::run(x, rv);
    if (x.mine) {
#pragma unroll
        for (int c = 0; c < kPanelMax; ++c) x.Am[(size_t)x.gi * n + k + c] = rv[c];
    }
}

// The columns an update touches: [lo, hi) without [ex0, ex1), numbered
// cp = 0 .. m-1 in increasing order.
struct GjeCols {
    int lo, hi, ex0, ex1;
    __host__ __device__ int count() const { return (hi - lo) - (ex1 - ex0); }
    __device__ int col(int cp) const {
        const int c = lo + cp;
        return c < ex0 ? c : c + (ex1 - ex0);
    }
};

constexpr int kSwapCols = 32;     // columns of one k_gje_swap_save workgroup
constexpr int kSwapRows = 4 * kPanelMax;

// Row interchanges ipiv[r0 .. r0+nbr) on the columns cs, then the panel's rows r0 ..
// copied to Rs [nbr][m] and zeroed in A.  One after the other the interchanges are a
// chain of nbr round trips to memory per column; here wave 0 first plays them on
// row numbers held in its lanes (slot j: panel row r0 + j; slot 128 + j: the row
// outside the panel that interchange j names, at its first naming), and then every
// row moves once, independent of the others.  Eight matrices of 1500, 24 outer blocks
// of 64 rows and 94 panels of 16: 1.67 -> 0.95 ms in all.  256 threads: 32 columns
// times 8 groups of rows; nbr <= 128.
__global__ __launch_bounds__(256) void k_gje_swap_save(double2 *__restrict__ A, int n, int r0, int nbr, GjeCols cs,
                                                       const int *__restrict__ ipiv, double2 *__restrict__ Rs) {
    __shared__ int piv[kSwapRows], slot[kSwapRows], from[2 * kSwapRows];
    extern __shared__ double2 out[];  // [nbr][kSwapCols]: new contents of the outside rows
    const int mat = blockIdx.y, tid = threadIdx.x;
    double2 *Am = A + (size_t)mat * n * n;
    const int m = cs.count();
    double2 *R = Rs + (size_t)mat * nbr * m;
    if (tid < nbr) {
        const int p = ipiv[(size_t)mat * n + r0 + tid];
        piv[tid] = p > r0 + tid && p < n ? p : r0 + tid;  // anything else: no interchange
    }
    __syncthreads();
    if (tid < nbr) {
        const int p = piv[tid];
        int s = p - r0;
        if (s >= nbr) {
            int j = 0;
            while (piv[j] != p) ++j;
            s = kSwapRows + j;
        }
        slot[tid] = s;
    }
    __syncthreads();
    if (tid < 64) {
        // row numbers in slots lane, 64 + lane, 128 + lane, 192 + lane
        int c[4], q[2];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int j = 64 * h + tid;
            c[h] = r0 + j;
            c[2 + h] = j < nbr ? piv[j] : 0;
            q[h] = j < nbr ? slot[j] : j;
        }
        for (int j = 0; j < nbr; ++j) {
            const int lj = j & 63;
            const int s = __builtin_amdgcn_readlane(j < 64 ? q[0] : q[1], lj), ls = s & 63;
            const int x = __builtin_amdgcn_readlane(j < 64 ? c[0] : c[1], lj);
            int y = 0;
#pragma unroll
            for (int h = 0; h < 4; ++h)
                if (s >> 6 == h) {
                    y = __builtin_amdgcn_readlane(c[h], ls);
                    if (tid == ls) c[h] = x;
                }
            if (tid == lj) {
                if (j < 64) c[0] = y;
                else c[1] = y;
            }
        }
#pragma unroll
        for (int h = 0; h < 4; ++h) from[64 * h + tid] = c[h];
    }
    __syncthreads();
    const int cl = tid % kSwapCols, rg = tid / kSwapCols, cp = blockIdx.x * kSwapCols + cl;
    const bool live = cp < m;
    const int col = live ? cs.col(cp) : 0;
    constexpr int NG = 256 / kSwapCols;
    if (live) {
#pragma unroll 4
        for (int j = rg; j < nbr; j += NG) {
            R[(size_t)j * m + cp] = Am[(size_t)from[j] * n + col];
            if (slot[j] == kSwapRows + j) out[j * kSwapCols + cl] = Am[(size_t)from[kSwapRows + j] * n + col];
        }
    }
    __syncthreads();
    if (live) {
#pragma unroll 4
        for (int j = rg; j < nbr; j += NG) {
            Am[(size_t)(r0 + j) * n + col] = make_double2(0.0, 0.0);
            if (slot[j] == kSwapRows + j) Am[(size_t)piv[j] * n + col] = out[j * kSwapCols + cl];
        }
    }
}

// A[:, cs] += P * R with P = A[:, r0:r0+nbr] (n x nbr) and R = Rs (nbr x m); the
// old values of the tile are fetched under the last stage's MFMAs.  Bound by the
// FP64 MFMAs at 128 columns per update (16 flops per byte of A moved) and by
// latency in the narrow updates within an outer block.  Eight matrices of 1500, whole
// inversions: 13.88 -> 13.02 ms against a tile loop that staged both operands through
// registers (11.3 with what the panels and interchanges have saved since).
template <int T>
__global__ __launch_bounds__(256, 2) void k_gje_update(double2 *__restrict__ A, int n, int r0, int nbr, GjeCols cs,
                                                    const double2 *__restrict__ Rs) {
    __shared__ PqLds<T> lds;
    double2 *Am = A + (size_t)blockIdx.z * n * n;
    const int m = cs.count(), I0 = blockIdx.x * T, C0 = blockIdx.y * T;
    double4_t cre[T / 32][T / 32], cim[T / 32][T / 32];
    double2 old[T / 32][T / 32][4];
    pq_sums<T, false, true>({Am + r0, n, n}, {Rs + (size_t)blockIdx.z * nbr * m, m, m}, nullptr, I0, C0, 0, nbr, cre,
                            cim, lds, [&] {
                                pq_each<T>([&](int a, int b, int r, int i, int c) {
                                    old[a][b][r] = make_double2(0.0, 0.0);
                                    if (I0 + i < n && C0 + c < m)
                                        old[a][b][r] = Am[(size_t)(I0 + i) * n + cs.col(C0 + c)];
                                });
                            });
    pq_each<T>([&](int a, int b, int r, int i, int c) {
        if (I0 + i < n && C0 + c < m)
            Am[(size_t)(I0 + i) * n + cs.col(C0 + c)] =
                make_double2(old[a][b][r].x + cre[a][b][r], old[a][b][r].y + cim[a][b][r]);
    });
}

// Column index map of the final column interchanges: start from the identity
// and swap entries j <-> ipiv[j] for j = n-1 down to 0.  One workgroup per
// matrix; the sequential swap chain runs on one thread over LDS copies.
__global__ void k_gje_perm(const int *__restrict__ ipiv, int n, int *__restrict__ idx) {
    extern __shared__ int perm_lds[];
    int *id = perm_lds, *ip = perm_lds + n;
    const int mat = blockIdx.x;
    for (int j = threadIdx.x; j < n; j += blockDim.x) {
        id[j] = j;
        const int p = ipiv[(size_t)mat * n + j];
        ip[j] = (p >= j && p < n) ? p : j;  // an out-of-range pivot: no interchange
    }
    __syncthreads();
    if (threadIdx.x == 0)
        for (int j = n - 1; j >= 0; --j) {
            const int p = ip[j];
            const int t = id[j];
            id[j] = id[p];
            id[p] = t;
        }
    __syncthreads();
    for (int j = threadIdx.x; j < n; j += blockDim.x) idx[(size_t)mat * n + j] = id[j];
}

// out[i][c] = A[i][idx[c]], one workgroup per row, row staged in LDS (in place).
__global__ void k_gje_colperm(double2 *__restrict__ A, int n, const int *__restrict__ idx) {
    extern __shared__ double2 row[];
    const int mat = blockIdx.y;
    double2 *a = A + ((size_t)mat * n + blockIdx.x) * n;
    const int *id = idx + (size_t)mat * n;
    for (int c = threadIdx.x; c < n; c += blockDim.x) row[c] = a[c];
    __syncthreads();
    for (int c = threadIdx.x; c < n; c += blockDim.x) a[c] = row[id[c]];
}

// The same for rows longer than LDS holds (n > 8192): every thread gathers
// its outputs' sources from the row in global memory into registers, waits
// for them, the block meets, then the row is overwritten.  n <= 256 * 48.
constexpr int kColPermPer = 48;
__global__ __launch_bounds__(256) void k_gje_colperm_reg(double2 *__restrict__ A, int n, const int *__restrict__ idx) {
    const int mat = blockIdx.y;
    double2 *a = A + ((size_t)mat * n + blockIdx.x) * n;
    const int *id = idx + (size_t)mat * n;
    double2 v[kColPermPer];
#pragma unroll
    for (int j = 0; j < kColPermPer; ++j) {
        const int c = threadIdx.x + 256 * j;
        v[j] = c < n ? a[id[c]] : make_double2(0.0, 0.0);
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // every read of the row has returned
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kColPermPer; ++j) {
        const int c = threadIdx.x + 256 * j;
        if (c < n) a[c] = v[j];
    }
}

// ------------------------------------------------------- one-workgroup panels
//
// Matrices with n <= kWgThreads * kWgMaxRows take their panels from one
// workgroup each: thread t holds the panel rows that start at positions
// t, t + 512, t + 1024 (panel width kWgNb) in registers, so a column step needs
// two workgroup barriers and no grid barrier.  The column steps are those of
// k_gje_panel: pivot = largest |Re|+|Im| among positions >= col (first
// position on ties), positions col and p exchanged, every other row
// eliminated, the pivot row scaled.  A row stays in its thread's registers;
// an interchange only swaps the positions recorded for the two rows, and each
// row is stored at its final position when the panel ends.
constexpr int kWgNb = 16;
constexpr int kWgThreads = 512;
constexpr int kWgMaxRows = 3;

namespace {
template <int CTRL>
__device__ __forceinline__ void argmax_dpp(double &v, int &key) {
    const unsigned long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_mov_dpp((int)(unsigned)b, CTRL, 0xF, 0xF, false);
    const int hi = __builtin_amdgcn_mov_dpp((int)(unsigned)(b >> 32), CTRL, 0xF, 0xF, false);
    const int ok = __builtin_amdgcn_mov_dpp(key, CTRL, 0xF, 0xF, false);
    const double ov = __longlong_as_double(((unsigned long long)(unsigned)hi << 32) | (unsigned)lo);
    if (ov > v || (ov == v && ok < key)) {
        v = ov;
        key = ok;
    }
}

// Largest v over the wavefront, smallest key on ties; every lane gets the
// result.  Quad swaps and the half-row and row mirrors agree the 16 lanes of
// each row, then the four rows are compared.
__device__ __forceinline__ void wave_argmax_dpp(double &v, int &key) {
    argmax_dpp<0xB1>(v, key);   // quad_perm [1,0,3,2]
    argmax_dpp<0x4E>(v, key);   // quad_perm [2,3,0,1]
    argmax_dpp<0x141>(v, key);  // row_half_mirror
    argmax_dpp<0x140>(v, key);  // row_mirror
    const unsigned long long b = __double_as_longlong(v);
    double bv = 0.0;
    int bk = 0;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int lo = __builtin_amdgcn_readlane((int)(unsigned)b, 16 * r);
        const int hi = __builtin_amdgcn_readlane((int)(unsigned)(b >> 32), 16 * r);
        const int kk = __builtin_amdgcn_readlane(key, 16 * r);
        const double x = __longlong_as_double(((unsigned long long)(unsigned)hi << 32) | (unsigned)lo);
        if (r == 0 || x > bv || (x == bv && kk < bk)) {
            bv = x;
            bk = kk;
        }
    }
    v = bv;
    key = bk;
}
}  // namespace

struct WgLds {
    double wv[kWgThreads / 64];
    int wk[kWgThreads / 64];
    double2 praw[kWgNb];
};

// Candidate of this thread for pivot column J (largest |Re|+|Im| among its
// rows at positions >= col, first position on ties), then of the wavefront,
// published in the LDS slots of the wavefront.
template <int ROWS, int J>
__device__ __forceinline__ void gje_wg_candidate(const double2 (&rv)[ROWS][kWgNb], const int (&pos)[ROWS], WgLds &L,
                                                 int n, int col) {
    double best = -1.0;
    int key = 0x7fffffff;
#pragma unroll
    for (int r = 0; r < ROWS; ++r) {
        if (pos[r] >= col && pos[r] < n) {
            const double v = cabs1(rv[r][J]);
            if (v > best || (v == best && pos[r] < key)) {
                best = v;
                key = pos[r];
            }
        }
    }
    wave_argmax_dpp(best, key);
    if ((threadIdx.x & 63) == 0) {
        L.wv[threadIdx.x >> 6] = best;
        L.wk[threadIdx.x >> 6] = key;
    }
}

// 1 / z with one division: z is scaled by a power of two first, so that
// |z|^2 can neither overflow nor underflow.
__device__ __forceinline__ double2 crecip(double2 z) {
    int e = 0;
    (void)frexp(fmax(fabs(z.x), fabs(z.y)), &e);
    const double x = ldexp(z.x, -e), y = ldexp(z.y, -e);
    const double t = ldexp(1.0 / (x * x + y * y), -e);
    return make_double2(x * t, -y * t);
}

// Column step J (compile-time, so every row element keeps a fixed register).
// pos[r]: current position of row r of this thread (>= n: padding row of
// zeros).  The candidates of column J were published by step J - 1 (by the
// caller for J = 0): right after column J + 1 is eliminated, before the
// other columns, so their search overlaps the rest of the elimination.
// What bounds a step is its serial chain (search, reciprocal, pivot row) beside
// some 200 FP64 operations per row; the pivot row is therefore read one element
// ahead of its use, and the eight wavefronts' candidates are compared across eight
// lanes and not one after the other: 94 panels of 16 columns of eight matrices of
// 1500 5.89 -> 4.91 ms.
template <int ROWS, int J>
__device__ __forceinline__ void gje_wg_column(double2 (&rv)[ROWS][kWgNb], int (&pos)[ROWS], WgLds &L, int n, int k,
                                              int jb, int nb, int *ip, int *info) {
    constexpr int NW = kWgThreads / 64;
    if (jb + J >= nb) return;  // uniform
    const int tid = threadIdx.x;
    const int col = k + jb + J;
    __syncthreads();
    // every eight lanes compare the wavefronts' candidates
    static_assert(NW == 8, "one candidate per lane of eight");
    double bv = L.wv[tid & 7];
    int p = L.wk[tid & 7];
    argmax_dpp<0xB1>(bv, p);   // quad_perm [1,0,3,2]
    argmax_dpp<0x4E>(bv, p);   // quad_perm [2,3,0,1]
    argmax_dpp<0x141>(bv, p);  // row_half_mirror
    // p >= col; no candidate at all (a column of NaNs): no interchange, info flags the matrix
    if (p >= n) p = col;
    int piv_r = -1;  // which of this thread's rows is the pivot row
#pragma unroll
    for (int r = 0; r < ROWS; ++r)
        if (pos[r] == p) piv_r = r;
    if (piv_r >= 0) {
#pragma unroll
        for (int r = 0; r < ROWS; ++r)
            if (r == piv_r) {
#pragma unroll
                for (int c = 0; c < kWgNb; ++c) L.praw[c] = rv[r][c];
            }
    }
    if (tid == 0) {
        ip[col] = p;
        if (!(bv > 0.0)) atomicCAS(info, 0, col + 1);
    }
    // interchange of positions col and p
#pragma unroll
    for (int r = 0; r < ROWS; ++r) pos[r] = pos[r] == p ? col : (pos[r] == col ? p : pos[r]);
    __syncthreads();
    double2 piv = L.praw[J];
    if (piv.x == 0.0 && piv.y == 0.0) piv = make_double2(1.0, 0.0);
    const double2 ipv = crecip(piv);
    // every row is eliminated with the pivot row, read from LDS once per
    // column element by element (padding rows hold zeros and stay zero);
    // the pivot row's own result is replaced below
    double2 fs[ROWS];
#pragma unroll
    for (int r = 0; r < ROWS; ++r) {
        fs[r] = cmul(rv[r][J], ipv);
        rv[r][J] = make_double2(-fs[r].x, -fs[r].y);
    }
    constexpr int JN = J + 1 < kWgNb ? J + 1 : J;  // next pivot column
    if (J + 1 < kWgNb) {
        const double2 pc = L.praw[JN];
#pragma unroll
        for (int r = 0; r < ROWS; ++r) rv[r][JN] = cfms(rv[r][JN], fs[r], pc);
        if (jb + J + 1 < nb) gje_wg_candidate<ROWS, JN>(rv, pos, L, n, col + 1);
    }
    // the pivot row read one element ahead (the barriers keep the reads from piling up
    // in registers)
    double2 pc = L.praw[(J + 2) % kWgNb];
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 2; i < kWgNb; ++i) {
        const int c = (J + i) % kWgNb;
        if (c == J || c == JN) continue;
        const double2 next = L.praw[(c + 1) % kWgNb];
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int r = 0; r < ROWS; ++r) rv[r][c] = cfms(rv[r][c], fs[r], pc);
        __builtin_amdgcn_sched_barrier(0);
        pc = next;
    }
    if (piv_r >= 0) {  // the pivot row, now at position col, becomes the scaled pivot row
#pragma unroll
        for (int r = 0; r < ROWS; ++r)
            if (r == piv_r) {
#pragma unroll
                for (int c = 0; c < kWgNb; ++c) rv[r][c] = c == J ? ipv : cmul(L.praw[c], ipv);
            }
    }
    // the next step writes praw only after its first barrier, which every
    // thread reaches after these reads; its candidates were written after
    // this step's second barrier, which every thread passed after reading
    // this step's candidates
}

template <int ROWS, int... Js>
__device__ __forceinline__ void gje_wg_columns(double2 (&rv)[ROWS][kWgNb], int (&pos)[ROWS], WgLds &L, int n, int k,
                                               int jb, int nb, int *ip, int *info, std::integer_sequence<int, Js...>) {
    (gje_wg_column<ROWS, Js>(rv, pos, L, n, k, jb, nb, ip, info), ...);
}

// One workgroup per matrix (blockIdx.x), panel columns [k, k + nb), nb <= kWgNb.
// The panel moves between A and the registers through an LDS stage of 512
// rows (row stride kWgNb + 1 elements, conflict-free row reads), so the
// global accesses are whole 256-byte row segments.
constexpr int kWgStageLd = kWgNb + 1;
constexpr int kWgUnroll = 2;  // column steps per pass of the panel loop
static_assert(kWgNb % kWgUnroll == 0 && kWgUnroll >= 1, "whole passes");
constexpr size_t kWgStageBytes = sizeof(double2) * kWgThreads * kWgStageLd;

template <int ROWS>
__global__ __launch_bounds__(kWgThreads) void k_gje_panel_wg(double2 *__restrict__ A, int n, int k, int nb,
                                                             int *__restrict__ ipiv, int *__restrict__ info) {
    __shared__ WgLds L;
    extern __shared__ double2 wg_stage[];  // [kWgThreads][kWgStageLd]
    const int mat = blockIdx.x;
    double2 *Am = A + (size_t)mat * n * n;
    const int tid = threadIdx.x;
    double2 rv[ROWS][kWgNb];
    int pos[ROWS];
#pragma unroll
    for (int r = 0; r < ROWS; ++r) {
        const int r0 = r * kWgThreads;
        const int cnt = min(kWgThreads, n - r0);  // >= 1
        pos[r] = r0 + tid;
        {
            // the block's 16 loads per thread in flight together
            double2 v[kWgNb];
#pragma unroll
            for (int it = 0; it < kWgNb; ++it) {
                const int e = tid + it * kWgThreads, i = e / kWgNb, c = e % kWgNb;
                v[it] = (i < cnt && c < nb) ? Am[(size_t)(r0 + i) * n + k + c] : make_double2(0.0, 0.0);
            }
#pragma unroll
            for (int it = 0; it < kWgNb; ++it) {
                const int e = tid + it * kWgThreads, i = e / kWgNb, c = e % kWgNb;
                if (i < cnt) wg_stage[i * kWgStageLd + c] = v[it];
            }
        }
        __syncthreads();
#pragma unroll
        for (int c = 0; c < kWgNb; ++c) rv[r][c] = tid < cnt ? wg_stage[tid * kWgStageLd + c] : make_double2(0.0, 0.0);
        __syncthreads();
    }
    gje_wg_candidate<ROWS, 0>(rv, pos, L, n, k);
    // kWgUnroll column steps per pass on register columns 0 .. kWgUnroll-1,
    // then the columns rotate left by kWgUnroll, so that the next pass again
    // starts at register column 0; after kWgNb / kWgUnroll passes every
    // column is back in its own register.  The pass is a real loop: fully
    // unrolled, the three-row panel is about 100 KB of code, more than the
    // instruction cache holds, and each launch fetches all of it once.
#pragma unroll 1
    for (int jb = 0; jb < kWgNb; jb += kWgUnroll) {
        gje_wg_columns<ROWS>(rv, pos, L, n, k, jb, nb, ipiv + (size_t)mat * n, info + mat,
                             std::make_integer_sequence<int, kWgUnroll>{});
        if (kWgUnroll < kWgNb) {
#pragma unroll
            for (int r = 0; r < ROWS; ++r) {
                double2 t[kWgNb];
#pragma unroll
                for (int c = 0; c < kWgNb; ++c) t[c] = rv[r][(c + kWgUnroll) % kWgNb];
#pragma unroll
                for (int c = 0; c < kWgNb; ++c) rv[r][c] = t[c];
            }
        }
    }
    // every row to its final position, one 512-position block at a time
#pragma unroll
    for (int b = 0; b < ROWS; ++b) {
        const int r0 = b * kWgThreads;
        const int cnt = min(kWgThreads, n - r0);
        __syncthreads();
#pragma unroll
        for (int r = 0; r < ROWS; ++r) {
            if (pos[r] >= r0 && pos[r] < r0 + cnt) {
#pragma unroll
                for (int c = 0; c < kWgNb; ++c) wg_stage[(pos[r] - r0) * kWgStageLd + c] = rv[r][c];
            }
        }
        __syncthreads();
#pragma unroll 4
        for (int it = 0; it < kWgNb; ++it) {
            const int e = tid + it * kWgThreads, i = e / kWgNb, c = e % kWgNb;
            if (i < cnt && c < nb) Am[(size_t)(r0 + i) * n + k + c] = wg_stage[i * kWgStageLd + c];
        }
    }
}

// ---------------------------------------------------------------- host side

int launch_eps_build(const double2 *chi, const double *v, int ng, int nw, double2 *eps, hipStream_t st) {
    const size_t total = (size_t)ng * ng * nw;
    const int blocks = (int)std::min<size_t>((total + 255) / 256, 65536);
    hipLaunchKernelGGL(k_eps_build, dim3(blocks), dim3(256), 0, st, chi, v, ng, nw, eps);
    BGW_HIP(hipGetLastError());
    return BGW_OK;
}

size_t gje_scratch_bytes(int nmat, int R) {
    size_t b = 0;
    b += sizeof(double) * nmat * 2 * R;
    b += sizeof(int) * nmat * 2 * R;
    b += sizeof(double2) * nmat * 2 * R * kPanelMax;
    b += sizeof(double2) * nmat * 2 * kPanelMax;
    b += sizeof(unsigned int) * nmat;
    return b + 6 * 256;
}

static char *align256(char *p) { return (char *)(((uintptr_t)p + 255) & ~(uintptr_t)255); }

// Width of the outer blocks: panels run kWgNb or kPanelMax columns at a time
// and update only the other columns of their outer block; the rest of the
// matrix takes one rank-(outer width) update per outer block.
static int gje_outer_nb(int n) { return n >= 3000 ? 4 * kPanelMax : 2 * kPanelMax; }

template <int T>
static void launch_gje_update_t(double2 *A, int n, int nmat, int r0, int nbr, GjeCols cs, const double2 *Rs,
                                hipStream_t st) {
    hipLaunchKernelGGL(HIP_KERNEL_NAME(k_gje_update<T>), dim3((n + T - 1) / T, (cs.count() + T - 1) / T, nmat),
                       dim3(256), 0, st, A, n, r0, nbr, cs, Rs);
}

// 64-wide tiles read half as much per product; of fewer than 2000 of them (eight per
// CU) the last ones leave most of the chip idle, and 32-wide tiles finish first.
// Whole inversions in 64- and in 32-wide tiles, with the tiles of an outer block's
// update: one matrix of 1500 (552) 7.19 and 6.76 ms, one of 2500 (1560) 24.76 and
// 24.03, four of 1500 (2208) 8.79 and 8.46, one of 3100 (2303) 31.84 and 31.73, two of
// 3100 (4606) 37.73 and 37.88, four of 4000 (15372) 83.0 and 86.2; the updates within
// an outer block, of fewer columns, are in 32-wide tiles at all of these.
static void launch_gje_update(double2 *A, int n, int nmat, int r0, int nbr, GjeCols cs, const double2 *Rs,
                              hipStream_t st) {
    const long long t64 = (long long)((n + 63) / 64) * ((cs.count() + 63) / 64) * nmat;
    if (t64 < 2000) launch_gje_update_t<32>(A, n, nmat, r0, nbr, cs, Rs, st);
    else launch_gje_update_t<64>(A, n, nmat, r0, nbr, cs, Rs, st);
}

// Row interchanges and rank-nbr update of the panel [r0, r0 + nbr) applied to
// the columns cs: A[:, cs] = swapped, panel rows saved and zeroed, += P Rs.
static int gje_apply(double2 *A, int n, int nmat, int r0, int nbr, GjeCols cs, const int *ipiv, double2 *Rs,
                     hipStream_t st) {
    const int m = cs.count();
    if (m <= 0) return BGW_OK;
    const size_t lds = sizeof(double2) * (size_t)nbr * kSwapCols;
    hipLaunchKernelGGL(k_gje_swap_save, dim3((m + kSwapCols - 1) / kSwapCols, nmat), dim3(256), lds, st, A, n, r0, nbr, cs,
                       ipiv, Rs);
    launch_gje_update(A, n, nmat, r0, nbr, cs, Rs, st);
    BGW_HIP(hipGetLastError());
    return BGW_OK;
}

// In-place inversion of `nmat` matrices A[nmat][n][n].  ws: device workspace of
// at least gje_workspace_bytes(n, nmat, R) bytes.  info: [nmat], zeroed here.
size_t gje_workspace_bytes(int n, int nmat, int R) {
    return gje_scratch_bytes(nmat, R) + sizeof(double2) * (size_t)nmat * gje_outer_nb(n) * n + 256 +
           sizeof(int) * (size_t)nmat * n * 2 + 512;
}

static size_t gje_panel_lds(int rows, int R) {
    return sizeof(double2) * ((size_t)rows * (kPanelMax + 1) + 2 * kPanelMax + (size_t)R * kPanelMax);
}

static size_t gje_panel_reg_lds(int R) { return sizeof(double2) * (kPanelMax + (size_t)R * kPanelMax); }

// rows of the panel held by one workgroup (one per thread): few workgroups per
// matrix keep the per-column grid barrier cheap
int gje_rows_per_wg(int n) { return std::min(256, n); }

// One workgroup per matrix panel for n <= 1536, unless BGW_GJE_PATH=coop asks
// for the cooperative multi-workgroup panels.
static bool gje_one_wg(int n) {
    if (n > kWgThreads * kWgMaxRows) return false;
    const char *e = std::getenv("BGW_GJE_PATH");
    return !(e && std::strcmp(e, "coop") == 0);
}

static int launch_gje_invert_wg(double2 *A, int n, int nmat, int *ipiv, int *info, double2 *Rs, hipStream_t st) {
    const int rows = (n + kWgThreads - 1) / kWgThreads;
    const void *kern = rows == 1 ? (const void *)k_gje_panel_wg<1>
                     : rows == 2 ? (const void *)k_gje_panel_wg<2>
                                 : (const void *)k_gje_panel_wg<3>;
    BGW_HIP(hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kWgStageBytes));
    const int nbo = gje_outer_nb(n);
    for (int k = 0; k < n; k += nbo) {
        const int ke = std::min(n, k + nbo);
        for (int ks = k; ks < ke; ks += kWgNb) {
            const int nb = std::min(kWgNb, ke - ks);
            void *args[] = {&A, (void *)&n, &ks, (void *)&nb, &ipiv, &info};
            BGW_HIP(hipLaunchKernel(kern, dim3(nmat), dim3(kWgThreads), args, kWgStageBytes, st));
            BGW_TRY(gje_apply(A, n, nmat, ks, nb, GjeCols{k, ke, ks, ks + nb}, ipiv, Rs, st));
        }
        BGW_TRY(gje_apply(A, n, nmat, k, ke - k, GjeCols{0, n, k, ke}, ipiv, Rs, st));
    }
    return BGW_OK;
}

static int launch_gje_invert_coop(double2 *A, int n, int nmat, int *info, GjeScratch sc, double2 *Rs, int *ipiv,
                                  int rows, int R, hipStream_t st);
static int launch_gje_unpermute(double2 *A, int n, int nmat, const int *ipiv, int *idx, hipStream_t st);

int launch_gje_invert(double2 *A, int n, int nmat, int *info, void *ws, int *ipiv_ws, hipStream_t st) {
    const int rows = gje_rows_per_wg(n);
    const int R = (n + rows - 1) / rows;
    char *p = align256((char *)ws);
    GjeScratch sc;
    sc.cand_val = (double *)p; p = align256(p + sizeof(double) * nmat * 2 * R);
    sc.cand_row = (int *)p; p = align256(p + sizeof(int) * nmat * 2 * R);
    sc.cand_rows = (double2 *)p; p = align256(p + sizeof(double2) * nmat * 2 * R * kPanelMax);
    sc.rowbuf = (double2 *)p; p = align256(p + sizeof(double2) * nmat * 2 * kPanelMax);
    sc.bar = (unsigned int *)p; p = align256(p + sizeof(unsigned int) * nmat);
    double2 *Rs = (double2 *)p; p = align256(p + sizeof(double2) * (size_t)nmat * gje_outer_nb(n) * n);
    int *ipiv = ipiv_ws;
    int *idx = ipiv + (size_t)nmat * n;

    hipLaunchKernelGGL(k_fill_u32, dim3(1), dim3(256), 0, st, sc.bar, (size_t)nmat, 0u);
    hipLaunchKernelGGL(k_fill_u32, dim3(1), dim3(64), 0, st, (unsigned int *)info, (size_t)nmat, 0u);
    BGW_HIP(hipGetLastError());

    BGW_HIP(hipFuncSetAttribute((const void *)k_gje_swap_save, hipFuncAttributeMaxDynamicSharedMemorySize,
                                (int)(sizeof(double2) * kSwapRows * kSwapCols)));
    if (gje_one_wg(n)) {
        BGW_TRY(launch_gje_invert_wg(A, n, nmat, ipiv, info, Rs, st));
    } else {
        BGW_TRY(launch_gje_invert_coop(A, n, nmat, info, sc, Rs, ipiv, rows, R, st));
    }
    return launch_gje_unpermute(A, n, nmat, ipiv, idx, st);
}

static int launch_gje_invert_coop(double2 *A, int n, int nmat, int *info, GjeScratch sc, double2 *Rs, int *ipiv,
                                  int rows, int R, hipStream_t st) {
    if (R > kGjeMaxR) return BGW_ERR_UNSUPPORTED;
    const size_t lds = gje_panel_lds(rows, R);
    BGW_HIP(hipFuncSetAttribute((const void *)k_gje_panel<kPanelMax>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                (int)lds));
    BGW_HIP(hipFuncSetAttribute((const void *)k_gje_panel<0>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    const size_t rlds_panel = gje_panel_reg_lds(R);
    unsigned int bar_done = 0;
    const int nbo = gje_outer_nb(n);
    for (int k = 0; k < n; k += nbo) {
        const int ke = std::min(n, k + nbo);
        for (int ks = k; ks < ke; ks += kPanelMax) {
            const int nb = std::min(kPanelMax, ke - ks);
            void *args[] = {&A, (void *)&n, &ks, (void *)&nb, (void *)&rows, (void *)&R, &ipiv, &info, &sc, &bar_done};
            if (nb == kPanelMax) {
                void *rargs[] = {&A, (void *)&n, &ks, (void *)&rows, (void *)&R, &ipiv, &info, &sc, &bar_done};
                BGW_HIP(hipLaunchCooperativeKernel((const void *)k_gje_panel_reg, dim3(R * nmat), dim3(256), rargs,
                                                   rlds_panel, st));
            } else {
                BGW_HIP(hipLaunchCooperativeKernel((const void *)k_gje_panel<0>, dim3(R * nmat), dim3(256), args, lds,
                                                   st));
            }
            bar_done += nb;
            BGW_TRY(gje_apply(A, n, nmat, ks, nb, GjeCols{k, ke, ks, ks + nb}, ipiv, Rs, st));
        }
        BGW_TRY(gje_apply(A, n, nmat, k, ke - k, GjeCols{0, n, k, ke}, ipiv, Rs, st));
    }
    return BGW_OK;
}

static int launch_gje_unpermute(double2 *A, int n, int nmat, const int *ipiv, int *idx, hipStream_t st) {
    const size_t plds = sizeof(int) * 2 * (size_t)n;
    BGW_HIP(hipFuncSetAttribute((const void *)k_gje_perm, hipFuncAttributeMaxDynamicSharedMemorySize, (int)plds));
    hipLaunchKernelGGL(k_gje_perm, dim3(nmat), dim3(256), plds, st, ipiv, n, idx);
    if (n > 8192) {
        if (n > 256 * kColPermPer) return BGW_ERR_UNSUPPORTED;
        hipLaunchKernelGGL(k_gje_colperm_reg, dim3(n, nmat), dim3(256), 0, st, A, n, idx);
        BGW_HIP(hipGetLastError());
        return BGW_OK;
    }
    const size_t rlds = sizeof(double2) * (size_t)n;
    BGW_HIP(hipFuncSetAttribute((const void *)k_gje_colperm, hipFuncAttributeMaxDynamicSharedMemorySize, (int)rlds));
    hipLaunchKernelGGL(k_gje_colperm, dim3(n, nmat), dim3(256), rlds, st, A, n, idx);
    BGW_HIP(hipGetLastError());
    return BGW_OK;
}

// Largest group of matrices inverted together: for cooperative panels, the
// matrices whose panel workgroups can be co-resident; one-workgroup panels
// need no co-residency (the cap bounds the workspace).
int gje_max_group(int n) {
    if (gje_one_wg(n)) return 64;
    const int rows = gje_rows_per_wg(n);
    const int R = (n + rows - 1) / rows;
    const size_t lds = gje_panel_lds(rows, R);
    int per_cu = 0;
    if (hipFuncSetAttribute((const void *)k_gje_panel<kPanelMax>, hipFuncAttributeMaxDynamicSharedMemorySize,
                            (int)lds) != hipSuccess)
        return 1;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, (const void *)k_gje_panel<kPanelMax>, 256, lds) !=
            hipSuccess ||
        per_cu <= 0)
        return 1;
    int dev = 0, cus = 0;
    (void)hipGetDevice(&dev);
    (void)hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    const long long slots = (long long)per_cu * cus;
    return (int)std::max<long long>(1, slots / R);
}


// ---------------------------------------------------------------------------
// Inversion without row interchanges, for chi Hermitian and negative
// semidefinite: chi0 at zero and at imaginary frequency, where every weight
// of the chi sum is negative.  With S = diag(v^1/2) (v > 0),
//   eps = 1 - v chi = S epst S^-1,   epst = 1 - S chi S,
// and epst is Hermitian with every eigenvalue >= 1.  Every leading principal
// block of epst is then >= 1 as well, so each elimination pivot (the ratio
// of consecutive leading minors, the same for eps and epst because a
// diagonal similarity keeps every principal minor) is real and >= 1:
// elimination needs no interchanges, and without them Gauss-Jordan is
// exactly as stable as on the Hermitian positive definite epst.  The column
// steps then need no search over the rows, and only the diagonal block of a
// panel is eliminated step by step:
//   k_nsd_check  max over (G, G') of sqrt(v_G v_G') |chi_GG' - conj chi_G'G|
//                and of sqrt(v_G v_G') |chi_GG'| (read before epsilon is
//                built in place), +inf when some v <= 0 or a value is not
//                finite;
//   k_nsd_build  epsilon, or epst;
//   k_nsd_diag   one workgroup per matrix inverts the panel's 64 x 64 diagonal
//                block, watching every pivot;
//   k_nsd_rows   the rest of the panel, one 64-term MFMA product per element;
//   k_nsd_update the rank update of the other columns, by outer blocks of one
//                panel (n < 3000) or two: the matrix then streams through memory
//                once per 128 columns, which at n = 4000 is what the MFMAs need.
// epst is Hermitian exactly where chi is, and elimination keeps it so up to a sign
// (rows eliminated against rows that are not: the conjugate transpose changes
// sign).  Such a matrix is therefore eliminated as epst, on and above the diagonal
// only: half the products.  W = Dinv R of the panel's rows R is also, conjugate
// transposed, the panel's columns, so that both operands of the update lie in rows.
// k_nsd_unscale makes the whole eps^-1 of it.  A matrix that is Hermitian only to
// 1e-8, not to the last bit (the lower triangle then holds information of its own; chi
// of the chi sum is, but not every product that is Hermitian on paper), is
// eliminated in general form, as eps, by the same launches; which of the two is
// decided on the device, from k_nsd_check.
// A matrix whose chi is not Hermitian to 1e-8 (relative, on the symmetrised
// scale) or has v <= 0 gets info = -2; one with a pivot whose real part is
// below 1/2, or that is not real to half of it, gets info = -3 (chi not
// negative semidefinite).  Either way epsinv is unspecified.
//
// Bounds and figures.  n = 1500: 2.35 -> 1.29 ms, three launches a panel, of which
// the diagonal block (a serial chain) takes 23 of 53 us, the update 20, the rows 8.
// Four matrices of 4000: 41.3 -> 22.6 ms, 17.2 of them in the update at 61 TFLOP/s
// of FP64 MFMA.  k_nsd_diag: 51 -> 23 us; its 64 pivots take 7.5 us of that (one
// wave, no LDS round trip or barrier per pivot), the MFMA steps 5, loads, stores
// and the launch the rest.  k_nsd_rows: 12.3 -> 8 us at n = 1500.  The general form takes
// twice the products: 1500 2.69 -> 1.47 ms, eight of 1500 7.59 -> 6.02, four of 4000 48.0
// -> 38.0.  (The Hermitian form's two k_nsd_inner launches per two panels, which return
// at once, are 0.2 of its 22.5 ms there.)
constexpr int kNsdNb = 64;        // panel width (diagonal block size)
constexpr int kNsdDiagThreads = 768;
constexpr int kNsdTile = 32;      // tile of the Hermitian check and of the unscaling
constexpr double kNsdHermTol = 1e-8;

__device__ __forceinline__ void atomic_max_nonneg(double *p, double x) {
    // non-negative doubles order like their bit patterns
    atomicMax((unsigned long long *)p, (unsigned long long)__double_as_longlong(x));
}

// Upper tile pairs (I <= J) of each matrix; chk[mat] = {non-Hermiticity, max}.
__global__ __launch_bounds__(256) void k_nsd_check(const double2 *__restrict__ chi, const double *__restrict__ v,
                                                   int n, int tiles, double *__restrict__ chk) {
    __shared__ double2 T[kNsdTile][kNsdTile + 1];
    __shared__ double red[2][4];
    const int mat = blockIdx.y;
    // blockIdx.x enumerates the pairs I <= J row by row
    int I = 0, rem = blockIdx.x;
    while (rem >= tiles - I) {
        rem -= tiles - I;
        ++I;
    }
    const int J = I + rem;
    const double2 *C = chi + (size_t)mat * n * n;
    const int tid = threadIdx.x, tx = tid & 31, ty = tid >> 5;
    const int I0 = I * kNsdTile, J0 = J * kNsdTile;
#pragma unroll
    for (int r = 0; r < kNsdTile; r += 8) {  // T[a][b] = chi[J0 + a][I0 + b]
        const int a = ty + r, row = J0 + a, col = I0 + tx;
        T[a][tx] = (row < n && col < n) ? C[(size_t)row * n + col] : make_double2(0.0, 0.0);
    }
    __syncthreads();
    double nh = 0.0, mx = 0.0;
    const int j = J0 + tx;
    const double vj = j < n ? v[j] : 1.0;
#pragma unroll
    for (int r = 0; r < kNsdTile; r += 8) {
        const int i = I0 + ty + r;
        if (i < n && j < n) {
            const double vi = v[i];
            const double2 x = C[(size_t)i * n + j];
            const double2 y = T[tx][ty + r];  // chi[j][i]
            const double sc = sqrt(vi * vj);
            double d = sc * sqrt((x.x - y.x) * (x.x - y.x) + (x.y + y.y) * (x.y + y.y));
            double m = sc * fmax(sqrt(x.x * x.x + x.y * x.y), sqrt(y.x * y.x + y.y * y.y));
            if (!(vi > 0.0) || !(vj > 0.0) || !(d <= DBL_MAX) || !(m <= DBL_MAX)) d = m = INFINITY;
            if (x.x != y.x || x.y != -y.y) d = fmax(d, DBL_MIN);  // zero only where the two are equal
            nh = fmax(nh, d);
            mx = fmax(mx, m);
        }
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        nh = fmax(nh, __shfl_xor(nh, off, 64));
        mx = fmax(mx, __shfl_xor(mx, off, 64));
    }
    if ((tid & 63) == 0) {
        red[0][tid >> 6] = nh;
        red[1][tid >> 6] = mx;
    }
    __syncthreads();
    if (tid == 0) {
        for (int w = 1; w < 4; ++w) {
            nh = fmax(nh, red[0][w]);
            mx = fmax(mx, red[1][w]);
        }
        atomic_max_nonneg(chk + 2 * mat, nh);
        atomic_max_nonneg(chk + 2 * mat + 1, mx);
    }
}

// The form a matrix takes (see above): Hermitian to the last bit, or general.  (To a few
// roundings of the largest element is not enough: with a head of v(q0 + 0) the small
// elements of the lower triangle then hold more than their rounding.)
__device__ __forceinline__ bool nsd_hermitian(const double *chk, int mat) {
    return chk[2 * mat] == 0.0 && chk[2 * mat + 1] <= DBL_MAX;
}

// epst (every 64-block on or above the diagonal) or eps.  One row per workgroup, grid
// (n, matrices); chi and out may be the same.
__global__ __launch_bounds__(256) void k_nsd_build(const double2 *chi, const double *__restrict__ v, int n,
                                                   const double *__restrict__ chk, double2 *out) {
    const int i = blockIdx.x;
    const size_t row = ((size_t)blockIdx.y * n + i) * n;
    const double vi = v[i], si = sqrt(vi);
    const bool herm = nsd_hermitian(chk, blockIdx.y);
    for (int j = (herm ? i & ~(kNsdNb - 1) : 0) + threadIdx.x; j < n; j += 256) {
        const double2 x = chi[row + j];
        const double f = herm ? si * sqrt(v[j]) : vi;
        out[row + j] = make_double2((i == j ? 1.0 : 0.0) - f * x.x, -f * x.y);
    }
}

// eps^-1 = S X S^-1 of a Hermitian matrix from the upper triangle of X = epst^-1, in
// place; tile pairs (I <= J) row by row, grid (pairs, matrices).
__global__ __launch_bounds__(256) void k_nsd_unscale(double2 *__restrict__ A, const double *__restrict__ v, int n,
                                                     int tiles, const double *__restrict__ chk) {
    __shared__ double2 X[kNsdTile][kNsdTile + 1];
    __shared__ double sv[2][kNsdTile], rv[2][kNsdTile];
    if (!nsd_hermitian(chk, blockIdx.y)) return;
    int I = 0, rem = blockIdx.x;
    while (rem >= tiles - I) {
        rem -= tiles - I;
        ++I;
    }
    const int J = I + rem, tid = threadIdx.x, tx = tid & 31, ty = tid >> 5;
    const int I0 = I * kNsdTile, J0 = J * kNsdTile;
    double2 *Am = A + (size_t)blockIdx.y * n * n;
    if (tid < 2 * kNsdTile) {
        const int g = (tid < kNsdTile ? I0 : J0) + tx;
        const double s = g < n ? sqrt(v[g]) : 1.0;
        sv[tid >> 5][tx] = s;
        rv[tid >> 5][tx] = 1.0 / s;
    }
#pragma unroll
    for (int r = 0; r < kNsdTile; r += 8) {
        const int i = I0 + ty + r, j = J0 + tx;
        X[ty + r][tx] = (i < n && j < n) ? Am[(size_t)i * n + j] : make_double2(0.0, 0.0);
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kNsdTile; r += 8) {
        const int i = I0 + ty + r, j = J0 + tx;
        if (i <= j && j < n) {
            const double f = sv[0][ty + r] * rv[1][tx];
            Am[(size_t)i * n + j] = make_double2(f * X[ty + r][tx].x, f * X[ty + r][tx].y);
        }
        const int h = J0 + ty + r, g = I0 + tx;  // the mirrored element (h, g)
        if (g < h && h < n) {
            const double f = sv[1][ty + r] * rv[0][tx];
            Am[(size_t)h * n + g] = make_double2(f * X[tx][ty + r].x, -f * X[tx][ty + r].y);
        }
    }
}

// c += a b, complex, four terms of the contraction
__device__ __forceinline__ void cmfma(double4_t &re, double4_t &im, double2 a, double2 b) {
    re = __builtin_amdgcn_mfma_f64_16x16x4f64(a.x, b.x, re, 0, 0, 0);
    im = __builtin_amdgcn_mfma_f64_16x16x4f64(a.x, b.y, im, 0, 0, 0);
    re = __builtin_amdgcn_mfma_f64_16x16x4f64(-a.y, b.y, re, 0, 0, 0);
    im = __builtin_amdgcn_mfma_f64_16x16x4f64(a.y, b.x, im, 0, 0, 0);
}

// x of lane C of every group of 16 lanes, and of lane 16 G + (own lane mod 16)
template <int C>
__device__ __forceinline__ double row_lane(double x) {
    return __longlong_as_double(__builtin_amdgcn_mov_dpp(__double_as_longlong(x), 0x150 + C, 0xf, 0xf, true));
}
template <int G>
__device__ __forceinline__ double group_lane(double x, int lane) {
    const long long b = __double_as_longlong(x);
    const int at = (16 * G + (lane & 15)) * 4;
    const int lo = __builtin_amdgcn_ds_bpermute(at, (int)b), hi = __builtin_amdgcn_ds_bpermute(at, (int)(b >> 32));
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}
template <int L>
__device__ __forceinline__ double one_lane(double x) {
    const long long b = __double_as_longlong(x);
    const int lo = __builtin_amdgcn_readlane((int)b, L), hi = __builtin_amdgcn_readlane((int)(b >> 32), L);
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

// Gauss-Jordan step C of a 16 x 16 block held by one wave, lane (r, g) = (lane mod 16,
// lane / 16) with columns 4 g .. 4 g + 3 of row r: with inv = 1 / pivot and the
// multipliers q_r = (old column C) inv, except q_C = -inv, every other column's
// entry becomes (r == C ? 0 : old) - q_r (old row C) and column C becomes -q_r.
template <int C>
__device__ __forceinline__ void inv16_step(double2 (&d)[4], int lane, bool &bad) {
    constexpr int Q = C % 4, G = C / 4;
    const bool prow = (lane & 15) == C, pcol = (lane >> 4) == G;
    const double2 p = make_double2(one_lane<16 * G + C>(d[Q].x), one_lane<16 * G + C>(d[Q].y));
    const double2 f = make_double2(group_lane<G>(d[Q].x, lane), group_lane<G>(d[Q].y, lane));
    bad |= !(p.x >= 0.5 && fabs(p.y) <= 0.5 * p.x);
    // 1 / |p|^2 (p >= 1/2, or the result is of no use) to an ulp: two Newton steps
    const double den = fma(p.x, p.x, p.y * p.y);
    double rden = __builtin_amdgcn_rcp(den);
    rden = fma(fma(-den, rden, 1.0), rden, rden);
    rden = fma(fma(-den, rden, 1.0), rden, rden);
    const double2 inv = make_double2(p.x * rden, -p.y * rden);
    double2 q = cmul(f, inv);
    if (prow) q = make_double2(-inv.x, -inv.y);
    const double keep = prow ? 0.0 : 1.0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int c = (C + 1 + i) % 4;  // the next pivot's column first
        const double2 row = make_double2(row_lane<C>(d[c].x), row_lane<C>(d[c].y));
        d[c] = cfms(make_double2(keep * d[c].x, keep * d[c].y), q, row);
    }
    if (pcol) d[Q] = make_double2(-q.x, -q.y);
}
template <int... C>
__device__ __forceinline__ void inv16(double2 (&d)[4], int lane, bool &bad, std::integer_sequence<int, C...>) {
    (inv16_step<C>(d, lane, bad), ...);
}

// D = A[K, K], K = [ks, ks + nb), padded to 64 with the identity, inverted in place and
// into Dinv (the whole 64 x 64), no interchanges, by blocks of 16: with Dk the
// inverse of diagonal block k,
//   row block k:     W = Dk D[k, :]       (k_th columns: Dk)
//   other blocks:    D[a, b] -= D[a, k] W[b],  D[a, k] = -D[a, k] Dk.
// One workgroup per matrix, D in LDS; 12 waves, one 16 x 16 MFMA product each per
// block step, wave 0 with the next diagonal block, which it then inverts in its
// registers while the others finish.
__global__ __launch_bounds__(kNsdDiagThreads) void k_nsd_diag(double2 *__restrict__ A, int n, int ks, int nb,
                                                              double2 *__restrict__ Dinv,
                                                              const double *__restrict__ chk, int *__restrict__ info) {
    constexpr int LD = 17;                          // padded rows of 16
    __shared__ double2 D[kNsdNb * kNsdNb];
    __shared__ double2 Cb[kNsdNb * LD];             // column block k before the step
    __shared__ double2 Dk[16 * LD];                 // inverse of diagonal block k
    const int mat = blockIdx.x;
    double2 *Am = A + (size_t)mat * n * n;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int li = lane & 15, lk = lane >> 4;
    for (int e = tid; e < kNsdNb * kNsdNb; e += kNsdDiagThreads) {
        const int i = e / kNsdNb, j = e % kNsdNb;
        D[e] = (i < nb && j < nb) ? Am[(size_t)(ks + i) * n + ks + j] : make_double2(i == j ? 1.0 : 0.0, 0.0);
    }
    __syncthreads();
    bool bad = false;
    const int nk = (nb + 15) / 16;
    // step -1 only inverts block 0 (the inversion's code, which every launch fetches
    // anew, stands once)
#pragma unroll 1
    for (int k = -1; k < nk; ++k) {
        if (k >= 0) {
            if (wave < 3) {  // W, in place of row block k
                const int b = (k + 1 + wave) & 3;
                double2 x[4];
#pragma unroll
                for (int t = 0; t < 4; ++t) x[t] = D[(16 * k + 4 * t + lk) * kNsdNb + 16 * b + li];
                double4_t re = {0.0, 0.0, 0.0, 0.0}, im = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
                for (int t = 0; t < 4; ++t) cmfma(re, im, Dk[li * LD + 4 * t + lk], x[t]);
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    D[(16 * k + 4 * r + lk) * kNsdNb + 16 * b + li] = make_double2(re[r], im[r]);
            } else if (wave < 6) {  // column block k, kept for the updates
                const int a = (k + wave - 2) & 3;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int i = 16 * a + 4 * r + lk;
                    Cb[i * LD + li] = D[i * kNsdNb + 16 * k + li];
                }
            } else if (wave == 6) {
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    D[(16 * k + 4 * r + lk) * kNsdNb + 16 * k + li] = Dk[(4 * r + lk) * LD + li];
            }
            __syncthreads();
        }
        // block (a, b): -D[a, k] Dk at b = k, else D[a, b] - D[a, k] W[b] (the product summed by
        // itself and added once: summed onto D, each MFMA would round at D's size)
        const int a = (k + 1 + wave / 4) & 3, b = (k + 1 + wave % 4) & 3;
        double4_t re = {0.0, 0.0, 0.0, 0.0}, im = {0.0, 0.0, 0.0, 0.0};
        double2 old[4];
#pragma unroll
        for (int r = 0; r < 4; ++r)
            old[r] = b == k ? make_double2(0.0, 0.0) : D[(16 * a + 4 * r + lk) * kNsdNb + 16 * b + li];
        if (k >= 0) {
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const double2 x = Cb[(16 * a + li) * LD + 4 * t + lk];
                cmfma(re, im, make_double2(-x.x, -x.y), D[(16 * k + 4 * t + lk) * kNsdNb + 16 * b + li]);
            }
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            re[r] += old[r].x;
            im[r] += old[r].y;
        }
        if (wave == 0 && k + 1 < nk) {  // the next diagonal block (4 r + lk, li), inverted into Dk
            double2 d[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) Dk[(4 * r + lk) * LD + li] = make_double2(re[r], im[r]);
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
            for (int c = 0; c < 4; ++c) d[c] = Dk[li * LD + 4 * lk + c];
            inv16(d, lane, bad, std::make_integer_sequence<int, 16>{});
#pragma unroll
            for (int c = 0; c < 4; ++c) Dk[li * LD + 4 * lk + c] = d[c];
        } else if (k >= 0) {
#pragma unroll
            for (int r = 0; r < 4; ++r)
                D[(16 * a + 4 * r + lk) * kNsdNb + 16 * b + li] = make_double2(re[r], im[r]);
        }
        __syncthreads();
    }
    double2 *Dm = Dinv + (size_t)mat * kNsdNb * kNsdNb;
    for (int e = tid; e < kNsdNb * kNsdNb; e += kNsdDiagThreads) {
        const int i = e / kNsdNb, j = e % kNsdNb;
        const double2 x = D[e];
        if (i < nb && j < nb) Am[(size_t)(ks + i) * n + ks + j] = x;
        Dm[e] = x;
    }
    if (tid == 0) {
        if (ks == 0) {
            const double nh = chk[2 * mat], mx = chk[2 * mat + 1];
            if (!(mx <= DBL_MAX && nh <= kNsdHermTol * mx)) info[mat] = -2;
        }
        if (bad && info[mat] == 0) info[mat] = -3;
    }
}

// The rest of panel K = [ks, ks + nb) of outer block O = [k, ke), 16 rows and columns g
// outside K per workgroup, one 16 x 16 MFMA tile of 64 terms per wave.
//
// Hermitian: W = Dinv R with R = A[K, g] (g before K: -conj(A[g, K])); R to Rs for
// g outside O, W in place of A[K, g] and, before K, conj(W) in place of A[g, K].  An
// outer block of two panels K1, K2 takes two passes: the first (MODE 1) leaves W1
// = D1 R1 and R2 - D21 W1 in rows K1 and K2; the second (MODE 2), after K2's
// diagonal block has been inverted, W2 = D2 (R2 - D21 W1) and W1 - (D1 D12) W2,
// which together are O's inverse applied to (R1, R2).  For g in O itself R stands
// for the identity's columns, and rows K of those columns become O's inverse; D1 D12
// is handed from the first pass to the second in Rs's unused columns K1, transposed.
//
// General: A[g, K] = -A[g, K] Dinv, and A[K, g] to Rs and zeroed.
template <int MODE>
__global__ __launch_bounds__(256) void k_nsd_rows(double2 *__restrict__ A, int n, int k, int ke, int ks, int nb,
                                                  const double2 *__restrict__ Dinv, double2 *__restrict__ Rs, int nbo,
                                                  const double *__restrict__ chk) {
    __shared__ double2 Wl[kNsdNb * 16];
    const int mat = blockIdx.y;
    double2 *Am = A + (size_t)mat * n * n, *R = Rs + (size_t)mat * nbo * n;
    const double2 *Dm = Dinv + (size_t)mat * kNsdNb * kNsdNb;
    const bool herm = nsd_hermitian(chk, mat);
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int li = lane & 15, lk = lane >> 4;
    const int g0 = blockIdx.x * 16, g = g0 + li, T0 = 16 * wave;
    const bool live = g < n, outer = g0 < k || g0 >= ke, own = g0 >= ks && g0 < ks + kNsdNb;
    const bool low = herm && g0 < k;
    const int K2 = k + kNsdNb, nb2 = ke - K2;  // MODE 1 and 2
    if (own && (MODE == 0 || !herm)) return;
    double4_t re = {0.0, 0.0, 0.0, 0.0}, im = {0.0, 0.0, 0.0, 0.0};
    if (own) {  // the identity's columns
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const double2 x = Dm[(T0 + 4 * r + lk) * kNsdNb + (g - ks)];
            re[r] = x.x;
            im[r] = x.y;
        }
    } else {
        double2 a[16], b[16];
#pragma unroll
        for (int s = 0; s < 16; ++s) {
            const int t = 4 * s + lk;
            a[s] = Dm[t * kNsdNb + T0 + li];
            b[s] = make_double2(0.0, 0.0);
            if (live && t < nb)
                b[s] = !herm || (low && MODE != 2) ? Am[(size_t)g * n + ks + t] : Am[(size_t)(ks + t) * n + g];
        }
        if (herm) {
#pragma unroll
            for (int s = 0; s < 16; ++s) {
                a[s].y = -a[s].y;  // Dinv[T][t] = conj(Dinv[t][T])
                if (low && MODE != 2) b[s].x = -b[s].x;
            }
            if (MODE != 2 && outer && live) {
#pragma unroll
                for (int s = 0; s < 16; ++s)
                    if (s / 4 == wave && 4 * s + lk < nb) R[(size_t)(4 * s + lk) * n + g] = b[s];
            }
        }
#pragma unroll
        for (int s = 0; s < 16; ++s) cmfma(re, im, a[s], b[s]);
    }
    if (MODE != 0 && herm) {
#pragma unroll
        for (int r = 0; r < 4; ++r) Wl[(T0 + 4 * r + lk) * 16 + li] = make_double2(re[r], im[r]);
    }
    __syncthreads();  // the block's reads are done, and Wl is there
    if (!herm) {
        const int at = MODE == 2 && outer ? kNsdNb : 0;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int t = T0 + 4 * r + lk;
            if (live && t < nb) {
                Am[(size_t)g * n + ks + t] = make_double2(-re[r], -im[r]);
                double2 *x = Am + (size_t)(ks + t) * n + g;
                R[(size_t)(at + t) * n + g] = *x;
                *x = make_double2(0.0, 0.0);
            }
        }
        return;
    }
    if (MODE == 0) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int t = T0 + 4 * r + lk;
            if (live && t < nb) {
                Am[(size_t)(ks + t) * n + g] = make_double2(re[r], im[r]);
                if (low) Am[(size_t)g * n + ks + t] = make_double2(re[r], -im[r]);
            }
        }
        return;
    }
    // the second product, summed by itself and then added: MODE 1 R2 - D21 W1, MODE 2 W1 -
    // (D1 D12) W2 (in every lane: the a of a lane past n is other lanes' operand)
    double4_t re2 = {0.0, 0.0, 0.0, 0.0}, im2 = {0.0, 0.0, 0.0, 0.0};
    double2 old[4];
    const bool in1 = g0 >= k && g0 < K2, in2 = g0 >= K2 && g0 < ke;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int t = T0 + 4 * r + lk;
        double2 x = make_double2(0.0, 0.0);
        if (MODE == 1) {
            if (live && !in1 && t < nb2) {
                x = low ? Am[(size_t)g * n + K2 + t] : Am[(size_t)(K2 + t) * n + g];
                if (low) x.x = -x.x;
                if (outer) R[(size_t)(kNsdNb + t) * n + g] = x;
            }
        } else if (live && !in2) {
            x = Am[(size_t)(k + t) * n + g];
        }
        old[r] = x;
    }
#pragma unroll
    for (int s = 0; s < 16; ++s) {
        const int t = 4 * s + lk;
        double2 a = make_double2(0.0, 0.0);
        if (MODE == 1) {
            if (T0 + li < nb2) a = Am[(size_t)(k + t) * n + K2 + T0 + li];  // conj(D21)
            a.x = -a.x;
        } else {
            if (t < nb2) a = R[(size_t)t * n + k + T0 + li];
            a = make_double2(-a.x, -a.y);
        }
        cmfma(re2, im2, a, Wl[t * 16 + li]);
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int t = T0 + 4 * r + lk;
        const double2 w = make_double2(re[r], im[r]), x = make_double2(old[r].x + re2[r], old[r].y + im2[r]);
        if (!live) continue;
        if (MODE == 1) {
            if (t < nb2) Am[(size_t)(K2 + t) * n + g] = x;
            if (in2) R[(size_t)(g - K2) * n + k + t] = w;
            else if (!in1) Am[(size_t)(k + t) * n + g] = w;
        } else {
            Am[(size_t)(k + t) * n + g] = x;
            if (low) Am[(size_t)g * n + k + t] = make_double2(x.x, -x.y);
            if (t < nb2 && !in2) {
                Am[(size_t)(K2 + t) * n + g] = w;
                if (low) Am[(size_t)g * n + K2 + t] = make_double2(w.x, -w.y);
            }
        }
    }
}

// One T x T tile of A at (I0, J0) plus s (the product), columns below jend.
template <int T, bool PLAIN>
__device__ __forceinline__ void nsd_tile(double2 *__restrict__ Am, int n, const PqOp &P, const PqOp &Q, int nbr,
                                         int I0, int J0, int jend, double s, PqLds<T> &lds) {
    double4_t cre[T / 32][T / 32], cim[T / 32][T / 32];
    double2 old[T / 32][T / 32][4];
    pq_sums<T, false, PLAIN>(P, Q, nullptr, I0, J0, 0, nbr, cre, cim, lds, [&] {
        pq_each<T>([&](int a, int b, int r, int i, int j) {
            old[a][b][r] = make_double2(0.0, 0.0);
            if (I0 + i < n && J0 + j < jend) old[a][b][r] = Am[(size_t)(I0 + i) * n + J0 + j];
        });
    });
    pq_each<T>([&](int a, int b, int r, int i, int j) {
        if (I0 + i < n && J0 + j < jend)
            Am[(size_t)(I0 + i) * n + J0 + j] =
                make_double2(fma(s, cre[a][b][r], old[a][b][r].x), fma(s, cim[a][b][r], old[a][b][r].y));
    });
}

// General form, inside an outer block of two panels: A[:, c0 .. c0 + 63] += A[:, K] R,
// the rows of R in Rs's columns c0 ...  Grid (64-row tiles, matrices).
__global__ __launch_bounds__(256) void k_nsd_inner(double2 *__restrict__ A, int n, int ks, int nb, int c0, int c1,
                                                   const double2 *__restrict__ Rs, int nbo,
                                                   const double *__restrict__ chk) {
    __shared__ PqLds<64> lds;
    if (nsd_hermitian(chk, blockIdx.y)) return;
    double2 *Am = A + (size_t)blockIdx.y * n * n;
    nsd_tile<64, true>(Am, n, {Am + ks, n, n}, {Rs + (size_t)blockIdx.y * nbo * n, n, c1}, nb, 64 * blockIdx.x, c0, c1,
                       1.0, lds);
}

// Bands of 8 tile rows, columns from the band's first row on: item u of a matrix.
__host__ __device__ inline int nsd_items(int nt) {
    int m = 0;
    for (int b = 0; b < nt; b += 8) m += 8 * (nt - b);
    return m;
}

// Rank-nbr update by outer block O = [k, ke) of everything outside it.  Hermitian: with W
// in rows O of A and R in Rs, tiles on and above the diagonal: A[i, j] -+= conj(W[:,
// i]) R[:, j] (+ for rows before O, whose part of column O has changed sign).
// General: A[:, j] += A[:, O] R[:, j].  Grid (items, a multiple of 8; matrices): an
// XCD takes a contiguous eighth of a matrix's bands, so that the panels its blocks
// share stay in its L2.
template <int T>
__global__ __launch_bounds__(256, 2) void k_nsd_update(double2 *__restrict__ A, int n, int k, int ke,
                                                       const double2 *__restrict__ Rs, int nbo,
                                                       const double *__restrict__ chk) {
    __shared__ PqLds<T> lds;
    constexpr int SUB = 64 / T;
    const int nt = (n + 63) / 64;
    double2 *Am = A + (size_t)blockIdx.y * n * n;
    const PqOp Q = {Rs + (size_t)blockIdx.y * nbo * n, n, n};
    const int per = gridDim.x / 8;
    if (nsd_hermitian(chk, blockIdx.y)) {
        const int item = (blockIdx.x % 8) * per + blockIdx.x / 8;
        int u = item / (SUB * SUB), b = 0;
        const int sub = item % (SUB * SUB);
        while (b < nt && u >= 8 * (nt - b)) {
            u -= 8 * (nt - b);
            b += 8;
        }
        const int I0 = (b + u % 8) * 64 + T * (sub / SUB), J0 = (b + u / 8) * 64 + T * (sub % SUB);
        if (b >= nt || I0 / 64 > J0 / 64 || I0 >= n || J0 >= n) return;
        if ((I0 >= k && I0 < ke) || (J0 >= k && J0 < ke)) return;
        nsd_tile<T, false>(Am, n, {Am + (size_t)k * n, n, n}, Q, ke - k, I0, J0, n, I0 < k ? 1.0 : -1.0, lds);
        return;
    }
    const int nT = (n + T - 1) / T;
    for (int u = blockIdx.x; u < nT * nT; u += gridDim.x) {
        const int I0 = (u % nT) * T, J0 = (u / nT) * T;
        if (J0 >= k && J0 < ke) continue;
        nsd_tile<T, true>(Am, n, {Am + k, n, n}, Q, ke - k, I0, J0, n, 1.0, lds);
    }
}

namespace {
struct NsdWs {
    double2 *Rs, *Dinv;
    double *chk;
};
NsdWs nsd_layout(void *ws, int n, int nmat, int nall) {
    char *p = align256((char *)ws);
    NsdWs w;
    w.chk = (double *)p; p = align256(p + sizeof(double) * 2 * (size_t)nall);
    w.Dinv = (double2 *)p; p = align256(p + sizeof(double2) * (size_t)nmat * kNsdNb * kNsdNb);
    w.Rs = (double2 *)p;
    return w;
}
}  // namespace

// Workspace of the interchange-free inversion: nmat matrices per group,
// nall matrices checked at once.
size_t nsd_workspace_bytes(int n, int nmat, int nall) {
    return 256 + ((sizeof(double) * 2 * (size_t)nall + 255) / 256) * 256 +
           ((sizeof(double2) * (size_t)nmat * kNsdNb * kNsdNb + 255) / 256) * 256 +
           sizeof(double2) * (size_t)nmat * gje_outer_nb(n) * n + 256;
}

int launch_nsd_check(const double2 *chi, const double *v, int n, int nall, int nmat, void *ws, hipStream_t st) {
    NsdWs w = nsd_layout(ws, n, nmat, nall);
    hipLaunchKernelGGL(k_fill_u32, dim3(1), dim3(256), 0, st, (unsigned int *)w.chk, (size_t)4 * nall, 0u);
    const int tiles = (n + kNsdTile - 1) / kNsdTile;
    const long long pairs = (long long)tiles * (tiles + 1) / 2;
    for (int m0 = 0; m0 < nall; m0 += 65535) {
        const int mm = std::min(65535, nall - m0);
        hipLaunchKernelGGL(k_nsd_check, dim3((unsigned)pairs, mm), dim3(256), 0, st, chi + (size_t)m0 * n * n, v, n,
                           tiles, w.chk + 2 * (size_t)m0);
    }
    BGW_HIP(hipGetLastError());
    return BGW_OK;
}

// epst or eps of every matrix (chi and out may be the same), after the check.
int launch_nsd_build(const double2 *chi, const double *v, int n, int nall, int nmat, double2 *out, void *ws,
                     hipStream_t st) {
    NsdWs w = nsd_layout(ws, n, nmat, nall);
    for (int m0 = 0; m0 < nall; m0 += 65535) {
        const int mm = std::min(65535, nall - m0);
        hipLaunchKernelGGL(k_nsd_build, dim3(n, mm), dim3(256), 0, st, chi + (size_t)m0 * n * n, v, n,
                           (const double *)w.chk + 2 * (size_t)m0, out + (size_t)m0 * n * n);
    }
    BGW_HIP(hipGetLastError());
    return BGW_OK;
}

template <int T>
static void launch_nsd_update(double2 *A, int n, int nmat, int k, int ke, const double2 *Rs, int nbo,
                              const double *chk, hipStream_t st) {
    const int items = nsd_items((n + 63) / 64) * (64 / T) * (64 / T);
    hipLaunchKernelGGL(HIP_KERNEL_NAME(k_nsd_update<T>), dim3((items + 7) / 8 * 8, nmat), dim3(256), 0, st, A, n, k, ke,
                       Rs, nbo, chk);
}

// In place: A[nmat][n][n] (matrices m0 .. m0 + nmat of the checked set).
int launch_nsd_invert(double2 *A, const double *v, int n, int nmat, int m0, int nall, int *info, void *ws,
                      hipStream_t st) {
    NsdWs w = nsd_layout(ws, n, nmat, nall);
    const double *chk = w.chk + 2 * (size_t)m0;
    double2 *Rs = w.Rs;
    hipLaunchKernelGGL(k_fill_u32, dim3(1), dim3(64), 0, st, (unsigned int *)info, (size_t)nmat, 0u);
    const int nbo = gje_outer_nb(n);
    const dim3 rg((n + 15) / 16, nmat), dg(nmat), t256(256), tdiag(kNsdDiagThreads), ig((n + 63) / 64, nmat);
    const int nt = (n + 63) / 64;
    // 64-wide tiles from eight per CU on, as for k_gje_update; in 64- and in 32-wide ones:
    // one matrix of 1500 (300 of them) 1.37 and 1.30 ms, one of 2500 (820) 3.27 and 2.97,
    // four of 1500 (1200) 2.49 and 2.51, one of 3100 (1225) 4.61 and 4.60, one of 4000 (2016)
    // 7.65 and 7.76, two of 3100 (2450) 6.91 and 7.18, four of 4000 (8064) 22.5 and 24.1
    const bool wide = (long long)nmat * nt * (nt + 1) / 2 >= 2000;
    for (int k = 0; k < n; k += nbo) {
        const int ke = std::min(n, k + nbo), K2 = k + kNsdNb;
        const int nb = std::min(kNsdNb, ke - k), nb2 = ke - K2;
        hipLaunchKernelGGL(k_nsd_diag, dg, tdiag, 0, st, A, n, k, nb, w.Dinv, chk, info);
        if (nb2 <= 0) {
            if (n <= nb) break;  // one panel is the whole matrix
            hipLaunchKernelGGL(HIP_KERNEL_NAME(k_nsd_rows<0>), rg, t256, 0, st, A, n, k, ke, k, nb, w.Dinv, Rs, nbo, chk);
        } else {
            hipLaunchKernelGGL(HIP_KERNEL_NAME(k_nsd_rows<1>), rg, t256, 0, st, A, n, k, ke, k, nb, w.Dinv, Rs, nbo, chk);
            hipLaunchKernelGGL(k_nsd_inner, ig, t256, 0, st, A, n, k, nb, K2, ke, Rs, nbo, chk);
            hipLaunchKernelGGL(k_nsd_diag, dg, tdiag, 0, st, A, n, K2, nb2, w.Dinv, chk, info);
            hipLaunchKernelGGL(HIP_KERNEL_NAME(k_nsd_rows<2>), rg, t256, 0, st, A, n, k, ke, K2, nb2, w.Dinv, Rs, nbo,
                               chk);
            hipLaunchKernelGGL(k_nsd_inner, ig, t256, 0, st, A, n, K2, nb2, k, K2, Rs, nbo, chk);
        }
        if (n > ke - k) {
            if (wide) launch_nsd_update<64>(A, n, nmat, k, ke, Rs, nbo, chk, st);
            else launch_nsd_update<32>(A, n, nmat, k, ke, Rs, nbo, chk, st);
        }
    }
    const int tiles = (n + kNsdTile - 1) / kNsdTile;
    hipLaunchKernelGGL(k_nsd_unscale, dim3(tiles * (tiles + 1) / 2, nmat), t256, 0, st, A, v, n, tiles, chk);
    BGW_HIP(hipGetLastError());
    return BGW_OK;
}

}  // namespace bgw
