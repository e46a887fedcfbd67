// The chi sum (epsilon section, static chi equation and its compact matrix
// form): chi(omega) = pf * M^H diag(w(omega)) M over the composite pair index
// t = (k*nv + v)*nc + c, on FP64 MFMA, for a whole batch of (q, omega)
// problems in one persistent launch.
//
// Complex arithmetic uses a real embedding along the contraction index: with
// M = A + iB and X = [A; B] interleaved per pair (k = 2t + part, which is the
// memory order of interleaved complex), Re chi = X_w^T X and
// Im chi = X_w^T Y with Y_{2t} = B_t, Y_{2t+1} = -A_t and X_w = diag(w) X.
// Only tiles on or above the diagonal are computed; the finalize kernel
// reduces the K-splits in a fixed order (bitwise reproducible), applies the
// prefactor and mirrors the lower triangle as the conjugate transpose.
#include <algorithm>

#include "common.h"
#include "f64_tile.h"

namespace bgw {

// Energy weights of one vector, Delta_t = (E_v,k+q - E_c,k) / Ha (see WeightKind):
//   imaginary axis:  w = Delta / (Delta^2 + omega^2)
//   real axis:       the real or the imaginary part of
//                    (1/2) [1/(Delta - E -+ i delta) + 1/(Delta + E +- i delta)],
//                    with a = Delta - E, b = Delta + E:
//                    Re = (a / (a^2 + delta^2) + b / (b^2 + delta^2)) / 2,
//                    Im = +-(delta / (a^2 + delta^2) - delta / (b^2 + delta^2)) / 2
//                    (the retarded sign; the finalize negates the advanced sum).
// grid.y: vector; every block strides over that vector's pairs.
__global__ void k_weights(const WProb *__restrict__ probs) {
    const WProb P = probs[blockIdx.y];
    const long long K = (long long)P.nk * P.nv * P.nc;
    for (long long t = blockIdx.x * (long long)blockDim.x + threadIdx.x; t < K;
         t += (long long)gridDim.x * blockDim.x) {
        const long long c = t % P.nc, kv = t / P.nc;
        const long long k = kv / P.nv;
        const double d = (P.ev[kv] - P.ec[k * P.nc + c]) / kHartreeEv;
        double w;
        if (P.kind == kWeightGiven) {
            w = P.ev[t];
        } else if (P.kind == kWeightImag) {
            w = d / (d * d + P.omega_ha * P.omega_ha);
        } else {
            const double a = d - P.omega_ha, b = d + P.omega_ha, dl = P.delta_ha;
            const double da = a * a + dl * dl, db = b * b + dl * dl;
            if (P.kind == kWeightRealRe) {
                w = 0.5 * (a / da + b / db);
            } else {
                w = 0.5 * (dl / da - dl / db);
            }
        }
        P.w[t] = w;
    }
}

namespace {
// One T x T tile of sum_t conj(P[t][G]) w_t Q[t][H] over t in [k0, k1): raw sums
// (no prefactor) to o, rows of ldo (tile rows >= P.n or columns >= Q.n are dropped).
template <int T, bool W>
__device__ __forceinline__ void pq_tile(const PqOp &P, const PqOp &Q, const double *__restrict__ w, int G0, int H0,
                                        long long k0, long long k1, double2 *__restrict__ o, long long ldo,
                                        PqLds<T> &lds) {
    double4_t cre[T / 32][T / 32], cim[T / 32][T / 32];
    pq_sums<T, W, false>(P, Q, w, G0, H0, k0, k1, cre, cim, lds, [] {});
    global_double2 *og = as_global(o);
    pq_each<T>([&](int a, int b, int r, int g, int h) {
        if (G0 + g < P.n && H0 + h < Q.n) {
            global_double2 &e = og[(size_t)(G0 + g) * ldo + H0 + h];
            e.x = cre[a][b][r];
            e.y = cim[a][b][r];
        }
    });
}

// The chi-sum tile: P = Q = M, rows of ng, weights w.
template <int T>
__device__ __forceinline__ void herk_tile(const double2 *__restrict__ M, int ng, const double *__restrict__ w,
                                          int G0, int H0, long long k0, long long k1, double2 *__restrict__ o,
                                          PqLds<T> &lds) {
    const PqOp op = {M, ng, ng};
    pq_tile<T, true>(op, op, w, G0, H0, k0, k1, o, ng, lds);
}
}  // namespace

// Persistent batched rank-K update for one output-tile size T.  Problem p
// owns the items p.item0 .. p.item0 + p.nitems (a multiple of 8).  Blocks
// stride over the items of the whole batch with a grid that is a multiple of
// 8, so item i always runs on XCD i % 8 (workgroups are dealt to the XCDs
// round-robin).  Within a problem, XCD x takes the x-th contiguous eighth of
// the (K split, tile) sequence, split-major with tiles in grouped order:
// the blocks resident on one XCD then stream the same K range of nearby row
// and column blocks of M through its L2.  Uneven problems (many q with
// different ng, many omega) share one launch per tile size.
template <int T>
__global__ __launch_bounds__(256, 3) void k_herk_f64(const HerkProb *__restrict__ probs, int nprob, long long i0,
                                                  long long i1) {
    __shared__ PqLds<T> lds;
    for (long long item = i0 + blockIdx.x; item < i1; item += gridDim.x) {
        int lo = 0, hi = nprob - 1;  // last problem with item0 <= item
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (probs[mid].item0 <= item) lo = mid;
            else hi = mid - 1;
        }
        const HerkProb &P = probs[lo];
        const long long local = item - P.item0;
        const long long chunk = P.nitems / 8;  // items per XCD
        const long long u = (local % 8) * chunk + local / 8;
        const long long ntile = (long long)P.nt * (P.nt + 1) / 2;
        if (u >= ntile * P.ns) continue;  // padding item
        const int split = (int)(u / ntile);
        int ti, tj;
        grouped_tile((int)(u % ntile), P.nt, ti, tj);
        const long long k0 = split * P.kper;
        const long long k1 = min(P.K, k0 + P.kper);
        herk_tile<T>(P.M, P.ng, P.w, ti * T, tj * T, k0, k1, P.out + (size_t)split * P.ng * P.ng, lds);
    }
}

// chi[G][H] (+)= pf * (A_GH + i B_GH), where A (and B, when part_im is set)
// are Hermitian with raw upper-triangle sums part[s][G][H], G <= H, reduced
// over the K splits s in fixed order; below the diagonal A_GH = conj(A_HG).
// Without B (imaginary axis) chi is Hermitian and its diagonal exactly real.
// In place (ns == 1, no B) chi's upper triangle holds the raw sums.  Row and
// column `skip` (>= 0) are left untouched (written by the FP64 head kernel).
// A block takes 8 x 32 tiles on or above the diagonal: it sums each element
// once and writes the mirror, in rows, through LDS (four matrices of 4000: 1.09 ms
// with the mirror's sums read down the columns, 0.29 now).
// grid.y: output matrix.
__global__ __launch_bounds__(256) void k_chi_finalize(const FinProb *__restrict__ probs) {
    __shared__ double2 tile[kFinRows][kFinTile + 1];
    const FinProb P = probs[blockIdx.y];
    const int ng = P.ng, nt = (ng + kFinTile - 1) / kFinTile, nr = (ng + kFinRows - 1) / kFinRows;
    const int tx = threadIdx.x % kFinTile, ty = threadIdx.x / kFinTile, mx = threadIdx.x % kFinRows, my = threadIdx.x / kFinRows;
    const size_t total = (size_t)ng * ng;
    const global_double2 *part = as_global(P.inplace ? P.chi : P.part), *part_im = as_global(P.part_im);
    global_double2 *chi = as_global(P.chi);
    auto store = [&](int G, int H, double2 val) {
        if (G == P.skip || H == P.skip) return;
        global_double2 &e = chi[(size_t)G * ng + H];
        if (P.accumulate) val = make_double2(e.x + val.x, e.y + val.y);
        e.x = val.x;
        e.y = val.y;
    };
    for (int u = blockIdx.x; u < nr * nt; u += gridDim.x) {
        const int G0 = u / nt * kFinRows, H0 = u % nt * kFinTile, G = G0 + ty, H = H0 + tx;
        if (G0 >= H0 + kFinTile) continue;
        const size_t at = (size_t)min(G, ng - 1) * ng + min(H, ng - 1);
        // (outside the matrix an element inside is summed, and dropped)
        double2 a = make_double2(0.0, 0.0), b = a;
        const int ns = P.inplace ? 1 : P.ns;
#pragma unroll 8
        for (int p = 0; p < ns; ++p) a = make_double2(a.x + part[p * total + at].x, a.y + part[p * total + at].y);
        if (P.part_im) {
#pragma unroll 8
            for (int p = 0; p < ns; ++p) b = make_double2(b.x + part_im[p * total + at].x, b.y + part_im[p * total + at].y);
            if (P.neg_im) b = make_double2(-b.x, -b.y);
        }
        if (G == H) a.y = b.y = 0.0;
        tile[ty][tx] = make_double2(P.pf * (a.x + b.y), P.pf * (b.x - a.y));
        __syncthreads();
        if (G <= H && H < ng) store(G, H, make_double2(P.pf * (a.x - b.y), P.pf * (a.y + b.x)));
        const int g = G0 + mx, h = H0 + my;  // the mirror
        if (g < h && h < ng) store(h, g, tile[mx][my]);
        __syncthreads();
    }
}

// C = P^H Q (rows t of P and Q contracted) for one problem, all T x T tiles of
// the m x n result, the contraction cut into ns ranges: raw sums of range s
// to out + s m n.  A persistent grid strides over the (range, tile) items.
template <int T>
__global__ __launch_bounds__(256, 3) void k_gemm_phq(const GemmProb G) {
    __shared__ PqLds<T> lds;
    const long long ntile = (long long)G.ntr * G.ntc;
    for (long long item = blockIdx.x; item < ntile * G.ns; item += gridDim.x) {
        const long long split = item / ntile, tile = item % ntile;
        const int tr = (int)(tile / G.ntc), tc = (int)(tile % G.ntc);
        const long long k0 = split * G.kper, k1 = min(G.K, k0 + G.kper);
        pq_tile<T, false>({G.P, G.ldp, G.m}, {G.Q, G.ldq, G.n}, nullptr, tr * T, tc * T, k0, k1,
                          G.out + (size_t)split * G.m * G.n, G.n, lds);
    }
}

// C (+)= scale * sum over s < ns of part[s] (m x n, complex).
__global__ void k_gemm_finalize(const double2 *__restrict__ part, int ns, long long mn, double scale,
                                double2 *__restrict__ C, int accumulate) {
    for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < mn; e += (long long)gridDim.x * blockDim.x) {
        double2 a = make_double2(0.0, 0.0);
        for (int p = 0; p < ns; ++p) a = cadd(a, part[p * mn + e]);
        a = make_double2(scale * a.x, scale * a.y);
        C[e] = accumulate ? cadd(C[e], a) : a;
    }
}

// MT[G][t] = M[t][G] for the K x ng matrix M (pairs x G), row `head` of MT
// zeroed (head < 0: none): the contraction over G of the Bethe-Salpeter
// exchange kernel becomes the contraction over the leading index that the
// chi-sum kernels perform.  grid.z batches: matrix z starts at M + z K ng and
// MT + z ng K.  32 x 32 tiles through LDS, both sides coalesced; grid
// (ceil(ng / 32), ceil(K / 32), batches), block (32, 8).
__global__ __launch_bounds__(256) void k_transpose_pairs(const double2 *__restrict__ M, long long K, int ng,
                                                         int head, double2 *__restrict__ MT) {
    __shared__ double2 tile[32][33];
    M += (size_t)blockIdx.z * K * ng;
    MT += (size_t)blockIdx.z * K * ng;
    const int g0 = blockIdx.x * 32;
    const long long t0 = (long long)blockIdx.y * 32;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const long long t = t0 + threadIdx.y + 8 * r;
        const int g = g0 + threadIdx.x;
        tile[threadIdx.y + 8 * r][threadIdx.x] = (t < K && g < ng) ? M[t * ng + g] : make_double2(0.0, 0.0);
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int g = g0 + threadIdx.y + 8 * r;
        const long long t = t0 + threadIdx.x;
        if (g < ng && t < K)
            MT[(size_t)g * K + t] = g == head ? make_double2(0.0, 0.0) : tile[threadIdx.x][threadIdx.y + 8 * r];
    }
}

// Self-energy operands.  w[i ng + G] = v[G] for i < ninner (the bare
// exchange's weights along the contraction index (i, G)).
__global__ void k_sigma_weights(const double *__restrict__ v, int ng, int ninner, double *__restrict__ w) {
    const long long n = (long long)ng * ninner;
    for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < n; e += (long long)gridDim.x * blockDim.x)
        w[e] = v[e % ng];
}

// WT[k][g] = conj(W[g][k]) with W[g][k] = (einv[g][k] - ch delta_gk) v[k]: the
// screened interaction (ch = 0) or its screening part (ch = 1), transposed
// and conjugated so that sum_k conj(WT[k][g]) A[k] = (W A)[g].  32 x 32 tiles
// through LDS; grid (ceil(ng / 32), ceil(ng / 32)), block (32, 8).
__global__ __launch_bounds__(256) void k_sigma_wt(const double2 *__restrict__ einv, const double *__restrict__ v,
                                                  int ng, int ch, double2 *__restrict__ WT) {
    __shared__ double2 tile[32][33];
    const int k0 = blockIdx.x * 32, g0 = blockIdx.y * 32;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int g = g0 + threadIdx.y + 8 * r, k = k0 + threadIdx.x;
        double2 e = make_double2(0.0, 0.0);
        if (g < ng && k < ng) {
            e = einv[(size_t)g * ng + k];
            if (ch && g == k) e.x -= 1.0;
            e = make_double2(e.x * v[k], -e.y * v[k]);
        }
        tile[threadIdx.y + 8 * r][threadIdx.x] = e;
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int k = k0 + threadIdx.y + 8 * r, g = g0 + threadIdx.x;
        if (k < ng && g < ng) WT[(size_t)k * ng + g] = tile[threadIdx.x][threadIdx.y + 8 * r];
    }
}

// B2[i ng + G][n] = B[G][i nouter + n]: the rows of W M regrouped by inner
// state, so that the last contraction runs over (i, G).
__global__ void k_sigma_regroup(const double2 *__restrict__ B, int ng, int ninner, int nouter,
                                double2 *__restrict__ B2) {
    const long long total = (long long)ng * ninner * nouter;
    for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < total;
         e += (long long)gridDim.x * blockDim.x) {
        const int n = (int)(e % nouter);
        const long long r = e / nouter;
        const int G = (int)(r % ng), i = (int)(r / ng);
        B2[e] = B[((size_t)G * ninner + i) * nouter + n];
    }
}

// ---------------------------------------------------------------- launchers

int launch_transpose_pairs(const double2 *M, long long K, int ng, int head, double2 *MT, hipStream_t st,
                           int batches) {
    hipLaunchKernelGGL(k_transpose_pairs, dim3((ng + 31) / 32, (unsigned)((K + 31) / 32), batches), dim3(32, 8), 0,
                       st, M, K, ng, head, MT);
    BGW_HIP(hipGetLastError());
    return BGW_OK;
}

int launch_weights_batch(const WProb *probs, int nprob, long long maxK, hipStream_t st) {
    const int blocks = (int)std::max<long long>(1, std::min<long long>((maxK + 255) / 256, 1024));
    hipLaunchKernelGGL(k_weights, dim3(blocks, nprob), dim3(256), 0, st, probs);
    BGW_HIP(hipGetLastError());
    return BGW_OK;
}

int herk_blocks_per_cu() {
    static int n = 0;
    if (!n) {
        int a = 0, b = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&a, k_herk_f64<64>, 256, 0) != hipSuccess || a < 1) a = 1;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&b, k_herk_f64<32>, 256, 0) != hipSuccess || b < 1) b = 1;
        // three blocks (three waves per SIMD) keep the MFMAs fed; a fourth would only add K splits
        n = std::min({a, b, 3});
    }
    return n;
}

// Items [i0, i1) all have output tile `tile`.
int launch_herk_batch(const HerkProb *probs, int nprob, long long i0, long long i1, int tile, int grid,
                      hipStream_t st) {
    if (i1 <= i0) return BGW_OK;
    const long long g = std::max<long long>(1, std::min<long long>(i1 - i0, grid));
    if (tile == 64) hipLaunchKernelGGL(k_herk_f64<64>, dim3((unsigned)g), dim3(256), 0, st, probs, nprob, i0, i1);
    else hipLaunchKernelGGL(k_herk_f64<32>, dim3((unsigned)g), dim3(256), 0, st, probs, nprob, i0, i1);
    BGW_HIP(hipGetLastError());
    return BGW_OK;
}

int device_cus();

int launch_gemm_phq(const GemmProb &G, int tile, hipStream_t st) {
    const long long items = (long long)G.ntr * G.ntc * G.ns;
    const long long g = std::max<long long>(1, std::min<long long>(items, (long long)device_cus() * 3));
    if (tile == 64) hipLaunchKernelGGL(k_gemm_phq<64>, dim3((unsigned)g), dim3(256), 0, st, G);
    else hipLaunchKernelGGL(k_gemm_phq<32>, dim3((unsigned)g), dim3(256), 0, st, G);
    BGW_HIP(hipGetLastError());
    return BGW_OK;
}

int launch_gemm_finalize(const double2 *part, int ns, long long mn, double scale, double2 *C, int accumulate,
                         hipStream_t st) {
    const int blocks = (int)std::max<long long>(1, std::min<long long>((mn + 255) / 256, 8192));
    hipLaunchKernelGGL(k_gemm_finalize, dim3(blocks), dim3(256), 0, st, part, ns, mn, scale, C, accumulate);
    BGW_HIP(hipGetLastError());
    return BGW_OK;
}

int launch_sigma_weights(const double *v, int ng, int ninner, double *w, hipStream_t st) {
    const long long n = (long long)ng * ninner;
    hipLaunchKernelGGL(k_sigma_weights, dim3((unsigned)std::min<long long>((n + 255) / 256, 4096)), dim3(256), 0, st,
                       v, ng, ninner, w);
    BGW_HIP(hipGetLastError());
    return BGW_OK;
}

int launch_sigma_wt(const double2 *einv, const double *v, int ng, int ch, double2 *WT, hipStream_t st) {
    hipLaunchKernelGGL(k_sigma_wt, dim3((ng + 31) / 32, (ng + 31) / 32), dim3(32, 8), 0, st, einv, v, ng, ch, WT);
    BGW_HIP(hipGetLastError());
    return BGW_OK;
}

int launch_sigma_regroup(const double2 *B, int ng, int ninner, int nouter, double2 *B2, hipStream_t st) {
    const long long n = (long long)ng * ninner * nouter;
    hipLaunchKernelGGL(k_sigma_regroup, dim3((unsigned)std::min<long long>((n + 255) / 256, 8192)), dim3(256), 0, st,
                       B, ng, ninner, nouter, B2);
    BGW_HIP(hipGetLastError());
    return BGW_OK;
}

int launch_finalize_batch(const FinProb *probs, int nprob, int maxng, hipStream_t st) {
    const int nt = (maxng + kFinTile - 1) / kFinTile, nr = (maxng + kFinRows - 1) / kFinRows;
    const int blocks = std::max(1, std::min(nr * nt, 65536 / std::max(1, nprob) + 1));
    hipLaunchKernelGGL(k_chi_finalize, dim3(blocks, nprob), dim3(256), 0, st, probs);
    BGW_HIP(hipGetLastError());
    return BGW_OK;
}

}  // namespace bgw
