// FP64 complex tile products on MFMA, operands straight from memory to LDS: the
// loop of the chi sum, the self-energy and the rank updates of epsilon^-1.
#pragma once

#include <algorithm>

#include "common.h"

namespace bgw {

typedef double double4_t __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) void lds_void_t;

constexpr int KC = 8;  // complex pairs per LDS stage

// Two LDS stages of a T-column tile: [stage][P, Q][KC pairs][T columns] complex.
template <int T>
struct PqLds {
    __attribute__((aligned(1024))) unsigned char b[2][2][KC * T * 16];
};

// An operand of a tile product, contracted over t: value (t, g) at p[t ld + g]
// (or, for P of a plain product, at p[g ld + t]), g < n.
struct PqOp {
    const double2 *p;
    long long ld;
    int n;
};

// What one block loads: waves 0 and 1 P, waves 2 and 3 Q.
struct PqSrc {
    const double2 *base;  // the wave's operand at the tile's first column (plain P: at its first row)
    long long ld;
    int bytes;            // of a row from there on, at most T columns (plain P: rows left of the operand)
    const double *w;
};

// Workgroup barrier: this wave's loads have landed, the weights among them, and
// its LDS reads are done.  (The load wait is the builtin, so that the compiler
// knows of it; the weights are named so that their loads stay before it.)
__device__ __forceinline__ void pq_meet(double (&wt)[KC / 4]) {
#pragma unroll
    for (int s = 0; s < KC / 4; ++s) asm volatile("" : "+v"(wt[s]));
    __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0)
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// One stage's rows straight into LDS and its weights into registers.  A row past
// k1 and a column past the operand's end read as zero (the buffers' range
// checks), so the loop has no tail and no vector address arithmetic.
//
// P of a plain product (PLAIN) is contracted along its rows: eight rows of 8
// values per load, the 16-byte slot of value c in row r being c ^ (r / 2 mod 8),
// so that the 16 rows that a read takes at one c fall on different banks.
template <int T, bool W, bool PLAIN>
__device__ __forceinline__ void pq_issue(unsigned char *__restrict__ stage, double (&wt)[KC / 4], const PqSrc &S,
                                         long long kk, long long k1, int wave, int lane) {
    if (PLAIN && wave < 2) {
        constexpr int NL = T / 16;  // loads of this wave
        unsigned char *dst = stage + wave * (T / 2) * 128;
        const int left = (int)min((long long)KC, k1 - kk);
        int off[2];
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const int c = (lane & 7) ^ (4 * q + (lane >> 4));
            off[q] = c < left ? ((lane >> 3) * (int)S.ld + c) * 16 : -16;  // -16: out of range, zero
        }
#pragma unroll
        for (int i = 0; i < NL; ++i) {
            const int row = wave * (T / 2) + 8 * i, rows = min(8, S.bytes - row);
            const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(
                (void *)(S.base + (long long)row * S.ld + kk), 0,
                rows > 0 ? ((rows - 1) * (int)S.ld + left) * 16 : 0, 0x00020000);
            __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (lds_void_t *)(dst + i * 1024), 16, off[i & 1], 0, 0, 0);
        }
    } else {
        unsigned char *dst = stage + ((wave >> 1) * KC + 4 * (wave & 1)) * T * 16;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const long long t = kk + 4 * (wave & 1) + i;
            const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(
                (void *)(S.base + t * S.ld), 0, t < k1 ? S.bytes : 0, 0x00020000);
            if (T == 64 || lane < T)
                __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (lds_void_t *)(dst + i * T * 16), 16, 16 * lane, 0, 0, 0);
        }
    }
    if (W) {
        const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(
            (void *)(S.w + kk), 0, (int)max(0ll, min((long long)KC, k1 - kk)) * 8, 0x00020000);
#pragma unroll
        for (int s = 0; s < KC / 4; ++s) {
            const auto v = __builtin_amdgcn_raw_buffer_load_b64(r, 8 * (lane >> 4) + 32 * s, 0, 0);
            __builtin_memcpy(&wt[s], &v, 8);
        }
    }
}

// The MFMAs of one stage `cur` while the next one comes into `nxt` (distinct
// restrict-qualified buffers: the loads in flight do not alias the reads).
// Four pairs at a time: lane (li, lk) reads the complex values of pair lk, one
// 16-byte read per operand block, and its real and imaginary parts feed two
// MFMAs each; the only vector arithmetic is w a and a sign, per block of P.
template <int T, bool W, bool PLAIN, bool LAST>
__device__ __forceinline__ void pq_step(const unsigned char *__restrict__ cur, unsigned char *__restrict__ nxt,
                                        double (&wt)[KC / 4], const PqSrc &S, long long kk, long long k1, int wave,
                                        int lane, double4_t (&cre)[T / 32][T / 32], double4_t (&cim)[T / 32][T / 32]) {
    constexpr int NB = T / 32, WT = T / 2;
    const int wr = wave >> 1, wc = wave & 1, li = lane & 15, lk = lane >> 4;
    double wn[KC / 4] = {};
    if (!LAST) pq_issue<T, W, PLAIN>(nxt, wn, S, kk + KC, k1, wave, lane);
    __builtin_amdgcn_sched_barrier(0);
    const unsigned char *A =
        PLAIN ? cur + (wr * WT + li) * 128 + ((lk ^ (li >> 1)) * 16) : cur + (lk * T + wr * WT + li) * 16;
    const unsigned char *A4 = PLAIN ? cur + (wr * WT + li) * 128 + (((4 + lk) ^ (li >> 1)) * 16) : A;
    const unsigned char *B = cur + (KC * T + lk * T + wc * WT + li) * 16;
#pragma unroll
    for (int s = 0; s < KC / 4; ++s) {
        double2 a[NB], b[NB];
#pragma unroll
        for (int i = 0; i < NB; ++i) {
            a[i] = *reinterpret_cast<const double2 *>(PLAIN ? (s ? A4 : A) + i * 16 * 128
                                                            : A + (4 * s * T + 16 * i) * 16);
            b[i] = *reinterpret_cast<const double2 *>(B + (4 * s * T + 16 * i) * 16);
        }
        // conj(a) b, or a b: the product of the two imaginary parts has the sign
        // in the one, that of a's imaginary and b's real part in the other
#pragma unroll
        for (int i = 0; i < NB; ++i) {
            if (W) a[i] = make_double2(wt[s] * a[i].x, wt[s] * a[i].y);
#pragma unroll
            for (int j = 0; j < NB; ++j) {
                cre[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[i].x, b[j].x, cre[i][j], 0, 0, 0);
                cim[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[i].x, b[j].y, cim[i][j], 0, 0, 0);
            }
        }
#pragma unroll
        for (int i = 0; i < NB; ++i) {
            const double na = -a[i].y;
#pragma unroll
            for (int j = 0; j < NB; ++j) {
                cre[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(PLAIN ? na : a[i].y, b[j].y, cre[i][j], 0, 0, 0);
                cim[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(PLAIN ? a[i].y : na, b[j].x, cim[i][j], 0, 0, 0);
            }
        }
    }
    __builtin_amdgcn_sched_barrier(0);  // the loads have all the MFMAs' time to land
    pq_meet(wn);
#pragma unroll
    for (int s = 0; s < KC / 4; ++s) wt[s] = wn[s];
}

// What bounds the tiles: the FP64 MFMAs, 16 of 64 cycles per wave and four pairs
// (T = 64), and with them every vector instruction: the two do not overlap on
// FP64, so the loop holds only what the sums need.  Loads go straight to LDS with
// scalar addresses, and operands stay interleaved complex, read 16 bytes at a
// time.  One static sum over 102400 pairs at 1500 vectors: 17.46 -> 15.27 ms per
// call, against 14.5 ms with the LDS reads and MFMAs alone
// and 12.2 ms at the rate of a large library FP64 product; the
// self-energy of 404 x 64 bands at 1500 vectors, 9.45 -> 8.48 ms.  8 pairs a stage: 16
// take 64 KB of LDS, fewer blocks fit a CU, and it was 16.7 ms.
//
// One T x T tile of sum_t conj(P[t][G]) w_t Q[t][H] (w_t = 1 without weights;
// PLAIN: sum_t P[G][t] Q[t][H]) over t in [k0, k1): 4 waves in a 2 x 2 layout,
// each owning a (T/2) x (T/2) block of 16 x 16 MFMA tiles, the sums of block (a,
// b) in cre[a][b] and cim[a][b] (pq_each visits them).  `last` runs before the
// last stage's MFMAs, where loads for the epilogue have them to land in.
template <int T, bool W, bool PLAIN, class Last>
__device__ __forceinline__ void pq_sums(const PqOp &P, const PqOp &Q, const double *__restrict__ w, int G0, int H0,
                                        long long k0, long long k1, double4_t (&cre)[T / 32][T / 32],
                                        double4_t (&cim)[T / 32][T / 32], PqLds<T> &lds, Last last) {
    constexpr int NB = T / 32;    // MFMA tiles per wave side
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
#pragma unroll
    for (int a = 0; a < NB; ++a)
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            cre[a][b] = (double4_t){0.0, 0.0, 0.0, 0.0};
            cim[a][b] = (double4_t){0.0, 0.0, 0.0, 0.0};
        }
    PqSrc S;
    S.base = wave >= 2 ? Q.p + H0 : PLAIN ? P.p + G0 * P.ld : P.p + G0;
    S.ld = wave < 2 ? P.ld : Q.ld;
    S.bytes = wave >= 2 ? min(T, Q.n - H0) * 16 : PLAIN ? P.n - G0 : min(T, P.n - G0) * 16;
    S.w = w;
    double wt[KC / 4] = {};
    pq_issue<T, W, PLAIN>(&lds.b[0][0][0], wt, S, k0, k1, wave, lane);
    pq_meet(wt);
    unsigned char *cur = &lds.b[0][0][0], *nxt = &lds.b[1][0][0];
    long long kk = k0;
#pragma unroll 1
    for (; kk + KC < k1; kk += KC) {
        pq_step<T, W, PLAIN, false>(cur, nxt, wt, S, kk, k1, wave, lane, cre, cim);
        unsigned char *t = cur;
        cur = nxt;
        nxt = t;
    }
    last();
    pq_step<T, W, PLAIN, true>(cur, nxt, wt, S, kk, k1, wave, lane, cre, cim);
}

// f(a, b, r, G, H) for every element of this lane: register r of block (a, b) is
// tile element (G, H) (D layout of v_mfma_f64_16x16x4: lane l, register r -> row
// 4 r + l / 16, column l % 16).
template <int T, class F>
__device__ __forceinline__ void pq_each(F f) {
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
#pragma unroll
    for (int a = 0; a < T / 32; ++a)
#pragma unroll
        for (int b = 0; b < T / 32; ++b)
#pragma unroll
            for (int r = 0; r < 4; ++r)
                f(a, b, r, (wave >> 1) * (T / 2) + 16 * a + 4 * r + (lane >> 4),
                  (wave & 1) * (T / 2) + 16 * b + (lane & 15));
}

}  // namespace bgw
