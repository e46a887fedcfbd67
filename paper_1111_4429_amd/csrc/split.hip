// Split-precision chi sum: chi = pf * X_w^T (X + iY) (real embedding of
// M^H diag(w) M, see chi.hip) computed from 8-bit digit slices on INT8 MFMA
// with exact INT32 accumulation, recombined in FP64.
//
// Digits.  The pairs are cut into chunks of 384 (twelve MFMA k-steps of 32),
// each of four runs of 96.  Within a run every column G of X has a power-of-two
// scale 2^eB (above the column's max of |Re M|, |Im M|), and every column of
// X_w, for each weight vector, a scale 2^eA above the max of |w_t Re M|, |w_t
// Im M| (both found by k_split_slice in its pass over M).  A run whose max lies
// at most a factor 2 (eB) or 8 (eA) below the chunk's shares the chunk's scale, a
// lower one has its own (run_exp): the INT32 sums of a tile then run over the
// whole chunk where the pairs are alike, and end at the runs in which some
// column of the tile changes its scale.  Each scaled
// value is rounded once to a 40-bit integer N = rint(x 2^(39-e)) and written as
// five signed base-256 digits, N = sum_i d_i 256^(4-i), -128 <= d_i <= 127.
// One FMA with the constant 1.5 2^52 + 0x8080808080 makes all five: the low 40
// bits of the result's mantissa are N + 0x8080808080, whose bytes are the
// digits plus 128 (toggling each byte's top bit makes them signed bytes).
// The unweighted side's digits do not depend on the frequency: k_split_slice
// stores them once per q (5 bytes per real value).  The weighted side is
// sliced inside the GEMM from M and w, in registers, for each frequency, so no
// weighted slices are stored at all.
//
// Re chi takes (Re, Im) of the weighted side against (Re, Im) of the other, Im
// chi takes (-Im, Re) against the same.  -Im is the bitwise complement of Im's
// digits: ~d = -d - 1, so the sums come out too small by the sum of the other
// side's Re digits, which k_split_slice stores as running sums per column
// (EC) and the chunk end adds back, exactly.
//
// Products (k_chi_split): all a_i b_j with i + j = p <= 4, one INT32 sum per
// p; every sum is exact (|sum| <= 5 2^14 768 < 2^26).  Fifteen INT8 MFMA
// products per (Re, Im); at each chunk end the five sums are combined in FP64
// with the chunk scales and added to FP64 accumulators.  Dropped: products of
// weight 2^-40 of the leading one and below, and the rounding of N: in all at
// most 74 2^-40 of a run's largest product, for the shared scales (8 + 2 units of
// rounding, 4 digit products of weight 2^-40 a factor 8 x 2 up).  Four 9-bit digits
// with a scale per 96 pairs, as BF16 products need them, leave 80.  One scale per
// chunk whatever its runs hold was up to the ratio of the runs worse.  A column
// with a value that is not finite gets the exponent kNotFinite, which makes its
// sums NaN.
//
// Why INT8: the card's INT8 MFMA has twice the BF16 rate, so fifteen exact
// 8-bit products cost 3/4 of the ten BF16 products that four 9-bit digits
// need for a result sixteen times coarser, and cutting a value takes one FMA
// and about three integer instructions where the BF16 digits took a chain of
// twelve FP64 operations.
//
// The head row/column (G = 0) is recomputed in FP64 from M (k_headwing)
// because v(q+G) ~ 1/q^2 amplifies it in epsilon.
#include <algorithm>
#include <cstdlib>

#include "common.h"

namespace bgw {

typedef int int4_t __attribute__((ext_vector_type(4)));
typedef int int6_t __attribute__((ext_vector_type(6)));

namespace {
constexpr int KSP = 32;       // pairs per MFMA k-step (16x16x64: 64 real rows)
constexpr int NKS = 12;       // k-steps per chunk
constexpr int SKP = KSP * NKS; // pairs per chunk
constexpr int RKS = 3;        // k-steps per run (96 pairs, one exponent per column)
constexpr int NRUN = NKS / RKS;
constexpr int RP = RKS * KSP; // pairs per run
constexpr int SLACK_A = 3, SLACK_B = 1;  // powers of two by which a run may lie below the scale it shares
constexpr int UKS = 2;        // K splits are cut at multiples of this many k-steps
constexpr int KSB = 2 * KSP;  // bytes of one column's digits of one slice and k-step
constexpr int NSL = 5;        // digits (stored slices of the unweighted side, INT32 product groups)
constexpr int NCB = 3;        // 16-column blocks of a wave
constexpr int TR = 64;        // output tile rows: weighted side, sliced in registers
constexpr int TC = 32 * NCB;  // output tile columns: unweighted side, digit slices through LDS
constexpr int XT = 512;       // GEMM block: 8 waves (two per SIMD), 4 x 2 over the tile
constexpr int kMinExp = -500; // chunk exponents are clamped here (values below 2^-539 count as zero)
constexpr int kNotFinite = 3071;    // exponent of a chunk column with a value that is not finite
constexpr int kZeroRun = -0x7fff;   // raw exponent of a run without a value
constexpr int kNotFiniteA = 127;    // the same in the weighted side's exponents, bytes relative to eB
constexpr double kFixBias = 6755399441055744.0 + 551911719040.0;  // 1.5 2^52 + 0x8080808080
constexpr unsigned kToggle = 0x80808080u;

__device__ inline double pow2(int e) { return __longlong_as_double((long long)(e + 1023) << 52); }

// e with mx <= 2^e / 1.005: |N| <= 2^39 / 1.005 + 1 then stays below the
// largest five-digit value 0x7f7f7f7f7f.
__device__ inline int chunk_exp(double mx) {
    if (!(mx <= 1.7e308)) return kNotFinite;
    int e = 0;
    if (mx > 0.0) (void)frexp(mx * 1.005, &e);
    return max(e, kMinExp);
}

// Exponent of run r from the chunk's raw ones: the chunk's largest where run r lies
// at most `slack` below it, else that less a multiple of slack + 1.  A run without a
// value takes a neighbour's (it would end the sums for nothing).
__device__ inline int run_exp(const int (&e)[NRUN], int r, int slack) {
    int top = kZeroRun, x = kZeroRun;
#pragma unroll
    for (int s = 0; s < NRUN; ++s) {
        top = max(top, e[s]);
        if (e[s] != kZeroRun && (s <= r || x == kZeroRun)) x = e[s];
    }
    if (top == kNotFinite || top == kZeroRun) return top;
    return top - (top - x) / (slack + 1) * (slack + 1);
}

// A stored eB: the exponent in 12 bits, and whether the column's scale differs from that of
// the run before: its own, or with any weight vector.  (The sums of all vectors end at the
// same runs, needed or not: blocks that read the same rows of M for several vectors
// otherwise drift apart and miss L2: six real frequencies of two q with 1500 and 731
// vectors, whose weights differ by up to 2^11 within most chunks, 34.6 ms against 30.0.)
constexpr int kExpBits = 0xfff, kExpBias = 1024, kOwnChange = 0x1000, kAnyChange = 0x2000;
__device__ __forceinline__ int exp_of(int stored) { return (stored & kExpBits) - kExpBias; }

// run_exp of run r = lane mod 4 from the four lanes' maxima
__device__ inline int quad_run_exp(double mx, int slack) {
    const int raw = mx == 0.0 ? kZeroRun : chunk_exp(mx), lane = threadIdx.x & 63;
    int e[NRUN];
#pragma unroll
    for (int s = 0; s < NRUN; ++s) e[s] = __shfl(raw, (lane & ~(NRUN - 1)) + s, 64);
    return run_exp(e, lane & (NRUN - 1), slack);
}

// The digits of N = rint(x s) plus 128 in the low 40 bits: lo holds digits 4
// (low byte) to 1, the low byte of hi digit 0.
__device__ __forceinline__ void fix40(double x, double s, unsigned &lo, unsigned &hi) {
    const unsigned long long b = (unsigned long long)__double_as_longlong(fma(x, s, kFixBias));
    lo = (unsigned)b;
    hi = (unsigned)(b >> 32);
}

// Digit dwords of four values: d[i] holds digit i of values 0..3 (low byte first).
__device__ __forceinline__ void digits4(const unsigned (&lo)[4], const unsigned (&hi)[4], unsigned (&d)[NSL]) {
    const unsigned t0 = __builtin_amdgcn_perm(lo[1], lo[0], 0x05010400u);
    const unsigned t1 = __builtin_amdgcn_perm(lo[1], lo[0], 0x07030602u);
    const unsigned u0 = __builtin_amdgcn_perm(lo[3], lo[2], 0x05010400u);
    const unsigned u1 = __builtin_amdgcn_perm(lo[3], lo[2], 0x07030602u);
    const unsigned h0 = __builtin_amdgcn_perm(hi[1], hi[0], 0x0c0c0400u);
    const unsigned h1 = __builtin_amdgcn_perm(hi[3], hi[2], 0x04000c0cu);
    d[0] = (h0 | h1) ^ kToggle;
    d[1] = __builtin_amdgcn_perm(u1, t1, 0x07060302u) ^ kToggle;
    d[2] = __builtin_amdgcn_perm(u1, t1, 0x05040100u) ^ kToggle;
    d[3] = __builtin_amdgcn_perm(u0, t0, 0x07060302u) ^ kToggle;
    d[4] = __builtin_amdgcn_perm(u0, t0, 0x05040100u) ^ kToggle;
}

// max(|re|, |im|), infinity when either is not finite
__device__ __forceinline__ double abs_max(double2 z) {
    const double a = fabs(z.x), b = fabs(z.y);
    return (a <= 1.7e308 && b <= 1.7e308) ? fmax(a, b) : INFINITY;
}
}  // namespace

// Digit slices of the unweighted side for the first nst k-steps (those that hold pairs <
// K) from run r0 of one q on, chunks counted from there, and the exponents of the weighted side of every weight vector.
// Block = one chunk x 32 columns, 768 threads.  Thread t owns column G = 32
// blockIdx.x + (t/4) % 32 and, in each of the k-steps 2 (t/128) and
// 2 (t/128) + 1, the eight pairs 8 (t%4) .. +7; with this assignment every
// 16-byte store instruction of a wave writes 1 KB of contiguous slice memory.
// S: [k-step][NSL][gpad][KSB] bytes, each group of 16 holding eight pairs as
// (Re t0..t7, Im t0..t7); E: [nchunk][gpad][NRUN], eB of the chunk's runs (exp_of); EA:
// [nvec][runs][apad], eA - eB (within a byte: the size of the weights; below 2^-128 a
// weight keeps fewer digits, above 2^126 it counts as not finite).
// EC: [k-step][NSL][gpad], entry p the sum of the Re digits 0
// .. p of the column over the chunk's k-steps up to this one.  Pairs >= K are zero.
// gpad: ng rounded up to 32 (this block), apad to 16 (a load of the GEMM).
constexpr int SLICE_T = 32 * 4 * (NKS / 2);  // 768
constexpr int SLICE_V = 4;                   // weight vectors per round
__global__ __launch_bounds__(SLICE_T) void k_split_slice(const double2 *__restrict__ M, long long K, int ng, int gpad,
                                                         long long r0, int nst, unsigned char *__restrict__ S,
                                                         short *__restrict__ E, const double *__restrict__ w,
                                                         long long wstride, int nvec, signed char *__restrict__ EA,
                                                         int apad, int *__restrict__ EC) {
    constexpr int NP = 4 * RKS;        // partial maxima per column and run
    __shared__ double red[SLICE_V][4 * NKS][33];
    __shared__ int ex[NRUN][32], changed[SLICE_V][NRUN][32];
    __shared__ int dsum[NKS][NSL][32];
    __shared__ double wa[SLICE_V][SKP];  // |w| of the chunk's pairs
    __shared__ int wbad[SLICE_V][NRUN];  // a weight of the run is not finite
    const int q = threadIdx.x & 3, cl = (threadIdx.x >> 2) & 31, kh = threadIdx.x >> 7;
    const int G = blockIdx.x * 32 + cl;
    const int chunk = blockIdx.y;
    const long long tb = r0 * RP + (long long)chunk * SKP + 2 * kh * KSP + 8 * q;  // k-step i, pair j: tb + KSP i + j
    const bool col = G < ng;
    // 128 threads reduce: thread t run t % 4 of column t / 4 (its cl), for the vector t / 128 of a round
    auto run_max = [&](int v) {
        double mx = 0.0;
#pragma unroll
        for (int k = 0; k < NP; ++k) mx = fmax(mx, red[v][NP * q + k][cl]);
        return mx;
    };
    auto changes = [&](int e) {  // from the run before to this thread's
        const int before = __shfl_up(e, 1, 64);
        return q > 0 && before != e;
    };
    double2 m[2][8];  // [k-step i][pair j]
    double mr[2][8];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const long long t = tb + KSP * i + j;
            m[i][j] = (t < K && col) ? M[t * ng + G] : make_double2(0.0, 0.0);
        }
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        double mx = 0.0;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            mr[i][j] = abs_max(m[i][j]);
            mx = fmax(mx, mr[i][j]);
        }
        red[0][4 * (2 * kh + i) + q][cl] = mx;
    }
    __syncthreads();
    if (kh == 0) {
        const int e = quad_run_exp(run_max(0), SLACK_B);
        ex[q][cl] = e == kZeroRun ? 0 : e;
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int e = ex[(2 * kh + i) / RKS][cl];
        const double up = e == kNotFinite ? 0.0 : pow2(39 - e);
        unsigned d[4][NSL];  // [Re t0..3, Re t4..7, Im t0..3, Im t4..7]
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            unsigned lo[4], hi[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) fix40(m[i][4 * h + j].x, up, lo[j], hi[j]);
            digits4(lo, hi, d[h]);
#pragma unroll
            for (int j = 0; j < 4; ++j) fix40(m[i][4 * h + j].y, up, lo[j], hi[j]);
            digits4(lo, hi, d[2 + h]);
        }
        unsigned char *o = S + ((size_t)chunk * NKS + 2 * kh + i) * NSL * gpad * KSB + (size_t)G * KSB + 16 * q;
#pragma unroll
        for (int sl = 0; sl < NSL; ++sl) {
            if (chunk * NKS + 2 * kh + i < nst)
                *reinterpret_cast<uint4 *>(o + (size_t)(sl * gpad) * KSB) =
                    make_uint4(d[0][sl], d[1][sl], d[2][sl], d[3][sl]);
            int t = __builtin_amdgcn_sdot4((int)d[0][sl], 0x01010101, 0, false);
            t = __builtin_amdgcn_sdot4((int)d[1][sl], 0x01010101, t, false);
            t += __shfl_xor(t, 1, 64);
            t += __shfl_xor(t, 2, 64);
            if (q == 0) dsum[2 * kh + i][sl][cl] = t;
        }
    }
    __syncthreads();
    if (threadIdx.x < NSL * 32) {  // one thread per entry and column: running sums over the k-steps
        const int sl = threadIdx.x >> 5, c = threadIdx.x & 31;
        int run = 0;
#pragma unroll
        for (int ks = 0; ks < NKS; ++ks) {
#pragma unroll
            for (int j = 0; j < NSL; ++j) run += j <= sl ? dsum[ks][j][c] : 0;
            if (chunk * NKS + ks < nst)
                EC[(((size_t)chunk * NKS + ks) * NSL + sl) * gpad + blockIdx.x * 32 + c] = run;
        }
    }
    // weighted side: |w| max(|Re M|, |Im M|) bounds the products the GEMM rounds.  Four vectors a
    // round, their weights through LDS: a small call has few blocks, each of which goes through
    // all vectors (100 vectors, 1000 pairs, 32 frequencies: 125 us with the weights loaded by
    // every thread, 37 now).
    const int nrun = (nst + RKS - 1) / RKS, run = chunk * NRUN + q, eb = ex[q][cl];
    bool any = false;
    for (int v0 = 0; v0 < nvec; v0 += SLICE_V) {
        __syncthreads();  // the previous round has been read
        if (threadIdx.x < SLICE_V * NRUN) (&wbad[0][0])[threadIdx.x] = 0;
        double wt[SLICE_V / 2];
#pragma unroll
        for (int i = 0; i < SLICE_V / 2; ++i) {
            const int v = v0 + 2 * i + (int)threadIdx.x / SKP, p = (int)threadIdx.x % SKP;
            const long long t = r0 * RP + (long long)chunk * SKP + p;
            wt[i] = v < nvec && t < K ? fabs(w[(size_t)v * wstride + t]) : 0.0;
        }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < SLICE_V / 2; ++i) {
            const int v = 2 * i + (int)threadIdx.x / SKP, p = (int)threadIdx.x % SKP;
            wa[v][p] = wt[i];
            if (!(wt[i] <= 1.7e308)) wbad[v][p / RP] = 1;
        }
        __syncthreads();
#pragma unroll
        for (int v = 0; v < SLICE_V; ++v)
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const double *wi = &wa[v][(2 * kh + i) * KSP + 8 * q];
                double mw = 0.0;
#pragma unroll
                for (int j = 0; j < 8; ++j) mw = fmax(mw, wi[j] * mr[i][j]);
                red[v][4 * (2 * kh + i) + q][cl] = mw;
            }
        __syncthreads();
        if (kh < SLICE_V && v0 + kh < nvec) {
            const bool bad = wbad[kh][q] || eb == kNotFinite;  // (0 times infinity is lost in the maximum)
            const int e = quad_run_exp(bad ? INFINITY : run_max(kh), SLACK_A);
            int rel = e == kZeroRun ? 0 : max(e - eb, -128);
            if (e == kNotFinite || rel >= kNotFiniteA) rel = kNotFiniteA;
            any |= changes(eb + rel);
            if (run < nrun && G < apad) EA[((size_t)(v0 + kh) * nrun + run) * apad + G] = (signed char)rel;
        }
    }
    if (kh < SLICE_V) changed[kh][q][cl] = any;
    __syncthreads();
    if (kh == 0) {
        const bool own = changes(eb);
#pragma unroll
        for (int v = 1; v < SLICE_V; ++v) any |= changed[v][q][cl] != 0;
        E[((size_t)chunk * gpad + G) * NRUN + q] =
            (short)((eb + kExpBias) | (own ? kOwnChange : 0) | (own || any ? kAnyChange : 0));
    }
}

namespace {
__device__ __forceinline__ int4_t as_int4(uint4 u) {
    int4_t r;
    __builtin_memcpy(&r, &u, 16);
    return r;
}
#define MFMA(a, b, c) __builtin_amdgcn_mfma_i32_16x16x64_i8((a), (b), (c), 0, 0, 0)

typedef __attribute__((address_space(3))) void lds_void_t;

// LDS stage of one k-step: the weighted side as FP64 complex, [32 pairs][64
// columns] (16 B each, 1 KB per pair row); the unweighted side's five digit
// slices, [slice][96 rows][64 B] with the four 16-B segments of row r stored
// in the order seg ^ ((r >> 1) & 3), so that the eight rows one 16-B read
// phase touches fall in distinct bank groups; the step's 32 weights.
// Besides the two stages, two chunk buffers hold eB of a chunk's 96 columns (int16,
// [column][run]), eA - eB of its 64 rows (int8, [run][row]), eB of its rows and the
// digit sums at the end of each run ([run][5][96] int32; of the last one at the
// item's last k-step in it): chunk c in buffer c % 2, staged with the first
// step that needs it and read where the sums start and end.  Every load to LDS is one
// of a whole wave (masked ones at the end of two branches the compiler has merged
// into one without their masks).
constexpr int A_LDS = KSP * TR * 16;          // 32 KB
constexpr int B_SLICE_LDS = TC * KSB;         // 6 KB
constexpr int W_OFF = A_LDS + NSL * B_SLICE_LDS;
constexpr int STG = W_OFF + 256;              // 62.25 KB
constexpr int EA_OFF = TC * NRUN * 2, EBR_OFF = EA_OFF + TR * NRUN, EC_OFF = EBR_OFF + 1024;
constexpr int EC_RUN = NSL * TC * 4, EC_PIECES = (NRUN * EC_RUN + 1023) / 1024, E_LDS = EC_OFF + EC_PIECES * 1024;
static_assert(EBR_OFF == 1024 && TR * NRUN * 2 <= 1024, "eB of the columns and eA - eB of the rows in one load");
constexpr int NWAVE = XT / 64;
constexpr int PA = KSP / NWAVE;               // 1-KB pieces of the A part per wave: 4
constexpr int NB_PIECES = NSL * B_SLICE_LDS / 1024;          // of the B part, all waves: 30
constexpr int PB = (NB_PIECES + NWAVE - 1) / NWAVE;

// vmcnt(n) alone (expcnt and lgkmcnt left at their maxima); vmcnt is split
// over bits 3:0 and 15:14 of the immediate
#define BGW_WAIT_VM(n) __builtin_amdgcn_s_waitcnt(0x0F70 | ((n) & 0xF) | (((n) >> 4) << 14))

// Workgroup barrier for the stage pipeline: the wave's LDS reads are complete
// (lgkmcnt) and its direct-to-LDS loads have been waited for explicitly, so no
// fence is needed; __syncthreads() would also wait for the loads still in
// flight for later stages.
__device__ __forceinline__ void stage_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// Sources of one item's stage loads: wave-uniform bases and offsets (scalar
// registers) plus one constant lane offset each.
struct StageSrc {
    const char *m;           // M (bytes) at the launch's first pair
    unsigned m_row;          // ng * 16
    int m_off;               // lane's column (clamped into M), bytes
    long long kmax;          // last pair from there on
    const char *b;           // slices
    unsigned b_slice;        // bytes of one slice of a k-step: gpad * KSB
    unsigned b0;             // the tile's first column in it
    int b_last;              // last 16 columns of it from there on that are stored
    int b_off;               // lane L of a piece: row L/4, source segment (L%4) ^ ((L/8) & 3)
    const double *w;         // weights of this vector at the launch's first pair
    const short *eb;         // EB: exponents of the slices, [nch][gpad][NRUN]
    const signed char *ea;   // EA of this vector: of the weighted side, less EB's, [nrun][apad]
    const int *ec;           // EC at the tile's first column
    int gpad, apad, nrun, G0, H0, s1;  // s1: the item's last k-step + 1
};

// One k-step x into one stage.  A piece i of wave w is pair row 4w + i of the
// k-step (past K the last pair again: it meets zero digits of the other side);
// B piece p = w + 8 i is slice p / 6, rows 16 (p % 6) .. +16 (past gpad, where no sums
// are stored, the last ones again).  Wave 7 loads the step's weights (half a one per
// lane; the vectors are padded by 128 entries) and wave 6 the exponents of the step's
// chunk when they are new.
__device__ __forceinline__ void stage_issue(unsigned char *__restrict__ stage, unsigned char *__restrict__ ebuf,
                                            const StageSrc &S, int x, bool first, int wave, int lane) {
    const long long t0 = (long long)x * KSP;
    const int rows = (int)min((long long)KSP, S.kmax + 1 - t0);
    const __amdgpu_buffer_rsrc_t ra = __builtin_amdgcn_make_buffer_rsrc(
        (void *)(S.m + t0 * S.m_row), 0, (int)(rows * S.m_row), 0x00020000);
#pragma unroll
    for (int i = 0; i < PA; ++i)
        __builtin_amdgcn_raw_ptr_buffer_load_lds(ra, (lds_void_t *)(stage + (PA * wave + i) * 1024), 16, S.m_off,
                                                 (int)(min(PA * wave + i, rows - 1) * S.m_row), 0, 0);
    const unsigned b_step = NSL * S.b_slice;
    const __amdgpu_buffer_rsrc_t rb =
        __builtin_amdgcn_make_buffer_rsrc((void *)(S.b + (size_t)x * b_step), 0, (int)b_step, 0x00020000);
#pragma unroll
    for (int i = 0; i < PB; ++i) {
        const int p = wave + NWAVE * i;
        if ((i + 1) * NWAVE <= NB_PIECES || p < NB_PIECES)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(
                rb, (lds_void_t *)(stage + A_LDS + p * 1024), 16, S.b_off,
                (int)(S.b0 + (p / (TC / 16)) * S.b_slice + min(p % (TC / 16), S.b_last) * 1024), 0, 0);
    }
    if (wave == NWAVE - 1) {
        __builtin_amdgcn_global_load_lds((const void *)((const char *)(S.w + t0) + 4 * lane),
                                         (lds_void_t *)(stage + W_OFF), 4, 0, 0);
    } else if (wave == NWAVE - 2 && (first || x % NKS == 0)) {
        const int ch = x / NKS;
        int l = lane;
        asm volatile("" : "+v"(l));  // the addresses are made here: kept over the steps they cost registers
        // eB of two columns per lane, eA - eB of 16 rows per lane (a run past the last repeats it; columns and
        // rows past the matrix, whose sums are not stored, others)
        const short *eb = S.eb + (size_t)ch * S.gpad * NRUN;
        const signed char *ea = S.ea + (size_t)min(S.nrun - 1, ch * NRUN + l % 16 / (TR / 16)) * S.apad +
                                min(S.G0 + l % (TR / 16) * 16, S.apad - 16);
        const void *e = l < TC / 2 ? (const void *)(eb + min(S.H0 + 2 * l, S.gpad - 2) * NRUN) : (const void *)ea;
        __builtin_amdgcn_global_load_lds(e, (lds_void_t *)ebuf, 16, 0, 0);
        __builtin_amdgcn_global_load_lds((const void *)(eb + min(S.G0 + 2 * (l % (TR / 2)), S.gpad - 2) * NRUN),
                                         (lds_void_t *)(ebuf + EBR_OFF), 16, 0, 0);
#pragma unroll
        for (int h = 0; h < EC_PIECES; ++h) {
            const int i = min(64 * h + l, NRUN * EC_RUN / 16 - 1);  // 16 bytes: four columns of an entry of a run
            const int last = min(S.s1, ch * NKS + RKS * (i / (EC_RUN / 16) + 1)) - 1, j = i % (EC_RUN / 16);
            __builtin_amdgcn_global_load_lds(
                (const void *)(S.ec + ((size_t)last * NSL + j / (TC / 4)) * S.gpad +
                               min(j % (TC / 4) * 4, S.gpad - S.H0 - 4)),
                (lds_void_t *)(ebuf + EC_OFF + h * 1024), 16, 0, 0);
        }
    }
}

__device__ __forceinline__ uint4 bfrag(const unsigned char *slice, int row, int lq) {
    return *reinterpret_cast<const uint4 *>(slice + row * KSB + 16 * (lq ^ ((row >> 1) & 3)));
}

struct SplitAcc {
    int4_t g[NCB][NSL][2];  // [col block][group][re/im]
    double re[NCB][4], im[NCB][4];
};

// Digit fragments of this lane's eight pairs y = w_t M_t(G) 2^(39 - eA): per
// digit six dwords (~Im t0..t7, Re t0..t7, Im t0..t7).  Dwords 2..5 are the
// operand of Re chi, 0..3 the operand of Im chi, against the same fragment (Re,
// Im) of the other side.
struct SplitFrags {
    int6_t d[NSL];
};

__device__ __forceinline__ void slice_frags(const unsigned char *src, const double (&sw)[8], SplitFrags &F) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        double2 m[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) m[j] = *reinterpret_cast<const double2 *>(src + (4 * h + j) * 1024);
        unsigned lo[4], hi[4], d[NSL];
#pragma unroll
        for (int j = 0; j < 4; ++j) fix40(m[j].x, sw[4 * h + j], lo[j], hi[j]);
        digits4(lo, hi, d);
#pragma unroll
        for (int sl = 0; sl < NSL; ++sl) F.d[sl][2 + h] = (int)d[sl];
#pragma unroll
        for (int j = 0; j < 4; ++j) fix40(m[j].y, sw[4 * h + j], lo[j], hi[j]);
        digits4(lo, hi, d);
#pragma unroll
        for (int sl = 0; sl < NSL; ++sl) {
            F.d[sl][4 + h] = (int)d[sl];
            F.d[sl][h] = (int)~d[sl];
        }
    }
}

// Fifteen INT8 products per (Re, Im) of the wave's row block and one column block.
__device__ __forceinline__ void split_mfma(const SplitFrags &A, const uint4 (&bf)[NSL], int4_t (&g)[NSL][2]) {
#pragma unroll
    for (int i = 0; i < NSL; ++i)
#pragma unroll
        for (int p = i; p < NSL; ++p) {
            g[p][0] = MFMA(__builtin_shufflevector(A.d[i], A.d[i], 2, 3, 4, 5), as_int4(bf[p - i]), g[p][0]);
            g[p][1] = MFMA(__builtin_shufflevector(A.d[i], A.d[i], 0, 1, 2, 3), as_int4(bf[p - i]), g[p][1]);
        }
}

// 2^(e - 7), NaN for a column with a value that is not finite
__device__ __forceinline__ double exp_scale(int e) { return e == kNotFinite ? NAN : pow2(e - 7); }

// eB of a column, eA of a row and the digit sums at the end of run r, from a chunk's buffer
__device__ __forceinline__ int col_exp(const unsigned char *E, int c, int r) {
    return exp_of(reinterpret_cast<const short *>(E)[NRUN * c + r]);
}
__device__ __forceinline__ int row_exp(const unsigned char *E, int g, int r) {
    const int b = exp_of(reinterpret_cast<const short *>(E + EBR_OFF)[NRUN * g + r]);
    const int a = reinterpret_cast<const signed char *>(E + EA_OFF)[TR * r + g];
    return a == kNotFiniteA ? kNotFinite : a + b;
}
__device__ __forceinline__ const int *digit_sums(const unsigned char *E, int r) {
    return reinterpret_cast<const int *>(E + EC_OFF + r * EC_RUN);
}

// Bit r: some column or row of the tile changes its scale at run r.
__device__ __forceinline__ int scale_changes(const unsigned char *E, int lane) {
    const uint2 *cols = reinterpret_cast<const uint2 *>(E), *rows = reinterpret_cast<const uint2 *>(E + EBR_OFF);
    const uint2 c0 = cols[lane], c1 = cols[64 + lane % (TC - 64)], rb = rows[lane];
    constexpr unsigned own = kOwnChange * 0x10001u, any = kAnyChange * 0x10001u;
    const unsigned r01 = ((c0.x | c1.x) & own) | (rb.x & any), r23 = ((c0.y | c1.y) & own) | (rb.y & any);
    return (__ballot(r01 >> 16 != 0) ? 2 : 0) | (__ballot((r23 & 0xffff) != 0) ? 4 : 0) |
           (__ballot(r23 >> 16 != 0) ? 8 : 0);
}

// End of the sums at a run's end: the five INT32 groups combined in FP64 with the
// scales 2^(eA + eB - 14) into the FP64 accumulators.  D layout of 16x16x64: lane
// l, register r -> row 4 (l/16) + r, col l % 16.  E: the chunk's buffer.
__device__ __forceinline__ void split_flush(SplitAcc &acc, const unsigned char *E, int run, int wave, int li, int lq) {
    const int *ec = digit_sums(E, run);
    double pa[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) pa[r] = exp_scale(row_exp(E, 16 * (wave >> 1) + 4 * lq + r, run));
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb) {
        const double pb = exp_scale(col_exp(E, 16 * NCB * (wave & 1) + 16 * cb + li, run));
        int corr[NSL];
#pragma unroll
        for (int p = 0; p < NSL; ++p) corr[p] = ec[p * TC + 16 * NCB * (wave & 1) + 16 * cb + li];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            double v[2];
#pragma unroll
            for (int ri = 0; ri < 2; ++ri) {
                double x = 0.0;
#pragma unroll
                for (int p = NSL - 1; p >= 0; --p)
                    x = fma(x, 0.00390625, (double)(acc.g[cb][p][ri][r] + (ri ? corr[p] : 0)));
                v[ri] = x * pa[r];
            }
            acc.re[cb][r] = fma(v[0], pb, acc.re[cb][r]);
            acc.im[cb][r] = fma(v[1], pb, acc.im[cb][r]);
        }
        __builtin_amdgcn_sched_barrier(0);  // one column block at a time
    }
}
}  // namespace

// One k-step x: stage step x + 1 into `nxt`, slice this lane's row of the
// weighted side from `cur`, 90 MFMAs over the three column blocks, then wait
// for step x + 1's loads and meet the block at the barrier.  The two stages
// are distinct restrict-qualified buffers, so the compiler knows that the
// loads in flight into one do not alias the reads of the other.
__device__ __forceinline__ void split_step(const unsigned char *__restrict__ cur, unsigned char *__restrict__ nxt,
                                           unsigned char *__restrict__ ebuf1, const StageSrc &S, int x, int s1,
                                           double up, int wave, int lane, int li, int lq, SplitAcc &acc) {
    __builtin_amdgcn_sched_barrier(0);
    if (x + 1 < s1) stage_issue(nxt, ebuf1, S, x + 1, false, wave, lane);
    __builtin_amdgcn_sched_barrier(0);
    // the weighted side of this lane's row, sliced into digits
    SplitFrags A;
    {
        const double *wl = reinterpret_cast<const double *>(cur + W_OFF) + 8 * lq;
        double sw[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) sw[j] = wl[j] * up;
        slice_frags(cur + (8 * lq) * 1024 + (16 * (wave >> 1) + li) * 16, sw, A);
    }
    const unsigned char *Bs = cur + A_LDS;
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb) {
        uint4 bf[NSL];
#pragma unroll
        for (int sl = 0; sl < NSL; ++sl)
            bf[sl] = bfrag(Bs + sl * B_SLICE_LDS, 16 * NCB * (wave & 1) + 16 * cb + li, lq);
        split_mfma(A, bf, acc.g[cb]);
    }
    BGW_WAIT_VM(0);
    stage_barrier();
}

// Persistent split-precision chi sum over every (q, weight vector, tile, K
// split) item of a launch.  Entry q owns the items q.item0 .. q.item0 +
// q.nitems (a multiple of 8); item i always runs on XCD i % 8 (a grid that
// is a multiple of 8, workgroups dealt to the XCDs round-robin), and XCD x
// takes the x-th contiguous eighth of the entry's (split, tile, vector)
// sequence, vector fastest: the blocks resident on one XCD work on the same
// tile for consecutive weight vectors (frequencies), reading the same rows of
// M and the same slices, which their L2 then serves.  With one weight vector
// the sequence walks the tiles in bands of eight row tiles.
// Block: 8 waves, two per SIMD; wave w owns rows 16 (w/2) .. +16 and columns
// 48 (w%2) .. +48 (three column blocks) of the 64 x 96 tile, so each row is
// sliced by the two waves that share it, and one wave's slicing and LDS
// reads run under the MFMAs of the other wave on its SIMD.  Three column
// blocks, not four: 120 INT32 and 48 FP64 accumulators with 30 registers of
// digit fragments of the weighted side and 20 of the other fit the 256
// registers of a wave (one wave per SIMD with 512 lost more to the moves
// between the two halves of its register file).
// Every k-step (32 pairs) the block stages 32 pair rows of M (the tile's 64
// columns), the five digit slices of the unweighted side (96 columns) and
// the 32 weights into LDS with direct global->LDS loads, one step ahead
// through two stages; each wave slices its 16 rows of w_t M_t(G) into
// digits in registers and issues 90 MFMAs.
// What bounds it (Ng = 4000, K = 40 960, four frequencies: 69.1 ms, 2.3 POPS;
// the BF16 form took 108.4): the MFMAs alone take 42.6 ms, at the 3.7 POPS
// that the card holds on such data (4.7 on zeros: the clock falls with the
// power); reading the fragments from LDS adds 7 ms, the barrier 3, the loads
// into LDS 10 when they hit L2 and 6 more as they miss.  Ending the sums at
// every run, four times a chunk, would make it 84 ms; the real-axis sums above,
// which do so at most runs, take 27.9 ms, and 23.4 with sums over whole chunks.
// out (+)= raw sums (no prefactor) of every element of the tile inside ng x ng.
__global__ __launch_bounds__(XT, 1) void k_chi_split(const SplitQ *__restrict__ qs, int nq, long long i0,
                                                     long long i1) {
    __shared__ __attribute__((aligned(1024))) unsigned char stage0[STG];
    __shared__ __attribute__((aligned(1024))) unsigned char stage1[STG];
    __shared__ __attribute__((aligned(512))) unsigned char ebufs[2][E_LDS];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int li = lane & 15, lq = lane >> 4;

    for (long long item = i0 + blockIdx.x; item < i1; item += gridDim.x) {
        int lo = 0, hi = nq - 1;  // last entry with item0 <= item
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (qs[mid].item0 <= item) lo = mid;
            else hi = mid - 1;
        }
        const SplitQ &Q = qs[lo];
        const long long local = item - Q.item0;
        const long long per = Q.nitems / 8;  // items per XCD
        const long long u = (local % 8) * per + local / 8;
        const long long total = (long long)Q.ntiles * Q.ns * Q.nvec;
        if (u >= total) continue;  // padding item
        const int v = (int)(u % Q.nvec);
        const long long r0 = u / Q.nvec;
        const int tile = (int)(r0 % Q.ntiles);
        const int split = (int)(r0 / Q.ntiles);
        const unsigned tw = __builtin_amdgcn_readfirstlane((int)Q.tiles[tile]);  // uniform: scalar addresses
        const int G0 = (int)(tw & 0xffff) * TR, H0 = (int)(tw >> 16) * TC;
        const int ng = Q.ng, gpad = Q.gpad;

        StageSrc S;
        S.m_row = (unsigned)ng * 16;
        S.m = reinterpret_cast<const char *>(Q.M) + (long long)Q.run0 * RP * S.m_row;
        S.m_off = min(G0 + lane, ng - 1) * 16;
        S.kmax = Q.K - 1 - (long long)Q.run0 * RP;
        S.b = reinterpret_cast<const char *>(Q.SB);
        S.b_slice = (unsigned)gpad * KSB;
        S.b0 = (unsigned)H0 * KSB;
        S.b_last = (gpad - H0) / 16 - 1;
        S.b_off = (lane >> 2) * KSB + 16 * ((lane & 3) ^ ((lane >> 3) & 3));
        S.w = Q.w + (size_t)v * Q.wstride + (long long)Q.run0 * RP;
        S.eb = Q.EB;
        S.nrun = (Q.nst + RKS - 1) / RKS;
        S.apad = Q.apad;
        S.ea = Q.EA + (size_t)v * S.nrun * Q.apad;
        S.gpad = gpad;
        S.G0 = G0;
        S.H0 = H0;
        S.ec = Q.EC + H0;

        SplitAcc acc;
#pragma unroll
        for (int cb = 0; cb < NCB; ++cb)
#pragma unroll
            for (int r = 0; r < 4; ++r) acc.re[cb][r] = acc.im[cb][r] = 0.0;

        // k-steps [s0, s1) of the launch's chunk range, s0 even
        const int nu = (Q.nst + UKS - 1) / UKS;
        const int s0 = (int)((long long)split * nu / Q.ns) * UKS;
        const int s1 = min(Q.nst, (int)((long long)(split + 1) * nu / Q.ns) * UKS);
        S.s1 = s1;
        const bool in = G0 + 16 * (wave >> 1) + li < ng;  // this lane's slicing row is inside the matrix

        stage_issue(stage0, ebufs[(s0 / NKS) & 1], S, s0, true, wave, lane);
        BGW_WAIT_VM(0);
        stage_barrier();

        int cut = 0;  // of the chunk
        for (int xc = s0; xc < s1;) {  // one chunk, or the part of it with one set of scales
            const int ch = xc / NKS, run = xc % NKS / RKS;
            const unsigned char *E = ebufs[ch & 1];
            unsigned char *En = ebufs[(ch + 1) & 1];
            int xe = (ch + 1) * NKS;
            if (xc == s0 || xc % NKS == 0) cut = scale_changes(E, lane);
#pragma unroll
            for (int r = NRUN - 1; r > 0; --r)
                if (r > run && (cut >> r & 1)) xe = ch * NKS + RKS * r;
            xe = min(s1, xe);
            // slicing scale of this lane's row: 2^(39 - eA)
            const int ea = row_exp(E, 16 * (wave >> 1) + li, run);
            const double up = in && ea != kNotFinite ? pow2(39 - ea) : 0.0;
#pragma unroll
            for (int cb = 0; cb < NCB; ++cb)
#pragma unroll
                for (int p = 0; p < NSL; ++p)
#pragma unroll
                    for (int ri = 0; ri < 2; ++ri) acc.g[cb][p][ri] = (int4_t){0, 0, 0, 0};
            if (xc % NKS) {  // started inside the chunk: the digit sums before it do not belong
                const bool at_run = xc % RKS == 0;
                const int *cl = digit_sums(E, at_run ? run - 1 : 0) + 16 * NCB * (wave & 1) + li;
                const global_int *cg = as_global(S.ec + (size_t)(xc - 1) * NSL * gpad);
                int c0 = 16 * NCB * (wave & 1) + li;
                asm volatile("" : "+v"(c0));  // (as in stage_issue)
#pragma unroll
                for (int cb = 0; cb < NCB; ++cb)
#pragma unroll
                    for (int p = 0; p < NSL; ++p) {
                        const int c =
                            at_run ? -cl[p * TC + 16 * cb] : -cg[p * gpad + min(c0 + 16 * cb, gpad - H0 - 1)];
                        acc.g[cb][p][1] = (int4_t){c, c, c, c};
                    }
            }
            int x = xc;
            if (x & 1) {
                split_step(stage1, stage0, En, S, x, s1, up, wave, lane, li, lq, acc);
                ++x;
            }
#pragma unroll 1
            for (; x < xe; x += 2) {  // step x uses stage x % 2
                split_step(stage0, stage1, En, S, x, s1, up, wave, lane, li, lq, acc);
                if (x + 1 < xe) split_step(stage1, stage0, En, S, x + 1, s1, up, wave, lane, li, lq, acc);
            }
            split_flush(acc, E, (xe - 1) % NKS / RKS, wave, li, lq);
            xc = xe;
        }

        global_double2 *o = as_global(Q.out + (size_t)v * Q.vstride + (size_t)split * ng * ng);
#pragma unroll
        for (int cb = 0; cb < NCB; ++cb)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int G = G0 + 16 * (wave >> 1) + 4 * lq + r;
                const int H = H0 + 16 * NCB * (wave & 1) + 16 * cb + li;
                if (G < ng && H < ng) {
                    global_double2 &e = o[(size_t)G * ng + H];
                    double re = acc.re[cb][r], im = acc.im[cb][r];
                    if (Q.add) re += e.x, im += e.y;
                    e.x = re;
                    e.y = im;
                }
            }
        __syncthreads();  // the stages and exponent buffers are reused by the block's next item
    }
}

// FP64 head rows of every weight vector of one q in one pass over M:
// hw[s][v][H] = sum_{t in K range s} w_v[t] conj(M_t(head)) M_t(H), for the
// vectors [v0, v0 + nv) (at most kHeadVec).  grid: (ng / 256, ranges).
constexpr int kHeadVec = 16;
__global__ __launch_bounds__(256) void k_headwing(const double2 *__restrict__ M, long long K, int ng, int head,
                                                  const double *__restrict__ w, long long wstride, int v0, int nv,
                                                  long long kper, double2 *__restrict__ hw, int nvec) {
    const int H = blockIdx.x * blockDim.x + threadIdx.x;
    if (H >= ng) return;
    const long long k0 = blockIdx.y * kper, k1 = min(K, k0 + kper);
    double sr[kHeadVec], si[kHeadVec];
#pragma unroll
    for (int v = 0; v < kHeadVec; ++v) sr[v] = si[v] = 0.0;
    // four pairs' loads in flight at a time; every sum keeps the order of t
    constexpr int U = 4;
    for (long long t0 = k0; t0 < k1; t0 += U) {
        double2 p[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const long long t = t0 + u;
            if (t < k1) {
                const double2 a = M[t * ng + head], b = M[t * ng + H];
                p[u] = make_double2(a.x * b.x + a.y * b.y, a.x * b.y - a.y * b.x);  // conj(a) b
            } else {
                p[u] = make_double2(0.0, 0.0);
            }
        }
#pragma unroll
        for (int v = 0; v < kHeadVec; ++v) {
            if (v < nv) {
                const double *wv = w + (size_t)(v0 + v) * wstride;
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const double wt = t0 + u < k1 ? wv[t0 + u] : 0.0;
                    sr[v] = fma(wt, p[u].x, sr[v]);
                    si[v] = fma(wt, p[u].y, si[v]);
                }
            }
        }
    }
#pragma unroll
    for (int v = 0; v < kHeadVec; ++v)
        if (v < nv) hw[((size_t)blockIdx.y * nvec + v0 + v) * ng + H] = make_double2(sr[v], si[v]);
}

// Row and column `head` of every output matrix of one q: with A from vector
// va and (real frequency axis) B from vector vb = va + 1,
// chi[head][H] (+)= pf (A_H + i B_H), chi[H][head] (+)= pf (conj A_H + i conj B_H),
// where A_H = sum_s hw[s][va][H] (B negated with neg_im); without B, chi is Hermitian and its head
// diagonal exactly real.  grid: (ng / 256, output matrices).
__global__ void k_headwing_write(const double2 *__restrict__ hw, int nsplit, int nvec, int ng, int head, double pf,
                                 double2 *__restrict__ chi, int two, int neg_im, int accumulate) {
    const int H = blockIdx.x * blockDim.x + threadIdx.x;
    if (H >= ng) return;
    const int f = blockIdx.y;
    const int va = two ? 2 * f : f;
    double2 a = make_double2(0.0, 0.0), b = make_double2(0.0, 0.0);
    for (int p = 0; p < nsplit; ++p) a = cadd(a, hw[((size_t)p * nvec + va) * ng + H]);
    if (two)
        for (int p = 0; p < nsplit; ++p) b = cadd(b, hw[((size_t)p * nvec + va + 1) * ng + H]);
    if (neg_im) b = make_double2(-b.x, -b.y);
    if (H == head) {
        a.y = 0.0;
        b.y = 0.0;
    }
    // row: A_H + i B_H; column: conj(A_H) + i conj(B_H)
    const double2 vr = make_double2(pf * (a.x - b.y), pf * (a.y + b.x));
    const double2 vc = make_double2(pf * (a.x + b.y), pf * (-a.y + b.x));
    double2 *cm = chi + (size_t)f * ng * ng;
    const size_t rowi = (size_t)head * ng + H, coli = (size_t)H * ng + head;
    if (accumulate) {
        cm[rowi] = cadd(cm[rowi], vr);
        if (H != head) cm[coli] = cadd(cm[coli], vc);
    } else {
        cm[rowi] = vr;
        if (H != head) cm[coli] = vc;
    }
}

// ---------------------------------------------------------------- host side

int device_cus() {
    static int cus = 0;
    if (!cus) {
        int dev = 0, v = 0;
        if (hipGetDevice(&dev) == hipSuccess &&
            hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && v > 0)
            cus = v;
        else
            cus = 256;
    }
    return cus;
}

int split_gpad(int ng) { return (ng + 31) / 32 * 32; }

long long split_runs(long long K) { return (K + RP - 1) / RP; }

long long split_steps(long long K, long long run0, long long nrun) {
    return std::min(nrun * RKS, (K - run0 * RP + KSP - 1) / KSP);
}

// A split keeps at least a run (96 pairs): its partial sums cost as much as they save
// below that.
long long split_max_ns(long long K) { return split_runs(K); }

long long split_range_ns(long long nst) { return (nst + UKS - 1) / UKS; }

long long split_min_runs(long long ns) { return (ns * UKS - 1 + RKS - 1) / RKS; }

size_t split_slices_only_bytes(long long nst, int ng) { return (size_t)nst * NSL * KSB * split_gpad(ng); }

size_t split_ec_bytes(long long nst, int ng) { return sizeof(int) * (size_t)nst * NSL * split_gpad(ng); }

size_t split_slice_bytes(long long nst, int ng) {
    const long long nch = (nst + NKS - 1) / NKS;
    return split_slices_only_bytes(nst, ng) + split_ec_bytes(nst, ng) +
           sizeof(short) * NRUN * (size_t)nch * split_gpad(ng);
}

size_t split_run_bytes(int ng) { return split_slice_bytes(RKS, ng); }

int split_apad(int ng) { return (ng + 15) / 16 * 16; }

size_t split_ea_bytes(long long nvec, long long nst, int ng) {
    return (size_t)nvec * ((nst + RKS - 1) / RKS) * split_apad(ng);
}

// Upper tiles (those with some G <= H) in walk order: bands of eight row
// tiles, each band walked column tile by column tile.
void split_tiles(int ng, std::vector<unsigned> &out) {
    const int nti = (ng + TR - 1) / TR, ntj = (ng + TC - 1) / TC;
    out.clear();
    for (int b0 = 0; b0 < nti; b0 += 8)
        for (int J = 0; J < ntj; ++J)
            for (int I = b0; I < std::min(nti, b0 + 8); ++I)
                if (TR * I <= TC * J + TC - 1) out.push_back((unsigned)I | ((unsigned)J << 16));
}

long long split_wide_tiles(int ng) {
    const int nti = (ng + TR - 1) / TR, ntj = (ng + 127) / 128;
    long long n = 0;
    for (int I = 0; I < nti; ++I) n += ntj - I / 2;  // those with 64 I <= 128 J + 127
    return n;
}

int split_grid() { return device_cus() / 8 * 8; }

int launch_split_slices(const double2 *M, long long K, int ng, long long r0, int nst, unsigned char *S,
                        short *E, const double *w, long long wstride, int nvec, signed char *EA, int *EC, hipStream_t st) {
    const int gpad = split_gpad(ng), nch = (nst + NKS - 1) / NKS;
    hipLaunchKernelGGL(k_split_slice, dim3(gpad / 32, nch), dim3(SLICE_T), 0, st, M, K, ng, gpad, r0, nst, S, E, w,
                       wstride, nvec, EA, split_apad(ng), EC);
    BGW_HIP(hipGetLastError());
    return BGW_OK;
}

int launch_chi_split(const SplitQ *qs, int nq, long long nitems, hipStream_t st) {
    if (nitems <= 0) return BGW_OK;
    const long long g = std::max<long long>(8, std::min<long long>(nitems, split_grid()));
    hipLaunchKernelGGL(k_chi_split, dim3((unsigned)g), dim3(XT), 0, st, qs, nq, 0ll, nitems);
    BGW_HIP(hipGetLastError());
    return BGW_OK;
}

int launch_headwing(const double2 *M, long long K, int ng, int head, const double *w, long long wstride, int nvec,
                    int nsplit, double2 *hw, hipStream_t st) {
    const long long kper = (K + nsplit - 1) / nsplit;
    for (int v0 = 0; v0 < nvec; v0 += kHeadVec) {
        const int nv = std::min(kHeadVec, nvec - v0);
        hipLaunchKernelGGL(k_headwing, dim3((ng + 255) / 256, nsplit), dim3(256), 0, st, M, K, ng, head, w, wstride,
                           v0, nv, kper, hw, nvec);
    }
    BGW_HIP(hipGetLastError());
    return BGW_OK;
}

int launch_headwing_write(const double2 *hw, int nsplit, int nvec, int ng, int head, double pf, double2 *chi, int nout,
                          int two, int neg_im, int accumulate, hipStream_t st) {
    hipLaunchKernelGGL(k_headwing_write, dim3((ng + 255) / 256, nout), dim3(256), 0, st, hw, nsplit, nvec, ng, head,
                       pf, chi, two, neg_im, accumulate);
    BGW_HIP(hipGetLastError());
    return BGW_OK;
}

}  // namespace bgw
