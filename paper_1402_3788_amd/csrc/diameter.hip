// Algorithm 2 steps 1-2 (the two steps the paper's GPU regime, Algorithm 4,
// sends to the GPU): the centre of gravity C of the whole set, and the
// diameter of Eq. (3) -- the pair of objects with the largest distance.
//
// Centre of gravity: X read as a flat array of n*M floats by G workgroups of
// T threads, T a multiple of M, so that thread t always meets feature t mod M;
// each thread keeps one fp64 sum, each workgroup adds its threads' sums per
// feature in ascending thread order, and one workgroup adds the G rows in
// ascending order and rounds fp32(sum / n). Every addition's order depends
// only on the shape.
//
// Diameter, squared: D2 = max over pairs k < l of |x_k - x_l|^2, with the
// lexicographically smallest pair reaching it. The all-pairs distances are a
// Gram matrix (a dense contraction over the features), screened on the fp16
// matrix cores with one product per 32 features, then made exact:
//   norms   y_i = fl(x_i - C) (centring keeps the norms, and so the error
//           bound, small against D2), n_i = fl(|y_i|^2), and the largest n_i;
//           s = 2^e scales it into [2^12, 2^14): every operand below fits fp16;
//   prep    operand rows a_i = [-2 s y_i, h_i, 1, l_i, 1, 0 ...],
//           b_j = [s y_j, 1, h_j, 1, l_j, 0 ...] (P = 32 ceil((M+2)/32)
//           features) in fp16, rounded to nearest, with h_i = fp16(s^2 n_i) and
//           l_i = fp16(s^2 n_i - h_i), so that a_i . b_j = s^2 (n_i + n_j - 2
//           y_i.y_j) ~ s^2 |x_i - x_j|^2 with no epilogue arithmetic; l is left
//           out where M + 4 features do not fit P; rows are stored in the
//           matrix instruction's lane order;
//   pass 1  every pair block is one v_mfma_f32_16x16x32_f16 per 32 features,
//           exact products summed in fp32; the maximum approximate value d~*
//           over all pairs is kept (integer atomic max of an order-preserving
//           key: order-free), and each work item's own maximum goes to its
//           result slot;
//   pass 2  items whose maximum is below the threshold d~* - 2B write an
//           empty result at once; the others form the same products again, and
//           where a wave's 64 x 32 pairs hold one with d~ >= d~* - 2B, it adds
//           the products with the operands' low parts, which gives values
//           d~2 with a bound B2 some 300 times smaller. Of those the pairs
//           k < l with d~2 >= (the largest d~2 found so far, by any wave) - 2
//           B2 are re-evaluated in fp64 in the fixed operation order
//           e = x_j - c_j, d = d + e*e (features ascending, each operation
//           rounded) and the lexicographic best (largest d, then lowest k,
//           then lowest l) is kept.
// B bounds |d~ - s^2 d| for every pair: with u = 2^-24, gamma_m = m u / (1 - m u)
// for this code's own round-to-nearest fp32 arithmetic and
// phi_m = 2 m u / (1 - 2 m u) for the matrix core's additions (assumed only
// faithful: each within 2^-23 relative, in any order or direction),
//   |d~ - s^2 d| <= E s^2 (|y_k|^2 + |y_l|^2) + A,
//   E = 4.01 u (centring) + 2.01 * 2^-11 (fp16 y: each factor within 2^-11, and
//       2 |y_k . y_l| <= |y_k|^2 + |y_l|^2) + 1.01 * 2^-22 (fp16 h + l; 1.01 *
//       2^-11 without l) + 1.01 gamma_M (the fp32 norms) + 2.02 phi_{P+2} (the
//       sums),
//   A = 2^-14 (2 sqrt(M) (|s y_k| + |s y_l|) + M 2^-13 + 4) for operand values
//       below the normal range of fp16 (2^-14), flushed or not; with
//       |s y| <= 2^7, A <= 0.27,
// so B = 1.25 (2.02 E s^2 max_i n_i + A) covers every pair (1.25: margin). The
// true pair has d~ >= s^2 D2 - B >= d~* - 2B, so it is always re-evaluated, and
// the result is exact whatever the fp16 products round to. The band 2B is 0.5 %
// of the largest norm: on random data a handful of pairs lie in it. (The three
// bf16 split products that this screening took before had a band of 0.06 % and
// three times the matrix work: pass 1 at n = 500,003, M = 25 took 15.5 ms,
// now 5.7.)
//
// The second screening. With v = s y, hi = fp16(v) (0 below 2^-14) and lo =
// fp16(2^11 (v - hi)), written by the prep launch, the wave adds
//   d~2 = d~ + 2^-11 sum(a_lo b_hi + a_hi b_lo),
// the norms' remainders 2^11 (s^2 n - h - l) standing at feature M of a_lo and M
// + 1 of b_lo against the ones of b_hi and a_hi. The true maximum is at least
// any d~2 - B2 and a pair's d at most its d~2 + B2, so a pair left out is
// strictly smaller than the maximum. B2 = 1.25 (2.02 E2 s^2 max_i n_i + A2),
//   E2 = 4.01 u (centring) + 3.01 * 2^-22 (the dropped v_lo w_lo and lo's own
//       rounding) + 1.01 * 2^-22 (the norms' remainders) + 1.01 gamma_M + 2.02
//       phi_{P+2} + 2.02 u (the last addition) + 3.1 * 2^-11 phi_{2P+2} (the
//       low sums, whose terms add up to at most 3.1 * 2^11 * 2^-11 (n_k + n_l)),
//   A2 = 2^-10: lo below the normal range (2^-13), low times low where hi is 0
//       (2^-13), h and l below it (2^-12), with 2^-11 more for the rest.
// The pairs that remain wait in LDS until 64 of them are taken together, one per
// lane. Without either, points on a circle (n = 20,000, M = 2) took 5,618 us and
// two tight groups (M = 25) 1,069, and 3,305 and 685 with the bf16 products; now
// 1,156 and 453 (n = 100,003: 9,425 and 1,290 with the bf16 products, now 3,525
// and 642).
//
// Work: pass items are (row block of 512 objects, column chunk of 16384);
// items wholly below the diagonal return at once, and within the diagonal
// chunk the column steps start at the row block. Each of 8 waves holds the A
// operands of 64 rows in registers; the workgroup stages 64 columns of B at a
// time in LDS (row stride padded by 16 bytes so the 16-byte reads of a
// 16-object column block spread over the banks), and each wave forms 4 x 4
// blocks of 16 x 16 pairs per step. The next step's operands are loaded into
// registers while the current step is computed, and written to the other of
// two LDS buffers after it: one barrier per step.
#include "lloyd_device.h"
#include "diameter.h"

#include <cfloat>
#include <climits>

namespace lloyd {

namespace {

typedef float f4v __attribute__((ext_vector_type(4)));
typedef _Float16 h8v __attribute__((ext_vector_type(8)));

__device__ inline h8v as_h8(const uint4 &u)
{
    return __builtin_bit_cast(h8v, u);
}

constexpr int kDiamWaves = 8;
constexpr int kDiamThreads = kDiamWaves * kWave;
constexpr int kRowBlock = kDiamWaves * 64;       // objects per item's row block
constexpr int kChunkSteps = 256;                 // 64-column steps per item
constexpr int kChunk = kChunkSteps * 64;         // columns per item
constexpr int kCentroidGroups = 256;

// Order-preserving key of an fp32 value (larger value, larger key).
__device__ inline uint32_t float_key(float v)
{
    const uint32_t b = __float_as_uint(v);
    return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}

__device__ inline float key_float(uint32_t k)
{
    return __uint_as_float((k & 0x80000000u) ? (k & 0x7FFFFFFFu) : ~k);
}

// ---------------------------------------------------------------------------
// Centre of gravity (Algorithm 2 step 2).

__global__ void __launch_bounds__(1024)
centroid_partial_kernel(const float *__restrict__ X, int64_t total, int M,
                        double *__restrict__ part)
{
    extern __shared__ double csum[];                  // [blockDim.x]
    const int T = blockDim.x;                         // a multiple of M
    const int64_t S = (int64_t)gridDim.x * T;
    double s = 0.0;
    // eight loads in flight; past the end the last element's value is not added
    constexpr int kAhead = 8;
    for (int64_t e = (int64_t)blockIdx.x * T + threadIdx.x; e < total; e += kAhead * S) {
        float v[kAhead];
#pragma unroll
        for (int u = 0; u < kAhead; ++u) v[u] = X[e + u * S < total ? e + u * S : total - 1];
#pragma unroll
        for (int u = 0; u < kAhead; ++u)
            if (e + u * S < total) s = s + (double)v[u];
    }
    csum[threadIdx.x] = s;
    __syncthreads();
    if (threadIdx.x < M) {
        double r = 0.0;
        for (int t = threadIdx.x; t < T; t += M) r = r + csum[t];
        part[(int64_t)blockIdx.x * M + threadIdx.x] = r;
    }
}

// Reads the G partial rows; writes the centroid (fp32) and resets the
// counters of the diameter passes. Row lane r of 16 adds rows r, r + 16, ... of
// its feature (every load before the first addition), then the 16 sums are
// added in ascending order. (One thread per feature adding the rows one by one
// took 60 us.)
constexpr int kFinalLanes = 16;

__global__ void __launch_bounds__(kFinalLanes * kWave)
centroid_final_kernel(const double *__restrict__ part, int G, int M, int64_t n,
                      float *__restrict__ centroid_ws, float *__restrict__ centroid_out,
                      uint32_t *__restrict__ counters)
{
    __shared__ double sums[kFinalLanes][kWave];
    const int r = threadIdx.x / kWave, j = threadIdx.x % kWave;
    double v[kCentroidGroups / kFinalLanes];
#pragma unroll
    for (int u = 0; u < kCentroidGroups / kFinalLanes; ++u) {
        const int g = r + kFinalLanes * u;
        v[u] = (g < G && j < M) ? part[(int64_t)g * M + j] : 0.0;
    }
    double s = 0.0;
#pragma unroll
    for (int u = 0; u < kCentroidGroups / kFinalLanes; ++u) s = s + v[u];
    sums[r][j] = s;
    __syncthreads();
    if (r == 0 && j < M) {
        double t = 0.0;
#pragma unroll
        for (int u = 0; u < kFinalLanes; ++u) t = t + sums[u][j];
        const float c = (float)(t / (double)n);
        if (centroid_ws) centroid_ws[j] = c;
        if (centroid_out) centroid_out[j] = c;
    }
    // max norm, key of d~*, non-finite coordinate seen, key of the largest d~2,
    // pairs taken in fp64
    if (counters && threadIdx.x < 5) counters[threadIdx.x] = 0;
}

// ---------------------------------------------------------------------------
// Norms and fp16 operands.

constexpr int kNormThreads = 1024;

// n_i = |x_i - C|^2 in fp32, their maximum and the non-finite flag: persistent
// workgroups, one atomic each.
__global__ void __launch_bounds__(kNormThreads)
diam_norm_kernel(const float *__restrict__ X, int64_t n, int M, const float *__restrict__ C,
                 float *__restrict__ norms, uint32_t *__restrict__ counters)
{
    __shared__ float smax[kNormThreads / kWave];
    float m = 0.f;
    bool finite = true;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x) {
        const float *x = X + i * M;
        float nrm = 0.f;
#pragma unroll 8
        for (int f = 0; f < M; ++f) {
            const float v = x[f], y = v - C[f];
            finite = finite && fabsf(v) < INFINITY;
            nrm = nrm + y * y;
        }
        norms[i] = nrm;
        m = fmaxf(m, nrm);
    }
    // a NaN or an infinite coordinate leaves the diameter undefined: the
    // passes return at once and the result is NaN with the pair (-1, -1)
    if (__ballot(!finite) != 0ull && threadIdx.x % kWave == 0) atomicOr(&counters[2], 1u);
#pragma unroll
    for (int off = kWave / 2; off > 0; off >>= 1) m = fmaxf(m, __shfl_xor(m, off));
    if (threadIdx.x % kWave == 0) smax[threadIdx.x / kWave] = m;
    __syncthreads();
    if (threadIdx.x == 0) {
        float r = smax[0];
        for (int w = 1; w < (int)(blockDim.x / kWave); ++w) r = fmaxf(r, smax[w]);
        atomicMax(&counters[0], __float_as_uint(r));          // r >= 0: bits order like values
    }
}

// Exponent e of the operands' scale s = 2^e: s^2 max n in [2^12, 2^14) (0 for
// an all-zero or an overflowed norm; the latter re-evaluates every pair).
__device__ inline int diam_scale_exp(const uint32_t *counters)
{
    const float maxn = __uint_as_float(counters[0]);
    if (!(maxn > 0.f) || !(maxn < INFINITY)) return 0;
    const int E = ilogbf(maxn);
    const int d = 13 - E;
    return d >= 0 ? d / 2 : -((1 - d) / 2);       // floor(d / 2)
}

// High part of a scaled coordinate: its fp16 value, 0 below the normal range.
__device__ inline float diam_high(float v)
{
    return fabsf(v) < 6.103515625e-5f ? 0.f : (float)(_Float16)v;
}

// Low parts are kept times 2^11, in the range of their high parts.
constexpr int kLowExp = 11;

// One thread per 16-byte group (8 features) of an operand row.
__global__ void __launch_bounds__(256)
diam_prep_kernel(const float *__restrict__ X, int64_t n, int64_t groups, int G4, int M,
                 const float *__restrict__ C, const float *__restrict__ norms,
                 const uint32_t *__restrict__ counters, uint4 *__restrict__ ah,
                 uint4 *__restrict__ bh, uint4 *__restrict__ low_ops)
{
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= groups) return;
    const int64_t i = t / G4;
    const int g = (int)(t % G4);
    const bool real = i < n;
    const bool low = M + 4 <= 8 * G4;             // room for the norms' low parts
    const int e = diam_scale_exp(counters);
    h8v a, b, lo;
    float nh = 0.f, nl = 0.f, rest = 0.f;
    if (real) {
        const float ns = ldexpf(norms[i], 2 * e);
        nh = (float)(_Float16)ns;
        nl = (float)(_Float16)(ns - nh);
        rest = ldexpf((ns - nh) - (low ? nl : 0.f), kLowExp);
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) {
        const int f = 8 * g + u;
        float av = 0.f, bv = 0.f, lv = 0.f;
        if (real && f < M) {
            const float v = ldexpf(X[i * M + f] - C[f], e), y = diam_high(v);
            av = -2.0f * y;
            bv = y;
            lv = ldexpf(v - y, kLowExp);
        } else if (real) {
            if (f == M) { av = nh; bv = 1.0f; lv = rest; }
            if (f == M + 1) { av = 1.0f; bv = nh; lv = rest; }
            if (low && f == M + 2) { av = nl; bv = 1.0f; }
            if (low && f == M + 3) { av = 1.0f; bv = nl; }
        }
        a[u] = (_Float16)av;
        b[u] = (_Float16)bv;
        lo[u] = (_Float16)lv;
    }
    ah[t] = __builtin_bit_cast(uint4, a);
    bh[t] = __builtin_bit_cast(uint4, b);
    low_ops[t] = __builtin_bit_cast(uint4, lo);
}

// ---------------------------------------------------------------------------
// The two all-pairs passes.

__device__ inline bool diam_better(double d, int k, int l, double bd, int bk, int bl_)
{
    return d > bd || (d == bd && (k < bk || (k == bk && l < bl_)));
}

__device__ inline float round_down(double v)
{
    float t = (float)v;
    if ((double)t > v) t = nextafterf(t, -INFINITY);
    return t;
}

// Threshold of pass 2: d~* - 2B, rounded down to fp32; minus infinity (every
// pair re-evaluated in fp64) when the largest norm is so large that an fp32
// norm may overflow (a pair value is at most 4 max n_i), or so small that the
// squares in it underflow by more than the margin covers: M of them lose at
// most M 2^-150 = 4.5e-44 together, 0.08 u of 1e-35. band2: 2 B2.
template <int KS>
__device__ inline float diam_threshold(const uint32_t *counters, int M, double &band2)
{
    constexpr int P = 32 * KS;
    const double u = 5.9604644775390625e-8;           // 2^-24
    auto gamma = [&](int m) { return m * u / (1.0 - m * u); };
    auto phi = [&](int m) { return 2.0 * m * u / (1.0 - 2.0 * m * u); };
    const double norm_err = M + 4 <= P ? 1.01 / 4194304.0 : 1.01 / 2048.0;
    const double sums = 4.01 * u + 1.01 * gamma(M) + 2.02 * phi(P + 2);
    const double E = sums + 2.01 / 2048.0 + norm_err;
    const double E2 = sums + 4.02 / 4194304.0 + 2.02 * u + 3.1 / 2048.0 * phi(2 * P + 2);
    const double maxn = (double)__uint_as_float(counters[0]);
    if (!(4.0 * maxn < (double)FLT_MAX) || maxn < 1e-35) return -INFINITY;
    const double scaled = 2.02 * ldexp(maxn, 2 * diam_scale_exp(counters));
    const double B = 1.25 * (E * scaled + 0.27);
    band2 = 2.0 * 1.25 * (E2 * scaled + 1.0 / 1024.0);
    return round_down((double)key_float(counters[1]) - 2.0 * B);
}

// fp64 squared distance of objects i and j in the fixed operation order (the
// rare exact re-evaluation of pass 2, kept out of line so that the matrix
// loop's registers are not sized for it).
__device__ __attribute__((noinline)) double diam_exact_d2(const float *__restrict__ X, int M,
                                                          int64_t i, int64_t j)
{
    const float *xi = X + i * M, *xj = X + j * M;
    double d = 0.0;
    for (int f = 0; f < M; ++f) {
        const double e = (double)xi[f] - (double)xj[f];
        const double sq = e * e;
        d = d + sq;
    }
    return d;
}

// Orders this wave's own LDS accesses (what its lanes wrote, its lanes read).
__device__ inline void wave_lds_fence()
{
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

template <int KS, bool kExact>
__device__ __forceinline__ void
diam_pass_body(const uint4 *__restrict__ ah, const uint4 *__restrict__ bh, int64_t n,
               int64_t nsteps_total, const float *__restrict__ X, int M,
               const uint4 *__restrict__ low_ops, uint32_t *__restrict__ counters, DiamBest *__restrict__ slots)
{
    constexpr int G4 = 4 * KS;                        // 16-byte groups per operand row
    constexpr int kLdsRow = G4 + 1;                   // uint4 per LDS row (16 bytes padding)
    constexpr int kQuads = 64 * G4;                   // 16-byte groups per step and array
    constexpr int kPer = (kQuads + kDiamThreads - 1) / kDiamThreads;   // groups a thread copies
    // two buffers: the step computed and the step being staged
    __shared__ uint4 sb[2][64 * kLdsRow];
    __shared__ int wmax[kDiamWaves];
    __shared__ DiamBest wbest[kDiamWaves];

    if (counters[2] != 0u) return;                    // non-finite input (uniform)
    const int lane = threadIdx.x % kWave, w = threadIdx.x / kWave;
    const int64_t I0 = (int64_t)blockIdx.x * kRowBlock;
    const int64_t J0 = (int64_t)blockIdx.y * kChunk;
    const int64_t slot = (int64_t)blockIdx.y * gridDim.x + blockIdx.x;
    const int64_t s_lo = (J0 > I0 ? J0 : I0) / 64;    // first 64-column step
    int64_t s_hi = (J0 + kChunk) / 64;
    if (s_hi > nsteps_total) s_hi = nsteps_total;
    if (s_lo >= s_hi) {                               // wholly below the diagonal or past n
        if (threadIdx.x == 0) slots[slot] = DiamBest{kExact ? -1.0 : -INFINITY, INT_MAX, INT_MAX};
        return;
    }

    float thr = 0.f;
    double band2 = 0.0;
    if constexpr (kExact) {
        // pass 1 left this item's largest value in its slot: an item with no
        // value at the threshold has no candidate pair (a NaN, possible only
        // when thr is minus infinity, is kept)
        thr = diam_threshold<KS>(counters, M, band2);
        if (slots[slot].d < (double)thr) {
            __syncthreads();                          // every thread has read the slot
            if (threadIdx.x == 0) slots[slot] = DiamBest{-1.0, INT_MAX, INT_MAX};
            return;
        }
    }

    // A operands of this wave's 64 rows: 4 row blocks x KS steps of 32 features
    uint4 a_op[4][KS];
    const int64_t r0 = I0 + 64 * w;
#pragma unroll
    for (int rb = 0; rb < 4; ++rb)
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
            a_op[rb][ks] = ah[(r0 + 16 * rb + lane % 16) * G4 + ks * 4 + lane / 16];

    // staging: thread t copies groups t, t + 512, ... (past the last: the last)
    uint4 pf[kPer];
    auto group_of = [&](int u) {
        const int q = threadIdx.x + kDiamThreads * u;
        return q < kQuads ? q : kQuads - 1;
    };
    auto fetch = [&](int64_t s) {
#pragma unroll
        for (int u = 0; u < kPer; ++u) pf[u] = bh[s * kQuads + group_of(u)];
    };
    auto stage = [&](int buf) {
#pragma unroll
        for (int u = 0; u < kPer; ++u) {
            const int q = group_of(u);
            sb[buf][(q / G4) * kLdsRow + q % G4] = pf[u];
        }
    };

    int vmax = 0;
    double bd = -1.0;
    int bk = INT_MAX, bl_ = INT_MAX;
    uint32_t taken = 0;                               // pairs in fp64 (whole wave)
    // pairs that wait for fp64, 64 at a time: row - r0 and column - J0 of each
    __shared__ uint32_t waiting[kExact ? kDiamWaves : 1][kExact ? 2 * kWave : 1];
    int nwait = 0;
    auto take = [&](int count) {
        if (lane < count) {
            const uint32_t q = waiting[w][lane];
            const int64_t i = r0 + (q & 63u), j = J0 + (q >> 6);
            const double d = diam_exact_d2(X, M, i, j);
            if (diam_better(d, (int)i, (int)j, bd, bk, bl_)) {
                bd = d;
                bk = (int)i;
                bl_ = (int)j;
            }
        }
        taken += count;
    };

    fetch(s_lo);
    stage(0);
    __syncthreads();
    for (int64_t s = s_lo; s < s_hi; ++s) {
        const int buf = (int)((s - s_lo) & 1);
        const bool more = s + 1 < s_hi;
        if (more) fetch(s + 1);                       // in flight during this step
        const uint4 *lh = sb[buf];

        // the step's 64 columns in two halves of 32 (2 column blocks)
#pragma unroll
        for (int half = 0; half < 2; ++half) {
            f4v acc[4][2];
#pragma unroll
            for (int rb = 0; rb < 4; ++rb)
#pragma unroll
                for (int cc = 0; cc < 2; ++cc) acc[rb][cc] = f4v{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                uint4 b[2];
#pragma unroll
                for (int cc = 0; cc < 2; ++cc)
                    b[cc] = lh[(16 * (2 * half + cc) + lane % 16) * kLdsRow + ks * 4 + lane / 16];
#pragma unroll
                for (int rb = 0; rb < 4; ++rb)
#pragma unroll
                    for (int cc = 0; cc < 2; ++cc)
                        acc[rb][cc] = __builtin_amdgcn_mfma_f32_16x16x32_f16(
                            as_h8(a_op[rb][ks]), as_h8(b[cc]), acc[rb][cc], 0, 0, 0);
            }

            // the largest value of the half in this lane, or 0: the order of
            // the bits of non-negative floats as integers (a positive NaN
            // above all), negative values (error around 0) below 0. One
            // three-way maximum per two values; the floating-point form made
            // the compiler quiet every operand first (9.5 ms against 5.7 in
            // pass 1). Padding rows and columns give exactly 0, and pairs i >=
            // j repeat pairs i < j.
            int smax = 0;
#pragma unroll
            for (int rb = 0; rb < 4; ++rb)
#pragma unroll
                for (int cc = 0; cc < 2; ++cc) {
                    auto bits = [&](int r) { return __float_as_int(acc[rb][cc][r]); };
                    smax = max(max(smax, bits(0)), bits(1));
                    smax = max(max(smax, bits(2)), bits(3));
                }
            if constexpr (!kExact) {
                vmax = max(vmax, smax);
            } else if (__builtin_amdgcn_ballot_w64(!(__int_as_float(smax) < thr)) != 0) {
                // rare: some pair of this wave's half step reaches the threshold
                const int64_t c0 = s * 64 + 32 * half;
                float thr2 = thr;
                if (thr > -INFINITY) {
                    // rows of the low operands: object by object, the norm's
                    // rest at both M and M + 1; as a's row times -2, 1 and 0,
                    // as b's times 1, 0 and 1
                    f4v lo[4][2];
#pragma unroll
                    for (int rb = 0; rb < 4; ++rb)
#pragma unroll
                        for (int cc = 0; cc < 2; ++cc) lo[rb][cc] = f4v{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int ks = 0; ks < KS; ++ks) {
                        const int g = ks * 4 + lane / 16;
                        uint4 ra[4], rc[2];
#pragma unroll
                        for (int rb = 0; rb < 4; ++rb)
                            ra[rb] = low_ops[(r0 + 16 * rb + lane % 16) * G4 + g];
#pragma unroll
                        for (int cc = 0; cc < 2; ++cc)
                            rc[cc] = low_ops[(c0 + 16 * cc + lane % 16) * G4 + g];
                        h8v ma, mb;
#pragma unroll
                        for (int u = 0; u < 8; ++u) {
                            const int f = 8 * g + u;
                            ma[u] = (_Float16)(f < M ? -2.f : f == M ? 1.f : 0.f);
                            mb[u] = (_Float16)(f == M ? 0.f : 1.f);
                        }
                        h8v bhi[2], blo[2];
#pragma unroll
                        for (int cc = 0; cc < 2; ++cc) {
                            bhi[cc] = as_h8(lh[(32 * half + 16 * cc + lane % 16) * kLdsRow + g]);
                            blo[cc] = as_h8(rc[cc]) * mb;
                        }
#pragma unroll
                        for (int rb = 0; rb < 4; ++rb) {
                            const h8v alo = as_h8(ra[rb]) * ma;
#pragma unroll
                            for (int cc = 0; cc < 2; ++cc) {
                                lo[rb][cc] = __builtin_amdgcn_mfma_f32_16x16x32_f16(
                                    alo, bhi[cc], lo[rb][cc], 0, 0, 0);
                                lo[rb][cc] = __builtin_amdgcn_mfma_f32_16x16x32_f16(
                                    as_h8(a_op[rb][ks]), blo[cc], lo[rb][cc], 0, 0, 0);
                            }
                        }
                    }
                    // d~2 in place of d~, and its largest value (padding gives 0)
                    float m = 0.f;
#pragma unroll
                    for (int rb = 0; rb < 4; ++rb)
#pragma unroll
                        for (int cc = 0; cc < 2; ++cc)
#pragma unroll
                            for (int r = 0; r < 4; ++r) {
                                acc[rb][cc][r] = acc[rb][cc][r] + lo[rb][cc][r] * (1.0f / 2048.0f);
                                m = fmaxf(m, acc[rb][cc][r]);
                            }
#pragma unroll
                    for (int off = kWave / 2; off > 0; off >>= 1) m = fmaxf(m, __shfl_xor(m, off));
                    const uint32_t key = float_key(m);
                    uint32_t best = __hip_atomic_load(&counters[3], __ATOMIC_RELAXED,
                                                      __HIP_MEMORY_SCOPE_AGENT);
                    if (key > best) {
                        if (lane == 0) atomicMax(&counters[3], key);
                        best = key;
                    }
                    thr2 = round_down((double)key_float(best) - band2);
                }
                // this lane's values at the threshold, one bit each (a NaN,
                // possible only when thr is minus infinity, is taken too)
                uint32_t mask = 0;
#pragma unroll
                for (int rb = 0; rb < 4; ++rb)
#pragma unroll
                    for (int cc = 0; cc < 2; ++cc)
#pragma unroll
                        for (int r = 0; r < 4; ++r)
                            if (!(acc[rb][cc][r] < thr2)) mask |= 1u << (8 * rb + 4 * cc + r);
                while (__builtin_amdgcn_ballot_w64(mask != 0u) != 0) {
                    const int b = mask != 0u ? __ffs(mask) - 1 : 0;
                    const int row = 16 * (b >> 3) + 4 * (lane / 16) + (b & 3);
                    const int64_t j = c0 + 16 * ((b >> 2) & 1) + lane % 16;
                    const bool close = mask != 0u && r0 + row < j && j < n;
                    mask &= mask - 1u;
                    const uint64_t vote = __builtin_amdgcn_ballot_w64(close);
                    if (close)
                        waiting[w][nwait + __popcll(vote & ((1ull << lane) - 1ull))] =
                            (uint32_t)row | (uint32_t)(j - J0) << 6;
                    nwait += __popcll(vote);
                    wave_lds_fence();
                    if (nwait >= kWave) {
                        take(kWave);
                        nwait -= kWave;
                        const uint32_t left = waiting[w][kWave + lane];
                        wave_lds_fence();
                        if (lane < nwait) waiting[w][lane] = left;
                        wave_lds_fence();
                    }
                }
            }
        }

        if (more) stage(buf ^ 1);                     // the other buffer: nobody reads it now
        __syncthreads();
    }

    if constexpr (!kExact) {
#pragma unroll
        for (int off = kWave / 2; off > 0; off >>= 1) vmax = max(vmax, __shfl_xor(vmax, off));
        if (lane == 0) wmax[w] = vmax;
        __syncthreads();
        if (threadIdx.x == 0) {
            int m = wmax[0];
            for (int k = 1; k < kDiamWaves; ++k) m = max(m, wmax[k]);
            const float v = __int_as_float(m);
            atomicMax(&counters[1], float_key(v));
            slots[slot] = DiamBest{(double)v, INT_MAX, INT_MAX};   // read by pass 2
        }
    } else {
        take(nwait);
#pragma unroll
        for (int off = kWave / 2; off > 0; off >>= 1) {
            const double d2 = __shfl_xor(bd, off);
            const int k2 = __shfl_xor(bk, off), l2 = __shfl_xor(bl_, off);
            if (diam_better(d2, k2, l2, bd, bk, bl_)) {
                bd = d2;
                bk = k2;
                bl_ = l2;
            }
        }
        if (lane == 0) {
            wbest[w] = DiamBest{bd, bk, bl_};
            if (taken != 0) atomicAdd(&counters[4], taken);
        }
        __syncthreads();
        if (threadIdx.x == 0) {
            DiamBest b = wbest[0];
            for (int k = 1; k < kDiamWaves; ++k)
                if (diam_better(wbest[k].d, wbest[k].k, wbest[k].l, b.d, b.k, b.l)) b = wbest[k];
            slots[slot] = b;
        }
    }
}

template <int KS, bool kExact>
__global__ void __launch_bounds__(kDiamThreads)
diam_pass_kernel(const uint4 *__restrict__ ah, const uint4 *__restrict__ bh, int64_t n,
                 int64_t nsteps_total, const float *__restrict__ X, int M,
                 const uint4 *__restrict__ low_ops, uint32_t *__restrict__ counters,
                 DiamBest *__restrict__ slots)
{
    diam_pass_body<KS, kExact>(ah, bh, n, nsteps_total, X, M, low_ops, counters, slots);
}

// The lexicographic best of all item slots. With n = 1 there is no pair:
// (0, 0, 0); with a non-finite coordinate in X: (NaN, -1, -1).
__global__ void __launch_bounds__(1024)
diam_final_kernel(const DiamBest *__restrict__ slots, int64_t nslots, int64_t n,
                  const uint32_t *__restrict__ counters, double *__restrict__ d2_out,
                  int32_t *__restrict__ pair_out)
{
    if (counters[2] != 0u) {
        if (threadIdx.x == 0) {
            *d2_out = __builtin_nan("");
            pair_out[0] = -1;
            pair_out[1] = -1;
        }
        return;
    }
    __shared__ DiamBest wb[1024 / kWave];
    double bd = -1.0;
    int bk = INT_MAX, bl_ = INT_MAX;
    for (int64_t s = threadIdx.x; s < nslots; s += blockDim.x) {
        const DiamBest b = slots[s];
        if (diam_better(b.d, b.k, b.l, bd, bk, bl_)) {
            bd = b.d;
            bk = b.k;
            bl_ = b.l;
        }
    }
#pragma unroll
    for (int off = kWave / 2; off > 0; off >>= 1) {
        const double d2 = __shfl_xor(bd, off);
        const int k2 = __shfl_xor(bk, off), l2 = __shfl_xor(bl_, off);
        if (diam_better(d2, k2, l2, bd, bk, bl_)) {
            bd = d2;
            bk = k2;
            bl_ = l2;
        }
    }
    const int lane = threadIdx.x % kWave, w = threadIdx.x / kWave;
    if (lane == 0) wb[w] = DiamBest{bd, bk, bl_};
    __syncthreads();
    if (threadIdx.x == 0) {
        DiamBest b = wb[0];
        for (int k = 1; k < (int)(blockDim.x / kWave); ++k)
            if (diam_better(wb[k].d, wb[k].k, wb[k].l, b.d, b.k, b.l)) b = wb[k];
        if (n < 2 || b.d < 0.0) b = DiamBest{0.0, 0, n > 1 ? 1 : 0};
        *d2_out = b.d;
        pair_out[0] = b.k;
        pair_out[1] = b.l;
    }
}

template <int KS>
hipError_t diam_launch_ks(const DiameterArgs &a, const DiameterPlan &pl, hipStream_t s)
{
    const int64_t want = (a.n + kNormThreads - 1) / kNormThreads;
    const dim3 gnorm((unsigned)(want < kCUs ? want : kCUs));
    hipLaunchKernelGGL(diam_norm_kernel, gnorm, dim3(kNormThreads), 0, s, a.X, a.n, a.M,
                       a.centroid_ws, a.norms, a.counters);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const int64_t groups = pl.npad * 4 * KS;
    hipLaunchKernelGGL(diam_prep_kernel, dim3((unsigned)((groups + 255) / 256)), dim3(256), 0, s,
                       a.X, a.n, groups, 4 * KS, a.M, a.centroid_ws, a.norms, a.counters, a.ah,
                       a.bh, a.low);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    const dim3 grid((unsigned)pl.row_blocks, (unsigned)pl.chunks);
    const int64_t nsteps = pl.npad / 64;
    auto pass1 = diam_pass_kernel<KS, false>;
    auto pass2 = diam_pass_kernel<KS, true>;
    hipLaunchKernelGGL(pass1, grid, dim3(kDiamThreads), 0, s, a.ah, a.bh, a.n,
                       nsteps, a.X, a.M, a.low, a.counters, a.slots);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    hipLaunchKernelGGL(pass2, grid, dim3(kDiamThreads), 0, s, a.ah, a.bh, a.n,
                       nsteps, a.X, a.M, a.low, a.counters, a.slots);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    hipLaunchKernelGGL(diam_final_kernel, dim3(1), dim3(1024), 0, s, a.slots,
                       (int64_t)pl.row_blocks * pl.chunks, a.n, a.counters, a.d2, a.pair);
    return hipGetLastError();
}

}  // namespace

CentroidPlan plan_centroid(int64_t n, int M)
{
    CentroidPlan pl{};
    pl.threads = (1024 / M) * M;
    const int64_t total = n * M;
    int64_t g = (total + pl.threads - 1) / pl.threads;
    pl.groups = (int)(g < kCentroidGroups ? g : kCentroidGroups);
    return pl;
}

hipError_t launch_centroid(const float *X, int64_t n, int M, double *part, float *centroid_ws,
                           float *centroid_out, uint32_t *counters, const CentroidPlan &pl,
                           hipStream_t s)
{
    hipLaunchKernelGGL(centroid_partial_kernel, dim3(pl.groups), dim3(pl.threads),
                       (size_t)pl.threads * sizeof(double), s, X, n * M, M, part);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(centroid_final_kernel, dim3(1), dim3(kFinalLanes * kWave), 0, s, part, pl.groups, M, n,
                       centroid_ws, centroid_out, counters);
    return hipGetLastError();
}

DiameterPlan plan_diameter(int64_t n, int M)
{
    DiameterPlan pl{};
    pl.ks = (M + 2 + 31) / 32;
    pl.npad = (n + kChunk - 1) / kChunk * kChunk;
    pl.row_blocks = (n + kRowBlock - 1) / kRowBlock;
    pl.chunks = pl.npad / kChunk;
    return pl;
}

hipError_t launch_diameter(const DiameterArgs &a, const DiameterPlan &pl, hipStream_t s)
{
    switch (pl.ks) {
    case 1: return diam_launch_ks<1>(a, pl, s);
    case 2: return diam_launch_ks<2>(a, pl, s);
    case 3: return diam_launch_ks<3>(a, pl, s);
    }
    return hipErrorInvalidValue;
}

}  // namespace lloyd
