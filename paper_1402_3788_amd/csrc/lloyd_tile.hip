// Fused assign + accumulate with the distances on the matrix cores, 64-object
// tiles against 16-centre blocks (any K).
//
// Expanded form of the squared distance of Eq. (2): for object x and centre c,
//     |x - c|^2 = |x|^2 + score,   score = |c|^2 - 2 x.c,
// and |x|^2 is the same for every centre, so the nearest centre is the one with
// the smallest score. For 16 centres and 16 objects the scores are one matrix
// product D[centre][object] = |c|^2 + sum_j (-2 c_j) x_j with A = -2C (built
// once per workgroup in LDS, in the lane order the instruction wants), B = X^T
// (read from the LDS tile) and the accumulator seeded with |c|^2, in up to
// three stages:
//   pass 1 (every tile): split precision on the bf16 matrix cores, operands
//     split into bf16 hi and lo parts rounded to nearest. 32 features take
//     three v_mfma_f32_16x16x32_bf16 per block (lo.hi, hi.lo, hi.hi); a last
//     chunk of at most 16 features puts hi and lo of A side by side in one
//     operand and takes two (against B's lo, then hi), one of at most 8
//     features puts both parts of both sides in one product. Each score is
//     within E (3|c|^2 + |x|^2) of the exact one (E below, assuming only that
//     the matrix core rounds each addition faithfully); the scores are scanned
//     as packed (score, index) keys, and a label is accepted when the two best
//     keys differ by more than twice that bound plus the keys' truncation
//     (with |c|^2 bounded by the largest centre norm and margins);
//   the other objects (close calls) stay out of the sums; the wave notes them,
//   each with its limit (best key + threshold: no centre whose score is above
//   it can be the nearest), in a list in LDS, and the workgroup decides them
//   after its last tile, in columns of 16: their scores are formed again, the
//   centres within the limit become candidates, and the fp64 distances to
//   those (the fixed operation order, lowest index on ties) decide. Up to four
//   candidates of a lane are kept as they are found; a wave with objects that
//   have more, up to kManyCand in a lane, forms their scores once more and
//   takes the distances as it finds them. Objects with more still, and all
//   objects of a wave whose list overflowed (they are then found again by the
//   negative mark left in their labels), take the direct fp32 form over all
//   centres, and fp64 over the centres within 4 gamma_{M+2} of its best.
//
// Why the close calls wait: on data whose clusters overlap a tenth of the
// objects is close, so almost every 64-object tile holds one. Recomputing such
// a tile with fp32 products and fp64 distances to every centre took 470 of
// the 620 us of a launch (n = 1e6, M = 37, K = 100); gathered, they cost a
// column each, and the streaming loop keeps no code or registers for them.
//
// Layout of the 16x16 products (64 lanes): D[i][j] is in lane j + 16(i/4),
// register i%4; A[i][k] in lane i + 16k (16x16x4) or lane i + 16(k/8), element
// k%8 (16x16x32), and B[k][j] likewise with j. So every lane holds the scores
// of 4 centres for the four objects it sees in the tile's four 16-object
// columns, and the four lanes that hold an object's centre rows exchange their
// results with row swaps (v_permlane16_swap, v_permlane32_swap).
//
// Each wavefront streams 64-object tiles (in wave-major rounds of the grid):
// the next tile's loads are in flight in registers while the current tile
// is staged in the wave's LDS slot; the round with the ragged last tile (n not
// a multiple of 64) is handled after the loop.
//
// Accumulation (the sums of Eq. (1)) has two forms, both with every addition in
// an order fixed by the problem shape (and the hardware's lane order):
//   wave    -- each wavefront adds its own tiles into private fp64 slabs
//              (accumulate_tile: LDS fp64 adds in program order, no barriers),
//              one slab per object of a step, or (when that leaves fewer
//              waves) one slab that the objects of a step share, the LDS
//              applying the lanes of one add in a fixed order; at the end the
//              workgroup adds the slabs in a fixed order. Used while W >= 6 (5)
//              waves' private slabs fit in LDS (small K*M).
//   ring    -- one fp64 slab per workgroup that the waves take turns to add
//              their tiles into, in the fixed cyclic order wave 0, 1, ..., W-1
//              of every step (a turn counter in LDS; no barriers): one lane per
//              object, one LDS fp64 add per feature, the LDS applying the lanes
//              of one add in a fixed order. A wave's turn overlaps the other
//              waves' distance work. Used for large K*M.
#include "lloyd.h"
#include "lloyd_device.h"

#include <float.h>
#include <math.h>

#include <array>
#include <type_traits>
#include <utility>

#include "lloyd_parts.h"

namespace lloyd {

namespace {

typedef float f4v __attribute__((ext_vector_type(4)));
// Four floats at any 4-byte-aligned address: rows of X start on any float.
typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));

constexpr int kCols = 4;      // 16-object columns per wave tile (64 objects)
// Index bits of a packed key: enough for the (padded) centres, at most 8;
// a group of 2^bits centres shares one running best / second best.
__host__ __device__ inline int key_bits(int KT)
{
    return KT <= 2 ? 5 : KT <= 4 ? 6 : KT <= 8 ? 7 : 8;
}
constexpr int kAccWave = 1;    // per-wave slabs, WaveAcc<M>::Pmax objects per step
constexpr int kAccRing = 2;    // one slab per workgroup, waves add in turn
constexpr int kAccWave1 = 3;   // one slab per wave, WaveAcc<M>::Pmax objects per step (less LDS)
constexpr int kMaxWaves = 8;
// Fewest waves the wave form is used with: with distances six; without, a wave
// spends its time on the sums and five with slabs of their own are the shorter
// way (a kmeans_update of n = 400,000, M = 57, K = 32: 44.0 us with eight waves
// in turn, 36.9 with five).
[[maybe_unused]] constexpr int min_wave_form(int mode) { return mode == kAccumLabels ? 5 : 6; }

// Candidates of an object in one lane (a quarter of the centres) up to which
// fp64 distances to them decide; more are mostly resolved by the direct form.
// An assignment with distances, all of a wave's centres by the direct form in
// fp64 where one object had more than four / now: n = 300,000, M = 16, K = 1024,
// objects and centres drawn from the same 512 points 2,006 / 193 us; n = 16,384,
// M = 25, K = 256, one object with a NaN 144 / 15.8.
constexpr int kManyCand = 16;
constexpr int kMaxList = 4096;     // noted close calls per wave, at most
// ... and at least, where the choice of waves allows it: a quarter of the 977
// objects of a wave at n = 2e6
[[maybe_unused]] constexpr int kMinList = 256;

// Operands of the split products for M features: 32-feature chunks, of which
// the last one (R features) takes one, two or three products.
template <int M>
struct Split {
    static constexpr int KC = (M + 31) / 32, R = M - 32 * (KC - 1);
    static constexpr int kForm = R <= 8 ? 1 : R <= 16 ? 2 : 3;        // products of the last chunk
    static constexpr int kA = 2 * (KC - 1) + (kForm == 3 ? 2 : 1);    // A operands per block
    static constexpr int kB = 2 * (KC - 1) + (kForm == 1 ? 1 : 2);    // B operands per column
    // additions per score on the matrix core: the products, the |c|^2 seed
    static constexpr int kAdds = 96 * (KC - 1) + 32 * kForm + 2;
    // dropped split terms, relative to |a b|, in units of 2^-16
    static constexpr float kDrop = (KC > 1 || kForm == 3) ? 3.02f : 2.01f;
};
__host__ __device__ inline int a_operands(int M)
{
    const int KC = (M + 31) / 32, R = M - 32 * (KC - 1);
    return 2 * (KC - 1) + (R <= 16 ? 1 : 2);
}

// LDS carve-up of a workgroup (dynamic shared memory).
struct MfmaLds {
    size_t abf, cnorm, misc, tiles, offs, slab, list;
    int tile_floats;
};

__host__ __device__ inline size_t al16(size_t v) { return (v + 15) & ~size_t(15); }

// Slabs per wave of a wave form.
__host__ __device__ inline int wave_acc_p(int M, int acc)
{
    if (acc == kAccWave1) return 1;
    const int lw = (M + 1 <= 2) ? 2 : (M + 1 <= 4) ? 4 : (M + 1 <= 8) ? 8
                 : (M + 1 <= 16) ? 16 : (M + 1 <= 32) ? 32 : 64;
    return kWave / lw;
}

// Row stride (doubles) of the ring form's slab: the M sums and the count,
// rounded up to an odd count, so that rows of different clusters start on
// different LDS banks (lanes of one add hit rows of arbitrary clusters).
__host__ __device__ constexpr int ring_row(int M) { return (M + 1) | 1; }

// 16-centre blocks, rounded up to an even count (the assignment loop works on
// pairs of blocks; the padding centres score +inf).
__host__ __device__ inline int centre_blocks(int K) { return ((K + 15) / 16 + 1) / 2 * 2; }

// Tile slot of a wave (floats): the 64 objects and the slack of TileGeom; at
// least the 128 objects that a wave whose list overflowed gathers there.
__host__ __device__ constexpr int tile_slot(int M)
{
    const int s = (kWave * M + (M > 4 ? M : 4) + 3) / 4 * 4;
    return s > 2 * kWave ? s : 2 * kWave;
}

// Rows of a wave form's slab: one more than there are clusters takes the adds
// of close calls, which sums from labels do not have.
__host__ __device__ inline int slab_rows(int K, int mode) { return mode == kAccumLabels ? K : K + 1; }

// (sums from labels need no centre operands)
__host__ __device__ inline MfmaLds mfma_lds(int M, int K, int W, int acc, int mode)
{
    const int KT = mode == kAccumLabels ? 0 : centre_blocks(K);
    MfmaLds L{};
    L.tile_floats = tile_slot(M);
    size_t o = 0;
    L.abf = o;     o = al16(o + (size_t)KT * a_operands(M) * kWave * 16);
    L.cnorm = o;   o = al16(o + (size_t)KT * 16 * 4);
    L.misc = o;    o = al16(o + 4 * (size_t)(2 * W + 1));  // the turn, the waves' counts and votes
    L.tiles = o;   o = al16(o + (size_t)W * L.tile_floats * 4);
    if (acc == kAccWave || acc == kAccWave1) {
        L.offs = o;    o = al16(o + (size_t)W * kWave * 4);
        L.slab = o;    o = al16(o + (size_t)W * wave_acc_p(M, acc) * slab_rows(K, mode) * (M + 1) * 8);
    } else if (acc == kAccRing) {
        L.slab = o;    o = al16(o + (size_t)K * ring_row(M) * 8);
    }
    L.list = o;
    return L;
}

// Close calls a wave can note: what the launch leaves of LDS. A launch argument,
// so that the kernel makes no 64-bit division.
[[maybe_unused]] inline int tile_list_cap(int M, int K, int W, int acc, int mode)
{
    if (mode == kAccumLabels) return 0;
    const size_t o = mfma_lds(M, K, W, acc, mode).list;
    const size_t left = o < (size_t)kMaxLds ? (size_t)kMaxLds - o : 0;
    const size_t cap = left / ((size_t)W * 8) / 2 * 2;
    return cap > (size_t)kMaxList ? kMaxList : (int)cap;
}

[[maybe_unused]] inline size_t tile_lds_bytes(int M, int K, int W, int acc, int mode)
{
    return mfma_lds(M, K, W, acc, mode).list + (size_t)W * tile_list_cap(M, K, W, acc, mode) * 8;
}

// Orders this wave's LDS accesses of different types (the hardware keeps a
// wave's LDS accesses in order by itself).
__device__ inline void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// Turns of the ring form. The counter in LDS holds the number of turns taken
// in the workgroup; wave w's turn of step s is number s*W + w. A wave waits for
// its number with a bounded number of polls (so that every wave finishes even
// if the order were ever broken; the caller reports a wait that gave up), and
// passes the turn on once its LDS adds have completed.
constexpr int kRingPolls = 1 << 22;

__device__ inline bool ring_wait(const uint32_t *turn, uint32_t want)
{
    for (int p = 0; p < kRingPolls; ++p) {
        const uint32_t now = __hip_atomic_load(turn, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        if (__builtin_amdgcn_readfirstlane(now) == want) {
            __atomic_signal_fence(__ATOMIC_SEQ_CST);   // the adds stay after the wait
            return true;
        }
        __builtin_amdgcn_s_sleep(1);
    }
    return false;
}

__device__ inline void ring_pass(uint32_t *turn, uint32_t next)
{
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
    __builtin_amdgcn_s_waitcnt(0xC07F);        // lgkmcnt(0): this wave's LDS adds are done
    __hip_atomic_store(turn, next, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

template <int M, int MODE, int ACC>
__global__ void __launch_bounds__(kMaxWaves * kWave)
lloyd_tile_kernel(const float *__restrict__ X, int64_t n, const float *__restrict__ C, int K,
                  int32_t *__restrict__ labels, const int32_t *__restrict__ labels_in,
                  float *__restrict__ min_d2, double *__restrict__ part_sums,
                  int32_t *__restrict__ part_counts, Ctl *__restrict__ ctl, int t, int fixed,
                  int force64, int lcap)
{
    using TG = TileGeom<M>;
    using SP = Split<M>;
    constexpr int KC = SP::KC, kA = SP::kA, kB = SP::kB;
    constexpr int kSlot = tile_slot(M);
    constexpr int V = TG::kVecPerLane;
    constexpr bool kAccum = MODE != kAssign;
    constexpr int kAcc = kAccum ? ACC : 0;
    constexpr bool kWaveForm = kAcc == kAccWave || kAcc == kAccWave1;
    constexpr int PA = 0;                                // most objects per step
    constexpr bool kShared = kAcc == kAccWave1;          // ... into one slab per wave
    constexpr int kP = kShared ? 1 : WaveAcc<M, PA>::P;  // slabs per wave
    extern __shared__ __align__(16) unsigned char smem[];
    const int W = blockDim.x / kWave;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int lane = threadIdx.x % kWave;
    const int tid = threadIdx.x;
    const int KT = centre_blocks(K);       // even
    const int kbits = key_bits(KT);        // index bits of the packed keys

    if (MODE != kAccumLabels && stop_before(ctl, t, fixed)) return;
    if (MODE == kAccumLabels && stop_after_assign(ctl, fixed)) return;

    const MfmaLds L = mfma_lds(M, K, W, kAcc, MODE);
    const int KR = slab_rows(K, MODE);
    float *tiles = reinterpret_cast<float *>(smem + L.tiles);
    float *tile = tiles + wave * kSlot;
    int32_t *offs = reinterpret_cast<int32_t *>(smem + L.offs) + wave * kWave;
    uint4 *abf = reinterpret_cast<uint4 *>(smem + L.abf);       // [KT][kA][64 lanes]
    float *cnorm = reinterpret_cast<float *>(smem + L.cnorm);
    uint32_t *turn = reinterpret_cast<uint32_t *>(smem + L.misc);
    // (object, limit) of the close calls of this wave
    int2 *list = reinterpret_cast<int2 *>(smem + L.list) + (size_t)wave * lcap;
    double *wslabs = reinterpret_cast<double *>(smem + L.slab) + (size_t)wave * kP * KR * (M + 1);

    // The grid works in rounds of G*W wave tiles; in round r, wave w of
    // workgroup b takes tile r*G*W + w*G + b. Rounds whose tiles are all full
    // (64 objects present) are streamed in the main loop; the one round after
    // them (the remaining tiles, fewer than G*W, the ragged one included) is
    // handled after it, its tiles going to waves 0, 1, ... of every
    // workgroup. Every workgroup runs the same rounds.
    const int64_t nq = (n + kWave - 1) / kWave;
    const int64_t nfull = n / kWave;
    const int64_t G = gridDim.x;
    const int64_t R = G * W;                   // tiles per round
    const int64_t nr_main = nfull / R;
    const int64_t qw = (int64_t)wave * G + blockIdx.x;   // this wave's tile in round 0

    // the first tile's loads go out before the prologue. One tile ahead is
    // enough: a tile's distance work (64 centres at least on the default
    // path) takes longer than a read of HBM, and a second buffer (40
    // registers at M = 37) spilled.
    float4 buf[V];
    if (nr_main > 0) load_tile<M>(X, qw, lane, buf);

    // ---- prologue: split A operands (-2C, bf16 hi and lo, in lane order),
    // centre norms, slabs. Every load is unconditional (clamped into C), a
    // batch of table entries in flight at a time: with a branch around each
    // load the table of 1024 centres took 19 us, half of the launch.
    if (kWaveForm) {
        double *slabs = reinterpret_cast<double *>(smem + L.slab);
        for (int i = tid; i < W * kP * KR * (M + 1); i += blockDim.x) slabs[i] = 0.0;
    } else if (kAcc == kAccRing) {
        double *slab = reinterpret_cast<double *>(smem + L.slab);
        for (int i = tid; i < K * ring_row(M); i += blockDim.x) slab[i] = 0.0;
        if (tid == 0) *turn = 0u;
    }
    {
        constexpr int kSlack = TG::kSlot - kWave * M;     // zeros after each tile
        for (int i = tid; i < W * kSlack; i += blockDim.x)
            tiles[(i / kSlack) * kSlot + kWave * M + (i % kSlack)] = 0.f;
    }
    if (MODE != kAccumLabels) {
        const int entries = KT * KC * kWave;
        auto build = [&](int i0, auto batch) {
            constexpr int kBatch = decltype(batch)::value;
            float raw[kBatch][8];
#pragma unroll
            for (int u = 0; u < kBatch; ++u) {
                const int idx = i0 + u * (int)blockDim.x;
                const int tt = idx / (KC * kWave), qc = (idx / kWave) % KC, lg = (idx >> 4) & 3;
                const int chunk = qc < KC - 1 || SP::kForm == 3 ? lg : SP::kForm == 2 ? (lg & 1) : 0;
                const int k = tt * 16 + (idx & 15), j0 = 32 * qc + 8 * chunk;
                const float *row = C + (int64_t)(k < K ? k : K - 1) * M;
#pragma unroll
                for (int e = 0; e < 8; ++e) raw[u][e] = row[j0 + e < M ? j0 + e : M - 1];
            }
#pragma unroll
            for (int u = 0; u < kBatch; ++u) {
                const int idx = i0 + u * (int)blockDim.x;
                const int tt = idx / (KC * kWave), qc = (idx / kWave) % KC, lg = (idx >> 4) & 3;
                const bool last = qc == KC - 1;
                const int chunk = !last || SP::kForm == 3 ? lg : SP::kForm == 2 ? (lg & 1) : 0;
                const int k = tt * 16 + (idx & 15), j0 = 32 * qc + 8 * chunk;
                float a[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) a[e] = (k < K && j0 + e < M) ? -2.0f * raw[u][e] : 0.0f;
                uint32_t hi[4], lo[4];
                split_bf16x8(a, hi, lo);
                if (idx >= entries) continue;
                uint4 *dst = abf + ((size_t)tt * kA + 2 * qc) * kWave + idx % kWave;
                if (!last || SP::kForm == 3) {
                    dst[0] = make_uint4(hi[0], hi[1], hi[2], hi[3]);
                    dst[kWave] = make_uint4(lo[0], lo[1], lo[2], lo[3]);
                } else {
                    const bool first = lg < 2;         // hi | lo side by side
                    dst[0] = make_uint4(first ? hi[0] : lo[0], first ? hi[1] : lo[1],
                                        first ? hi[2] : lo[2], first ? hi[3] : lo[3]);
                }
            }
        };
        // (batches of four as far as they go: half-empty ones cost an assignment
        // of few objects to 256 centres 1 us)
        const int rounds = (KT * KC + W - 1) / W;
        int r = 0;
        for (; r + 4 <= rounds; r += 4)
            build(tid + r * (int)blockDim.x, std::integral_constant<int, 4>{});
        if (rounds - r >= 2) {
            build(tid + r * (int)blockDim.x, std::integral_constant<int, 2>{});
            r += 2;
        }
        if (rounds - r > 0) build(tid + r * (int)blockDim.x, std::integral_constant<int, 1>{});
        // |c_k|^2 in fp32, features in order; padding centres (k >= K) get
        // the largest finite norm: their scores stay finite (a packed key of an
        // infinite score would be a NaN)
        for (int k = tid; k < KT * 16; k += blockDim.x) {
            const float *row = C + (int64_t)(k < K ? k : K - 1) * M;
            float nk = 0.f;
#pragma unroll
            for (int j = 0; j < M; ++j) {
                const float c = row[j];
                nk = __builtin_fmaf(c, c, nk);
            }
            cnorm[k] = k < K ? nk : FLT_MAX;
        }
    }
    __syncthreads();
    // the largest centre norm, in every wave
    float cmax = 0.f;
    if (MODE != kAccumLabels) {
        for (int k = lane; k < K; k += kWave) cmax = fmaxf(cmax, cnorm[k]);
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) cmax = fmaxf(cmax, __shfl_xor(cmax, off, kWave));
    }
    const int g = lane >> 4, l16 = lane & 15;
    int ncl = 0;             // close calls of this wave
    uint32_t ring_seq = 0;   // steps taken (ring form)
    bool ring_ok = true;     // every turn wait of this wave succeeded

    // B operands of the wave's tile: lane (g, l16) holds, for every 16-object
    // column c, features 32q + 8g .. 32q + 8g + 7 of object 16c + l16 split
    // into bf16 hi and lo; a last chunk of at most 16 features repeats its
    // features 8(g & 1) .. in both halves, one of at most 8 in all four lane
    // groups (hi in the even ones, lo in the odd ones). Past M the A operands
    // are zero, so the B values there only need to be finite: with M >= 16 the
    // tile's zero slack covers the last row's reads past M and the rows are
    // read straight through (the next object's features), else the reads are
    // clamped to the row.
    auto b_column = [&](const float *row, uint32_t (&bop)[kB][4]) {
        constexpr bool kClampReads = M < 16;
#pragma unroll
        for (int qc = 0; qc < KC; ++qc) {
            const bool last = qc == KC - 1;
            const int chunk = !last || SP::kForm == 3 ? g : SP::kForm == 2 ? (g & 1) : 0;
            float v[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const int f = 32 * qc + 8 * chunk + e;
                v[e] = kClampReads ? row[f < M ? f : M - 1] : row[f];
            }
            uint32_t hi[4], lo[4];
            split_bf16x8(v, hi, lo);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                if (last && SP::kForm == 1) {
                    bop[2 * qc][e] = (g & 1) ? lo[e] : hi[e];
                } else {
                    bop[2 * qc][e] = hi[e];
                    bop[2 * qc + (kB > 1 ? 1 : 0)][e] = lo[e];
                }
            }
        }
    };
    auto b_operands = [&](uint32_t (&bop)[kCols][kB][4]) {
#pragma unroll
        for (int c = 0; c < kCols; ++c) b_column(tile + (16 * c + l16) * M, bop[c]);
    };
    struct Ops {
        uint32_t a[kA][4];
        f4v c0;
    };
    auto load_ops = [&](int tt, Ops &o) {
#pragma unroll
        for (int q = 0; q < kA; ++q) {
            const uint4 v = abf[((size_t)tt * kA + q) * kWave + lane];
            o.a[q][0] = v.x;
            o.a[q][1] = v.y;
            o.a[q][2] = v.z;
            o.a[q][3] = v.w;
        }
        o.c0 = *reinterpret_cast<const f4v *>(cnorm + tt * 16 + 4 * g);
    };
    // products of a score, on top of |c|^2: per full chunk lo(A) hi(B) +
    // hi(A) lo(B) + hi(A) hi(B), then the last chunk's
    auto each_product = [&](auto &&product) {
#pragma unroll
        for (int qc = 0; qc < KC; ++qc) {
            if (qc < KC - 1 || SP::kForm == 3) product(2 * qc + (kA > 1 ? 1 : 0), 2 * qc);
            if (qc < KC - 1 || SP::kForm >= 2) product(2 * qc, 2 * qc + (kB > 1 ? 1 : 0));
            product(2 * qc, 2 * qc);
        }
    };
    // block o against the four columns
    auto chain = [&](const Ops &o, const uint32_t (&bop)[kCols][kB][4], f4v (&d)[kCols]) {
#pragma unroll
        for (int c = 0; c < kCols; ++c) d[c] = o.c0;
        each_product([&](int qa, int qb) {
#pragma unroll
            for (int c = 0; c < kCols; ++c)
                d[c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf8(o.a[qa]), as_bf8(bop[c][qb]),
                                                               d[c], 0, 0, 0);
        });
    };
    // two blocks against one column
    auto chain_pair = [&](const Ops (&o)[2], const uint32_t (&bop)[kB][4], f4v (&d)[2]) {
        d[0] = o[0].c0;
        d[1] = o[1].c0;
        each_product([&](int qa, int qb) {
#pragma unroll
            for (int u = 0; u < 2; ++u)
                d[u] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf8(o[u].a[qa]), as_bf8(bop[qb]),
                                                               d[u], 0, 0, 0);
        });
    };

    // One wave tile: stage it in LDS, put the loads of the wave's next tile
    // in flight in the same registers, assign, accumulate.
    // full: a round of the main loop (every wave tile present and full; the
    // loads of the next round are issued here) rather than the last one
    auto step = [&](int64_t r, auto full) {
        constexpr bool kFullTile = decltype(full)::value;
        const int64_t q = r * R + qw;
        const bool have = kFullTile || q < nq;
        if (have) store_tile<M>(tile, lane, buf);
        __builtin_amdgcn_wave_barrier();
        if (kFullTile && r + 1 < nr_main) load_tile<M>(X, q + R, lane, buf);
        const int64_t i = q * kWave + lane;
        const bool valid = kFullTile || (have && i < n);
        int my_lab = -1;

        if (have && MODE == kAccumLabels) {
            if (valid) {
                my_lab = labels_in[i];
                if (my_lab < 0 || my_lab >= K) my_lab = -1;
            }
        } else if (have) {
            // |x|^2 of the lane's own object (row `lane` of the tile), features
            // in order; it enters only the guard bands, whose margins cover its
            // fp32 rounding
            float mx = 0.f;
#pragma unroll
            for (int j = 0; j < M; ++j) {
                const float v = tile[lane * M + j];
                mx = __builtin_fmaf(v, v, mx);
            }
            uint32_t bop[kCols][kB][4];
            b_operands(bop);
            // Scan with packed keys: a score with its low `bits` bits
            // replaced by the centre's index within its group of 2^bits
            // centres, so that min / med3 / min keep the best and second
            // best keys and the label comes with the best one. Per group
            // each lane gathers the keys of its own object from the four
            // lanes that hold its centre rows, and the group folds into
            // the lane's running (best, second, label).
            const int gblocks = (1 << kbits) / 16;            // even
            const uint32_t kmask = ~((1u << kbits) - 1u);
            float g1 = INFINITY, g2 = INFINITY;
            int gl = 0;
            float k1[kCols], k2[kCols];
            int kt0 = 0;
            auto scan_key = [&](int tt, const f4v (&d)[kCols]) {
                // the four index values of the lane's centre rows, shared
                // by the four columns; one and-or per key, and per column
                // two (med3, min3) pairs and a min3 for the running second
                // best
                const uint32_t i0 = (uint32_t)((tt - kt0) * 16 + 4 * g);
                const uint32_t iv[4] = {i0, i0 + 1, i0 + 2, i0 + 3};
#pragma unroll
                for (int c = 0; c < kCols; ++c) {
                    float sk[4];
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        sk[r] = __uint_as_float((__float_as_uint(d[c][r]) & kmask) | iv[r]);
                    const float ma = __builtin_amdgcn_fmed3f(k1[c], sk[0], sk[1]);
                    const float b1 = fminf(fminf(k1[c], sk[0]), sk[1]);
                    const float mb = __builtin_amdgcn_fmed3f(b1, sk[2], sk[3]);
                    k1[c] = fminf(fminf(b1, sk[2]), sk[3]);
                    k2[c] = fminf(fminf(k2[c], ma), mb);
                }
            };
            Ops oA, oB;
            for (; kt0 < KT; kt0 += gblocks) {
                const int kt1 = KT - kt0 < gblocks ? KT : kt0 + gblocks;
#pragma unroll
                for (int c = 0; c < kCols; ++c) {
                    k1[c] = INFINITY;
                    k2[c] = INFINITY;
                }
                // blocks kt0 .. kt1-1 (an even count), two accumulator sets
                // and two operand sets: the matrix cores compute one block
                // while the vector ALU scans the previous one and the next
                // block's operands arrive
                f4v dA[kCols], dB[kCols];
                load_ops(kt0, oA);
                load_ops(kt0 + 1, oB);
                chain(oA, bop, dA);
                int tt = kt0;
                for (; tt + 2 < kt1; tt += 2) {
                    load_ops(tt + 2, oA);
                    chain(oB, bop, dB);
                    scan_key(tt, dA);
                    load_ops(tt + 3, oB);
                    chain(oA, bop, dA);
                    scan_key(tt + 1, dB);
                }
                chain(oB, bop, dB);
                scan_key(tt, dA);
                scan_key(tt + 1, dB);
                float b1, b2;
                own_column_keys(k1, k2, lane, b1, b2);
                const int lab = kt0 * 16 + (int)(__float_as_uint(b1) & ~kmask);
                const bool take = b1 < g1;
                g2 = second_of(g1, g2, b1, b2);
                g1 = take ? b1 : g1;
                gl = take ? lab : gl;
            }
            // Error of a score against the exact score |c|^2 - 2 x.c: with
            // a = ah + al + ea, b = bh + bl + eb (|ea| <= 2^-16 |a|, |al|
            // <= 2^-8 (1 + 2^-8) |a|, likewise b) the dropped terms
            // (a - ea) eb + al bl + ea b are below 3.02 * 2^-16 |a b| per
            // feature (2.01 * 2^-16 in a chunk that forms al bl too); the
            // products are exact in fp32 and their sums with |c|^2 take at
            // most kAdds roundings on the matrix core, each assumed only
            // faithful (within 2^-23 relative, any order or direction), so
            // they add kAdds 2^-23 of the terms' magnitudes; |c|^2 in fp32
            // adds M 2^-24 |c|^2. With 2|c_j x_j| <= c_j^2 + x_j^2 each score is
            // within E (|x|^2 + 3|c|^2), E = kDrop 2^-16 + 1.01 (kAdds + M/6) 2^-23.
            // A packed key moves its score by less than 2^(bits - 23) of the
            // score's magnitude, itself below (1 + E)(|x|^2 + 3|c|^2). So the
            // label stands when the two best keys differ by more than twice
            // E + 1.01 * 2^(bits - 23) (with margins); and a centre whose
            // score is above the best key by more than that is not the
            // nearest one.
            const float key_rel = __uint_as_float((uint32_t)(127 - 23 + kbits) << 23);   // 2^(bits-23)
            const float e1 = SP::kDrop * 1.5258789e-05f +
                             1.01f * ((float)SP::kAdds + (float)M / 6.0f) * 1.1920929e-07f +
                             1.01f * key_rel;
            const float thr = 2.02f * e1 * (3.02f * cmax + 1.0001f * mx) + 1e-30f;
            const bool ok = !force64 && ((K == 1) || (g2 - g1 > thr));
            // a padding centre (index >= K, |c|^2 = FLT_MAX) wins only when
            // every real score overflows; keep such a label in range
            const int ml = gl < K ? gl : K - 1;
            const bool close = valid && !ok;
            const uint64_t cm = __ballot(close);
            if (cm != 0ull) {
                const int pos = ncl + (int)__builtin_amdgcn_mbcnt_hi(
                    (uint32_t)(cm >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)cm, 0u));
                if (close && pos < lcap) list[pos] = make_int2((int)i, __float_as_int(g1 + thr));
                ncl += (int)__popcll(cm);
            }
            if (valid) {
                labels[i] = close ? -1 : ml;
                if (MODE == kAssign && min_d2 != nullptr && !close) {
                    const float *c = C + (int64_t)ml * M;
                    float d = 0.f;
#pragma unroll
                    for (int j = 0; j < M; ++j) {
                        const float e = tile[lane * M + j] - c[j];
                        d = __builtin_fmaf(e, e, d);
                    }
                    min_d2[i] = d;
                }
                // a close call's features go to the spare row of the wave
                // forms and, in the ring form, nowhere
                my_lab = !close ? ml : kWaveForm ? K : -1;
            }
        }

        if (kWaveForm) {
            // (labels read back may be out of range even in a full tile)
            if (have)
                accumulate_tile<M, PA, kFullTile && MODE != kAccumLabels, kShared>(
                    valid ? my_lab : -1, tile, offs, wslabs, KR, lane);
        } else if (kAcc == kAccRing) {
            // This wave's turn of the step (every wave takes it, with or
            // without objects): lane l adds object l's features and count to
            // its cluster's row of the workgroup slab. The features are read
            // from the wave's own tile before the wait.
            const bool adds = valid && my_lab >= 0;
            float xv[M];
#pragma unroll
            for (int j = 0; j < M; ++j) xv[j] = tile[lane * M + j];
            const uint32_t want =
                __builtin_amdgcn_readfirstlane(ring_seq * (uint32_t)W + (uint32_t)wave);
            if (ring_ok) ring_ok = ring_wait(turn, want);
            if (adds) {
                constexpr int RS = ring_row(M);
                double *row = reinterpret_cast<double *>(smem + L.slab) + (int64_t)my_lab * RS;
#pragma unroll
                for (int j = 0; j < M; ++j)
                    __hip_atomic_fetch_add(row + j, (double)xv[j], __ATOMIC_RELAXED,
                                           __HIP_MEMORY_SCOPE_WORKGROUP);
                __hip_atomic_fetch_add(row + M, 1.0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            }
            ring_pass(turn, want + 1);
            ++ring_seq;
        }
    };

    // Every wave of a workgroup runs the same steps (the ring form needs every
    // wave's turn in every step).
    for (int64_t r = 0; r < nr_main; ++r) step(r, std::true_type{});
    if (nr_main * R < nq) {
        const int64_t q = nr_main * R + qw;
        if (q < nfull) load_tile<M>(X, q, lane, buf);
        else if (q < nq) load_tail_tile<M>(X, n, q, lane, buf);
        step(nr_main, std::false_type{});
    }

    // ---- the close calls
    auto load_row = [&](int i, float (&x)[M]) {
        const float *xr = X + (int64_t)i * M;
#pragma unroll
        for (int j = 0; j + 4 <= M; j += 4) {
            const f4u v = *reinterpret_cast<const f4u *>(xr + j);
            x[j] = v[0];
            x[j + 1] = v[1];
            x[j + 2] = v[2];
            x[j + 3] = v[3];
        }
#pragma unroll
        for (int j = M / 4 * 4; j < M; ++j) x[j] = xr[j];
    };
    // label of the lane's object x (open lanes) by the direct form over all
    // centres: each fp32 distance is within gamma_{M+1} of the exact one, and
    // fp64 among the centres that this leaves within 4 gamma_{M+2} of the best
    // decides where there are several. An object with a NaN or an infinity is
    // at no finite distance from any centre: label 0.
    auto is_finite = [&](const float (&x)[M]) {
        bool f = true;
#pragma unroll
        for (int j = 0; j < M; ++j) f = f && fabsf(x[j]) < INFINITY;
        return f;
    };
    auto direct = [&](const float (&x)[M], bool open) -> int {
        constexpr float kTau = 4.0f * (float)(M + 2) * 5.9604645e-8f;
        auto dist = [&](int k) {
            float d = 0.f;
#pragma unroll
            for (int j = 0; j < M; ++j) {
                const float e = x[j] - C[k * M + j];
                d = __builtin_fmaf(e, e, d);
            }
            return d;
        };
        float b1 = INFINITY, b2 = INFINITY;
        int ld = 0;
        if (!force64)
#pragma unroll (M <= 16 ? 4 : 1)
            for (int k = 0; k < K; ++k) {
                const float d = dist(k);
                const bool lt = d < b1;
                b2 = __builtin_amdgcn_fmed3f(b1, b2, d);
                b1 = lt ? d : b1;
                ld = lt ? k : ld;
            }
        const bool sure = !force64 && ((K == 1) || (b2 - b1 > kTau * b2 && b2 >= 1e-30f));
        const bool unsure = open && !sure && is_finite(x);
        if (__ballot(unsure) != 0ull) {
            double bd = INFINITY;
            int l64 = 0;
            for (int k = 0; k < K; ++k) {
                bool in = unsure;
                if (!force64) {
                    const float d = dist(k);
                    // (a NaN or an overflowed distance stays in question)
                    in = unsure && !(d - b1 > kTau * d && d >= 1e-30f);
                }
                if (__ballot(in) == 0ull) continue;
                const double dk = dist_fp64<M>(x, C + (int64_t)k * M);
                if (in && dk < bd) {
                    bd = dk;
                    l64 = k;
                }
            }
            ld = unsure ? l64 : ld;
        }
        return is_finite(x) ? ld : 0;
    };
    auto store_label = [&](const float (&x)[M], int i, int lab, int mark) {
        labels[i] = lab ^ mark;
        if (MODE == kAssign && min_d2 != nullptr)
            min_d2[i] = reported_d2<M>(x, C + (int64_t)lab * M);
    };
    int first[kMaxWaves + 1];      // list position of each wave's first object
    first[0] = 0;
    int total = 0;                 // objects in the lists
    uint32_t over = 0;             // waves whose list overflowed
    // place of list position p: in the list of the last wave that starts at
    // or before it
    auto entry = [&](int p) -> int2 * {
        int w = 0, base = 0;
#pragma unroll
        for (int v = 1; v < kMaxWaves; ++v)
            if (p >= first[v]) {
                w = v;
                base = first[v];
            }
        return reinterpret_cast<int2 *>(smem + L.list) + (size_t)w * lcap + (p - base);
    };
    if (MODE != kAccumLabels) {
        // The close calls of the workgroup's waves, one list after the other,
        // in columns of 16 objects dealt to the waves in turn (a wave alone
        // rarely has many, and a column costs a quarter of a tile or more).
        // The four lanes (g, l16) of an object hold its features and find the
        // candidates among their own centre rows.
        int *wcount = reinterpret_cast<int *>(smem + L.misc) + 1;
        if (lane == 0) wcount[wave] = ncl;
        __syncthreads();
        int all = 0, batches = 0;
#pragma unroll
        for (int w = 0; w < kMaxWaves; ++w) {
            const int c = w < W ? wcount[w] : 0;
            all += c;
            if (c > lcap) {
                batches += (c + kWave - 1) / kWave;
                over |= 1u << w;
            }
            first[w + 1] = first[w] + (c <= lcap ? c : 0);
        }
        total = __builtin_amdgcn_readfirstlane(first[kMaxWaves]);
        over = __builtin_amdgcn_readfirstlane(over);
        const int columns = (total + 15) / 16;
        batches += columns;
        // features of a column's objects, the four lanes of each holding them
        // all, and their operands
        auto load_column = [&](int i, float (&x)[M], uint32_t (&bop)[kB][4]) {
            load_row(i, x);
            wave_sync();
            if (g == 0)
#pragma unroll
                for (int j = 0; j < M; ++j) tile[l16 * M + j] = x[j];
            wave_sync();
            b_column(tile + l16 * M, bop);
        };
        // one add per workgroup: adds of 2048 waves to one word take 20 us
        if (ctl != nullptr && tid == 0 && all > 0) {
            atomicAdd(&ctl->fallbacks, all);
            atomicAdd(&ctl->reruns, batches);
        }
        // Where the guard band is wide against the distances between the
        // centres (clusters far from the origin), most centres are candidates,
        // and the direct form, one object per lane, is the shorter way (n =
        // 300,000, M = 25, K = 256, offset 20 times the spread: 200 us, 640
        // column by column): a wave that meets such a column takes its columns
        // four at a time from then on. A column's sums have the same turn and
        // order either way.
        bool wide = force64 != 0;       // (uniform)
        for (int col = wave; col < columns;) {
            if (wide) {
                const int mine = col + g * W;               // lane (g, l16): object l16 of it
                const int p = 16 * mine + l16;
                const bool act = p < total;
                const int i = entry(act ? p : 16 * col)->x;
                float x[M];
                load_row(i, x);
                const int lab = direct(x, act);
                if (act) store_label(x, i, lab, 0);
                for (int c = 0; kAcc != 0 && c < 4 && col + c * W < columns; ++c) {
                    const uint32_t want = ring_seq * (uint32_t)W + (uint32_t)(col + c * W);
                    if (kAcc == kAccRing && ring_ok) ring_ok = ring_wait(turn, want);
                    if (act && g == c) {
                        double *row = kWaveForm
                            ? wslabs + (size_t)lab * (M + 1)
                            : reinterpret_cast<double *>(smem + L.slab) + (int64_t)lab * ring_row(M);
#pragma unroll
                        for (int j = 0; j < M; ++j)
                            __hip_atomic_fetch_add(row + j, (double)x[j], __ATOMIC_RELAXED,
                                                   __HIP_MEMORY_SCOPE_WORKGROUP);
                        __hip_atomic_fetch_add(row + M, 1.0, __ATOMIC_RELAXED,
                                               __HIP_MEMORY_SCOPE_WORKGROUP);
                    }
                    if (kAcc == kAccRing) ring_pass(turn, want + 1);
                }
                col += 4 * W;
                continue;
            }
            const int p = 16 * col + l16;
            const bool act = p < total;
            const int2 e = *entry(act ? p : 16 * col);
            const int i = e.x;
            const float lim = act ? __int_as_float(e.y) : -INFINITY;
            float x[M];
            uint32_t bop[kB][4];
            load_column(i, x, bop);
            int lab = 0;
            bool open;
            {
                // up to four candidates of this lane, 16 bits each
                uint64_t cand = 0;
                int nc = 0;
                Ops o[2], nx[2];
                load_ops(0, nx[0]);
                load_ops(1, nx[1]);
                for (int tt = 0; tt < KT; tt += 2) {
                    o[0] = nx[0];
                    o[1] = nx[1];
                    const int tn = tt + 2 < KT ? tt + 2 : tt;
                    load_ops(tn, nx[0]);
                    load_ops(tn + 1, nx[1]);
                    f4v d[2];
                    chain_pair(o, bop, d);
                    // a NaN score (which the sum keeps) or limit makes the
                    // centre a candidate
                    const float lo = fminf(fminf(fminf(d[0][0], d[0][1]), fminf(d[0][2], d[0][3])),
                                           fminf(fminf(d[1][0], d[1][1]), fminf(d[1][2], d[1][3])));
                    const float sum = ((d[0][0] + d[0][1]) + (d[0][2] + d[0][3])) +
                                      ((d[1][0] + d[1][1]) + (d[1][2] + d[1][3]));
                    if (__ballot(!(lo > lim) || sum != sum) == 0ull) continue;
#pragma unroll
                    for (int u = 0; u < 2; ++u)
#pragma unroll
                        for (int r = 0; r < 4; ++r) {
                            const int k = (tt + u) * 16 + 4 * g + r;
                            const bool in = !(d[u][r] > lim) && k < K;
                            cand = in ? (cand << 16) | (uint64_t)k : cand;
                            nc += in ? 1 : 0;
                        }
                }
                int most = nc, some = nc;
#pragma unroll
                for (int m = 16; m <= 32; m <<= 1) {
                    const int om = __shfl_xor(most, m, kWave);
                    most = om > most ? om : most;
                    some += __shfl_xor(some, m, kWave);
                }
                // (an object that is not finite has every centre for a candidate)
                bool finite = true;
                open = false;
                bool many = false;
                if (__ballot(act && (most > 4 || some == 0)) != 0ull) {
                    finite = is_finite(x);
                    open = act && finite && (most > kManyCand || some == 0);
                    many = act && finite && most > 4 && most <= kManyCand;
                    if (__popcll(__ballot(open)) >= kWave / 4) {
                        wide = true;
                        continue;              // this column too
                    }
                }
                double bd = INFINITY;
                auto consider = [&](int k, bool take) {
                    const double dk = dist_fp64<M>(x, C + (int64_t)k * M);
                    if (take && (dk < bd || (dk == bd && dk < INFINITY && k < lab))) {
                        bd = dk;
                        lab = k;
                    }
                };
                if (finite && most <= 4)
                    for (int u = 0; u < nc; ++u)
                        consider((int)((cand >> (16 * u)) & 0xffffu), true);
                if (__ballot(many) != 0ull) {
                    // more than the four that were kept: the scores once more,
                    // the candidates' distances as they turn up
                    for (int tt = 0; tt < KT; tt += 2) {
                        load_ops(tt, o[0]);
                        load_ops(tt + 1, o[1]);
                        f4v d[2];
                        chain_pair(o, bop, d);
                        uint32_t in = 0u;
#pragma unroll
                        for (int u = 0; u < 2; ++u)
#pragma unroll
                            for (int r = 0; r < 4; ++r)
                                in |= many && !(d[u][r] > lim) && (tt + u) * 16 + 4 * g + r < K
                                          ? 1u << (4 * u + r) : 0u;
                        for (; __ballot(in != 0u) != 0ull; in &= in - 1u) {
                            const int bit = in != 0u ? __builtin_ctz(in) : 0;
                            consider(in != 0u ? (tt + (bit >> 2)) * 16 + 4 * g + (bit & 3) : 0,
                                     in != 0u);
                        }
                    }
                }
#pragma unroll
                for (int m = 16; m <= 32; m <<= 1) {
                    const double od = __shfl_xor(bd, m, kWave);
                    const int ol = __shfl_xor(lab, m, kWave);
                    if (od < bd || (od == bd && ol < lab)) {
                        bd = od;
                        lab = ol;
                    }
                }
            }
            if (__ballot(open) != 0ull) {
                const int ld = direct(x, open);
                lab = open ? ld : lab;
            }
            if (act && g == 0) store_label(x, i, lab, 0);
            if (kAcc != 0) {
                // lane (g, l16) adds features g, g + 4, ... of its object, to
                // the wave's first slab or, in the column's turn, to the
                // workgroup's
                const uint32_t want = ring_seq * (uint32_t)W + (uint32_t)col;
                if (kAcc == kAccRing && ring_ok) ring_ok = ring_wait(turn, want);
                if (act) {
                    double *row = kWaveForm
                        ? wslabs + (size_t)lab * (M + 1)
                        : reinterpret_cast<double *>(smem + L.slab) + (int64_t)lab * ring_row(M);
#pragma unroll
                    for (int j = 0; j < M; j += 4) {
                        float a0 = x[j], a1 = x[j + 1 < M ? j + 1 : j];
                        float a2 = x[j + 2 < M ? j + 2 : j], a3 = x[j + 3 < M ? j + 3 : j];
                        asm("" : "+v"(a0), "+v"(a1), "+v"(a2), "+v"(a3));   // values, not addresses
                        const float v01 = (g & 1) ? a1 : a0, v23 = (g & 1) ? a3 : a2;
                        const float v = g < 2 ? v01 : v23;
                        if (j + 4 <= M || j + g < M)
                            __hip_atomic_fetch_add(row + j + g, (double)v, __ATOMIC_RELAXED,
                                                   __HIP_MEMORY_SCOPE_WORKGROUP);
                    }
                    if (g == 0)
                        __hip_atomic_fetch_add(row + M, 1.0, __ATOMIC_RELAXED,
                                               __HIP_MEMORY_SCOPE_WORKGROUP);
                }
                if (kAcc == kAccRing) ring_pass(turn, want + 1);
            }
            col += W;
        }
        // A list that overflowed is not used: its wave's tiles are read again
        // for marked labels, through a buffer of 128 objects (the list's
        // place, or the idle tile slot).
        if (ncl > lcap) {
            if (lcap < kWave) wave_sync();
            int *sbuf = lcap >= kWave ? reinterpret_cast<int *>(list) : reinterpret_cast<int *>(tile);
            int have = 0;
            int64_t q = qw;
            for (;;) {
                while (have < kWave && q < nq) {
                    const int64_t i = q * kWave + lane;
                    const bool mark = i < n && labels[i] < 0;
                    const uint64_t mm = __ballot(mark);
                    const int pos = have + (int)__builtin_amdgcn_mbcnt_hi(
                        (uint32_t)(mm >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mm, 0u));
                    if (mark) sbuf[pos] = (int)i;
                    have += (int)__popcll(mm);
                    q += R;
                }
                wave_sync();
                if (have == 0) break;
                const int m = have < kWave ? have : kWave;
                have -= m;
                const bool act = lane < m;
                const int i = sbuf[have + (act ? lane : 0)];
                wave_sync();
                float x[M];
                load_row(i, x);
                const int lab = direct(x, act);
                // in the ring form the label keeps its mark until the sums below
                if (act) {
                    store_label(x, i, lab, kAcc == kAccRing ? -1 : 0);
                    if (kWaveForm) {
                        // one lane per object: the LDS applies the lanes of
                        // an add in a fixed order
                        double *row = wslabs + (size_t)lab * (M + 1);
#pragma unroll
                        for (int j = 0; j < M; ++j)
                            __hip_atomic_fetch_add(row + j, (double)x[j], __ATOMIC_RELAXED,
                                                   __HIP_MEMORY_SCOPE_WAVEFRONT);
                        __hip_atomic_fetch_add(row + M, 1.0, __ATOMIC_RELAXED,
                                               __HIP_MEMORY_SCOPE_WAVEFRONT);
                    }
                }
            }
        }
    }
    if (kAcc == kAccRing && MODE != kAccumLabels && over != 0) {
        // The sums of the marked objects of the waves whose list overflowed, in
        // a fixed order: waves ascending, their tiles ascending, lanes
        // ascending. Each wave adds its own share of the features of all of
        // them (the count goes with feature 0), so that no sum is shared
        // between waves.
        constexpr int RS = ring_row(M);
        constexpr int kPer = (M + kMaxWaves - 1) / kMaxWaves;   // features at a time
        constexpr int kAhead = 4;                               // batches in flight
        double *slab = reinterpret_cast<double *>(smem + L.slab);
        const int j0 = M * wave / W, j1 = M * (wave + 1) / W;
        // batch: kAhead x 64 objects i with labels lab (-1: none)
        auto add_batch = [&](const int64_t (&i)[kAhead], const int (&lab)[kAhead]) {
            for (int jc = j0; jc < j1; jc += kPer) {
                float v[kAhead][kPer];
#pragma unroll
                for (int u = 0; u < kAhead; ++u)
#pragma unroll
                    for (int j = 0; j < kPer; ++j)
                        v[u][j] = X[i[u] * M + (jc + j < j1 ? jc + j : j0)];
#pragma unroll
                for (int u = 0; u < kAhead; ++u)
                    if (lab[u] >= 0) {
                        double *row = slab + (int64_t)lab[u] * RS;
#pragma unroll
                        for (int j = 0; j < kPer; ++j)
                            if (jc + j < j1)
                                __hip_atomic_fetch_add(row + jc + j, (double)v[u][j],
                                                       __ATOMIC_RELAXED,
                                                       __HIP_MEMORY_SCOPE_WORKGROUP);
                        if (jc == 0)
                            __hip_atomic_fetch_add(row + M, 1.0, __ATOMIC_RELAXED,
                                                   __HIP_MEMORY_SCOPE_WORKGROUP);
                    }
            }
        };
        __syncthreads();                           // every object is decided
        for (int w = 0; w < W; ++w) {
            if (((over >> w) & 1u) == 0u) continue;
            for (int64_t q = (int64_t)w * G + blockIdx.x; q < nq; q += kAhead * R) {
                int64_t i[kAhead];
                int lab[kAhead];
#pragma unroll
                for (int u = 0; u < kAhead; ++u) {
                    const int64_t iu = (q + u * R) * kWave + lane;
                    i[u] = iu < n ? iu : 0;
                    lab[u] = iu < n ? ~labels[iu] : -1;
                }
                add_batch(i, lab);
            }
        }
        __syncthreads();                           // every mark has been read
        if (ncl > lcap)
            for (int64_t q = qw; q < nq; q += R) {
                const int64_t i = q * kWave + lane;
                if (i < n) {
                    const int v = labels[i];
                    if (v < 0) labels[i] = ~v;
                }
            }
    }

    if (kAcc == kAccRing && ctl != nullptr && lane == 0 && !ring_ok) atomicAdd(&ctl->ring_stalls, 1);

    if (kWaveForm) {
        __syncthreads();
        write_wave_partials<M, PA, kShared>(reinterpret_cast<const double *>(smem + L.slab), W, K, KR,
                               part_sums + (int64_t)blockIdx.x * K * M,
                               part_counts + blockIdx.x, gridDim.x);
    } else if (kAcc == kAccRing) {
        __syncthreads();
        constexpr int RS = ring_row(M);
        const double *slab = reinterpret_cast<const double *>(smem + L.slab);
        double *out = part_sums + (int64_t)blockIdx.x * K * M;
        for (int e = tid; e < K * (M + 1); e += blockDim.x) {
            const int k = e / (M + 1), j = e % (M + 1);
            const double v = slab[k * RS + j];
            if (j < M) out[(int64_t)k * M + j] = v;
            else part_counts[(int64_t)k * gridDim.x + blockIdx.x] = (int32_t)v;
        }
    }
}

template <int M>
hipError_t launch_m(const StepArgs &a, Mode mode, const AccumPlan &p, hipStream_t s)
{
    const dim3 grid(p.groups), block(p.waves * kWave);
#define LLOYD_MFMA_LAUNCH(MD, AC)                                                              \
    do {                                                                                       \
        auto kern = lloyd_tile_kernel<M, MD, AC>;                                              \
        static const size_t st = static_lds_bytes(reinterpret_cast<const void *>(kern));       \
        if (st > (size_t)kMaxLds || st + p.lds_bytes > (size_t)kMaxLds)                        \
            return hipErrorInvalidConfiguration;                                               \
        LLOYD_STEP_LAUNCH(kern, grid, block, p.lds_bytes, s, a,                                \
                              a.X, a.n, a.C, a.K, a.labels, a.labels_in, a.min_d2,            \
                              a.part_sums, a.part_counts, a.ctl, a.t, a.fixed, a.force64,     \
                              p.list_cap);                                                    \
    } while (0)
    switch (mode) {
    case kAssign: LLOYD_MFMA_LAUNCH(kAssign, 0); break;
    case kAssignAccum:
        if (p.accum == kAccWave) LLOYD_MFMA_LAUNCH(kAssignAccum, kAccWave);
        else if (p.accum == kAccWave1) LLOYD_MFMA_LAUNCH(kAssignAccum, kAccWave1);
        else LLOYD_MFMA_LAUNCH(kAssignAccum, kAccRing);
        break;
    case kAccumLabels:
        if (p.accum == kAccWave) LLOYD_MFMA_LAUNCH(kAccumLabels, kAccWave);
        else if (p.accum == kAccWave1) LLOYD_MFMA_LAUNCH(kAccumLabels, kAccWave1);
        else LLOYD_MFMA_LAUNCH(kAccumLabels, kAccRing);
        break;
    }
#undef LLOYD_MFMA_LAUNCH
    return hipGetLastError();
}

using LaunchFn = hipError_t (*)(const StepArgs &, Mode, const AccumPlan &, hipStream_t);

// This translation unit instantiates the kernels for the feature counts of
// one part of [1, kMaxM] (the build compiles it once per part, in parallel).
constexpr int kPartLo = LLOYD_PART * kMaxM / LLOYD_PARTS + 1;
constexpr int kPartN = kMaxM / LLOYD_PARTS;

template <int... Is>
constexpr auto make_table(std::integer_sequence<int, Is...>)
{
    return std::array<LaunchFn, sizeof...(Is)>{&launch_m<kPartLo + Is>...};
}

}  // namespace

hipError_t LLOYD_PART_FN(launch_tile_part)(const StepArgs &a, Mode mode, const AccumPlan &plan, hipStream_t s)
{
    static constexpr auto table = make_table(std::make_integer_sequence<int, kPartN>{});
    if (a.M < kPartLo || a.M >= kPartLo + kPartN) return hipErrorInvalidValue;
    const LaunchFn fn = table[a.M - kPartLo];
    return fn ? fn(a, mode, plan, s) : hipErrorInvalidValue;
}

#if LLOYD_PART == 0
namespace {

// Most waves of a workgroup whose state fits in LDS with a list of kMinList
// each (sums from labels note no close calls), or one wave with what is left
// (0: not even one fits).
int most_waves(int M, int K, int acc, Mode mode)
{
    for (int w = kMaxWaves; w > 0; --w) {
        if (tile_lds_bytes(M, K, w, acc, mode) <= (size_t)kMaxLds &&
            (w == 1 || mode == kAccumLabels || tile_list_cap(M, K, w, acc, mode) >= kMinList))
            return w;
    }
    return 0;
}

// Accumulation form and waves of an accumulating launch: private slabs (the
// most objects per step that leaves the most waves) while at least
// min_wave_form waves fit, else one shared slab, which leaves more waves.
int accum_form(int M, int K, Mode mode, int &waves)
{
    const int w_p = most_waves(M, K, kAccWave, mode), w_1 = most_waves(M, K, kAccWave1, mode);
    if (w_p >= min_wave_form(mode) && w_p >= w_1) {
        waves = w_p;
        return kAccWave;
    }
    if (w_1 >= min_wave_form(mode)) {
        waves = w_1;
        return kAccWave1;
    }
    waves = most_waves(M, K, kAccRing, mode);
    return kAccRing;
}

}  // namespace

AccumPlan plan_tile(int64_t n, int M, int K, Mode mode)
{
    AccumPlan p{};
    p.path = kPathTile;
    const int64_t nq = (n + kWave - 1) / kWave;
    int W = kMaxWaves, acc = 0;
    if (mode == kAssign) W = most_waves(M, K, 0, mode);
    else acc = accum_form(M, K, mode, W);
    // no more waves than there are 64-object tiles
    while (W > 1 && W / 2 >= nq) W /= 2;
    int64_t groups = (nq + W - 1) / W;
    if (groups > kCUs) groups = kCUs;       // one persistent workgroup per compute unit
    p.waves = W;
    p.groups = (int)groups;
    p.accum = acc;
    p.list_cap = tile_list_cap(M, K, W, acc, mode);
    p.lds_bytes = tile_lds_bytes(M, K, W, acc, mode);
    return p;
}

// The shapes that a forced matrix-core path takes: centre operands of two
// 16-byte parts per 32 features and lane, one tile and the workgroup slab in
// one workgroup's LDS (an upper bound of what the launches need).
bool tile_fits(int M, int K)
{
    const size_t table = (size_t)centre_blocks(K) * ((M + 31) / 32) * kWave * 32;
    const size_t norms = al16((size_t)centre_blocks(K) * 16 * 4) + 16;
    const size_t tile = al16((size_t)((kWave * M + (M > 4 ? M : 4) + 3) / 4 * 4) * 4);
    return al16(table + norms + tile) + al16((size_t)K * ring_row(M) * 8) <= (size_t)kMaxLds;
}

bool tile_sums_in_turn(int M, int K)
{
    int W = 0;
    return accum_form(M, K, kAccumLabels, W) == kAccRing;
}

int tile_waves(int M, int K, Mode mode)
{
    int W = 0;
    if (mode == kAssign) W = most_waves(M, K, 0, mode);
    else accum_form(M, K, mode, W);
    return W;
}

hipError_t launch_tile(const StepArgs &a, Mode mode, const AccumPlan &plan, hipStream_t s)
{
    if (a.M < 1 || a.M > kMaxM || plan.waves < 1) return hipErrorInvalidValue;
    switch ((a.M - 1) / (kMaxM / LLOYD_PARTS)) {
#define LLOYD_CASE(P) case P: return launch_tile_part_##P(a, mode, plan, s);
        LLOYD_PART_CASES
#undef LLOYD_CASE
    }
    return hipErrorInvalidValue;
}
#endif

}  // namespace lloyd
