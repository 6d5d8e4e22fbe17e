// The sums of Eq. (1) from labels, for shapes whose K x M fp64 slab does not fit
// in LDS beside the distance kernel's state: the second of the two launches
// that such an iteration (or kmeans_update) makes in place of the fused one.
//
// What bounds it: K x M = 16384 sums take 128 KB as one slab, so a workgroup
// with all features holds one slab that its waves share in turns, and 256
// workgroups write 34 MB of partials that the centres launch reads again (31 us
// at K = 1024, M = 16). Instead a workgroup takes S features: a wave's private
// slab is then K x S sums (32 KB at K = 1024, S = 4), no wave waits for another,
// and the M / S slices share the chip with G row groups, so that G x M / S
// workgroups fill it while only G rows of partials are written (64 at M = 16:
// 8.4 MB). Each slice reads its S features of every row, so the lines of X are
// asked for by M / S workgroups, and with rows that are no multiple of 16 bytes
// in pieces across them: S is the largest of 16, 8 and 4 that leaves six waves
// their slabs and fills the chip (a kmeans_update of n = 400,000: M = 57, K = 140
// 105 us with S = 4, 34.6 with S = 16; M = 37, K = 200 95.6 and 43.0; fewer waves
// with more features: M = 25, K = 512, n = 16,384 23.4 us with four, 18.9 with
// eight).
//
// Lane l of a wave holds object l of its tile and adds each of its features to
// the row of its cluster with an LDS fp64 add; the slab is feature-major, so
// lanes of different clusters spread over the banks, and lanes of one cluster
// are applied by the LDS in ascending order. A wave's tiles are ascending and
// the waves' slabs are added in wave order: the order of every sum is fixed by
// the shape.
#include "lloyd.h"

namespace lloyd {

namespace {

// Four floats at any 4-byte-aligned address: one 16-byte load per object (four
// 4-byte loads of 64 different lines each bound the launch: 23.5 us at n =
// 262147, M = 16, K = 1024)
typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));
constexpr int kAccWaves = 8;         // waves per workgroup, at most
constexpr int kAccMinWaves = 6;      // ... and at least, with more than 4 features each

// row stride of a feature of the slab: odd, so that the features of a cluster
// start on different banks when the slabs are added
__host__ __device__ inline int slab_row(int K) { return K | 1; }

__host__ __device__ inline size_t slab_bytes(int K, int slice)
{
    return (size_t)slice * slab_row(K) * 8 + (size_t)((K + 1) / 2 * 2) * 4;
}

template <int kSlice>
__global__ void __launch_bounds__(kAccWaves * kWave)
accum_labels_kernel(const float *__restrict__ X, int64_t n, int M,
                    const int32_t *__restrict__ labels, int K, double *__restrict__ part_sums,
                    int32_t *__restrict__ part_counts, const Ctl *__restrict__ ctl, int fixed)
{
    if (stop_after_assign(ctl, fixed)) return;
    extern __shared__ __align__(16) unsigned char smem[];
    const int W = blockDim.x / kWave;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int lane = threadIdx.x % kWave;
    const int KS = slab_row(K);
    double *sums = reinterpret_cast<double *>(smem);                       // [W][kSlice][KS]
    int32_t *cnts = reinterpret_cast<int32_t *>(sums + (size_t)W * kSlice * KS);   // [W][K]
    const int f0 = blockIdx.y * kSlice;
    const int nf = M - f0 < kSlice ? M - f0 : kSlice;
    for (int e = threadIdx.x; e < W * kSlice * KS; e += blockDim.x) sums[e] = 0.0;
    for (int e = threadIdx.x; e < W * K; e += blockDim.x) cnts[e] = 0;

    const int64_t nq = (n + kWave - 1) / kWave;
    const int64_t stride = (int64_t)gridDim.x * W;
    double *mine = sums + (size_t)wave * kSlice * KS;
    int32_t *count = cnts + (size_t)wave * K;

    const bool whole = nf == kSlice;
    struct Tile {
        float x[kSlice];
        int lab;
    };
    // (a tile past the end reads the last object and adds nothing)
    auto fetch = [&](int64_t q, Tile &t) {
        const int64_t i = q * kWave + lane;
        const int64_t r = i < n ? i : n - 1;
        const float *row = X + r * M;
        if (M < 4) {
#pragma unroll
            for (int j = 0; j < kSlice; ++j) t.x[j] = row[f0 + (j < nf ? j : 0)];
        } else if (whole) {
#pragma unroll
            for (int j = 0; j < kSlice; j += 4) {
                const f4u v = *reinterpret_cast<const f4u *>(row + f0 + j);
#pragma unroll
                for (int u = 0; u < 4; ++u) t.x[j + u] = v[u];
            }
        } else {
            // pieces past the row start at its last four features and are moved
            // down to their own (what is past the row's end is not added)
#pragma unroll
            for (int j = 0; j < kSlice; j += 4) {
                const int at = f0 + j + 4 <= M ? f0 + j : M - 4, sh = f0 + j - at;
                const f4u v = *reinterpret_cast<const f4u *>(row + at);
                t.x[j] = sh == 0 ? v[0] : sh == 1 ? v[1] : sh == 2 ? v[2] : v[3];
                t.x[j + 1] = sh == 0 ? v[1] : sh == 1 ? v[2] : v[3];
                t.x[j + 2] = sh == 0 ? v[2] : v[3];
                t.x[j + 3] = v[3];
            }
        }
        const int lab = labels[r];
        t.lab = (i < n && lab >= 0 && lab < K) ? lab : -1;
    };
    auto add = [&](const Tile &t) {
        if (t.lab >= 0) {
#pragma unroll
            for (int j = 0; j < kSlice; ++j)
                if (j < nf)
                    __hip_atomic_fetch_add(mine + j * KS + t.lab, (double)t.x[j], __ATOMIC_RELAXED,
                                           __HIP_MEMORY_SCOPE_WAVEFRONT);
            if (blockIdx.y == 0) atomicAdd(count + t.lab, 1);
        }
    };
    __syncthreads();
    // tiles in flight (32 features of an object) while those before are added
    constexpr int kAhead = 32 / kSlice;
    const int64_t q0 = (int64_t)wave * gridDim.x + blockIdx.x;
    auto fetch_set = [&](int64_t q, Tile (&t)[kAhead]) {
#pragma unroll
        for (int u = 0; u < kAhead; ++u) fetch(q + u * stride, t[u]);
    };
    auto add_set = [&](const Tile (&t)[kAhead]) {
#pragma unroll
        for (int u = 0; u < kAhead; ++u) add(t[u]);
    };
    Tile a[kAhead], b[kAhead];
    fetch_set(q0, a);
    for (int64_t q = q0; q < nq; q += 2 * kAhead * stride) {
        fetch_set(q + kAhead * stride, b);
        add_set(a);
        fetch_set(q + 2 * kAhead * stride, a);
        add_set(b);
    }
    __syncthreads();
    double *out = part_sums + (int64_t)blockIdx.x * K * M + f0;
    for (int e = threadIdx.x; e < K * kSlice; e += blockDim.x) {
        const int k = e / kSlice, j = e % kSlice;
        if (j < nf) {
            double s = 0.0;
            for (int w = 0; w < W; ++w) s = s + sums[((size_t)w * kSlice + j) * KS + k];
            out[(int64_t)k * M + j] = s;
        }
    }
    if (blockIdx.y == 0)
        for (int k = threadIdx.x; k < K; k += blockDim.x) {
            int32_t s = 0;
            for (int w = 0; w < W; ++w) s += cnts[(size_t)w * K + k];
            part_counts[(int64_t)k * gridDim.x + blockIdx.x] = s;
        }
}

}  // namespace

AccumPlan plan_accum(int64_t n, int M, int K)
{
    AccumPlan p{};
    p.path = kPathSplit;
    const int64_t nq = (n + kWave - 1) / kWave;
    int slice = 16, W = 0, slices = 0;
    for (;; slice /= 2) {
        W = (int)((size_t)kMaxLds / slab_bytes(K, slice));
        if (W > kAccWaves) W = kAccWaves;
        slices = (M + slice - 1) / slice;
        if (slice == 4) break;
        if (slice / 2 < M && W >= kAccMinWaves && slices * ((nq + W - 1) / W) >= kCUs) break;
    }
    while (W > 1 && W / 2 >= nq) W /= 2;
    p.lds_bytes = (size_t)W * slab_bytes(K, slice);
    // a workgroup for every compute unit, and no more rows of partials than that
    // takes (with two, M = 57, K = 32: 42.3 us, now 34.0 at n = 400,000)
    int64_t groups = kCUs / slices;
    if (groups > (nq + W - 1) / W) groups = (nq + W - 1) / W;
    p.waves = W;
    p.groups = groups < 1 ? 1 : (int)groups;
    p.accum = slice;
    return p;
}

hipError_t launch_accum(const StepArgs &a, const AccumPlan &plan, hipStream_t s)
{
    if (plan.waves < 1 || plan.groups < 1 || plan.groups > kCUs ||
        plan.lds_bytes > (size_t)kMaxLds || a.M < 1 || a.M > kMaxM || a.K < 1 || a.K > kMaxK)
        return hipErrorInvalidValue;
    if (plan.accum != 4 && plan.accum != 8 && plan.accum != 16) return hipErrorInvalidValue;
    const auto kern = plan.accum == 16  ? accum_labels_kernel<16>
                      : plan.accum == 8 ? accum_labels_kernel<8>
                                        : accum_labels_kernel<4>;
    const dim3 grid(plan.groups, (a.M + plan.accum - 1) / plan.accum);
    hipLaunchKernelGGL(kern, grid, dim3(plan.waves * kWave), plan.lds_bytes, s, a.X, a.n, a.M,
                       a.labels_in, a.K, a.part_sums, a.part_counts, a.ctl, a.fixed);
    return hipGetLastError();
}

}  // namespace lloyd
