// The sums of Eq. (1) from labels, for shapes whose K x M fp64 slab does not fit
// in LDS beside the distance kernel's state: the second of the two launches
// that such an iteration (or kmeans_update) makes in place of the fused one.
//
// What bounds it: K x M = 16384 sums take 128 KB as one slab, so a workgroup
// with all features holds one slab that its waves share in turns, and 256
// workgroups write 34 MB of partials that the centres launch reads again (31 us
// at K = 1024, M = 16). Instead a workgroup takes four features (16 bytes of a
// row): a wave's private slab is then K x 4 sums (32 KB at K = 1024), no wave
// waits for another, and the M / 4 slices share the chip with G row groups, so
// that G x M / 4 workgroups fill it while only G rows of partials are written
// (64 at M = 16: 8.4 MB). X is read once in all, in 16-byte pieces of the same
// cache lines by the M / 4 slices.
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
constexpr int kSlice = 4;            // features per workgroup
constexpr int kAccWaves = 8;         // waves per workgroup, at most

// row stride of a feature of the slab: odd, so that the features of a cluster
// start on different banks when the slabs are added
__host__ __device__ inline int slab_row(int K) { return K | 1; }

__host__ __device__ inline size_t slab_bytes(int K)
{
    return (size_t)kSlice * slab_row(K) * 8 + (size_t)((K + 1) / 2 * 2) * 4;
}

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
        f4u x;
        int lab;
    };
    // (a tile past the end reads the last object and adds nothing)
    auto fetch = [&](int64_t q, Tile &t) {
        const int64_t i = q * kWave + lane;
        const int64_t r = i < n ? i : n - 1;
        if (whole) {
            t.x = *reinterpret_cast<const f4u *>(X + r * M + f0);
        } else if (M >= kSlice) {
            // the row's last features, moved down to the slice's
            const f4u v = *reinterpret_cast<const f4u *>(X + r * M + M - kSlice);
            t.x[0] = nf == 3 ? v[1] : nf == 2 ? v[2] : v[3];
            t.x[1] = nf == 3 ? v[2] : v[3];
            t.x[2] = v[3];
            t.x[3] = 0.f;
        } else {
#pragma unroll
            for (int j = 0; j < kSlice; ++j) t.x[j] = X[r * M + (j < nf ? j : 0)];
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
    // eight tiles in flight while the eight before them are added
    constexpr int kAhead = 8;
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
    int W = (int)((size_t)kMaxLds / slab_bytes(K));
    if (W > kAccWaves) W = kAccWaves;
    const int64_t nq = (n + kWave - 1) / kWave;
    while (W > 1 && W / 2 >= nq) W /= 2;
    p.lds_bytes = (size_t)W * slab_bytes(K);
    // enough workgroups for the compute units (two each where two fit), and
    // no more rows of partials than that takes
    const int slices = (M + kSlice - 1) / kSlice;
    int64_t groups = (p.lds_bytes <= (size_t)kMaxLds / 2 ? 2 * kCUs : kCUs) / slices;
    if (groups > kCUs) groups = kCUs;
    if (groups > (nq + W - 1) / W) groups = (nq + W - 1) / W;
    p.waves = W;
    p.groups = groups < 1 ? 1 : (int)groups;
    p.accum = slices;
    return p;
}

hipError_t launch_accum(const StepArgs &a, const AccumPlan &plan, hipStream_t s)
{
    if (plan.waves < 1 || plan.groups < 1 || plan.groups > kCUs ||
        plan.lds_bytes > (size_t)kMaxLds || a.M < 1 || a.M > kMaxM || a.K < 1 || a.K > kMaxK)
        return hipErrorInvalidValue;
    hipLaunchKernelGGL(accum_labels_kernel, dim3(plan.groups, plan.accum), dim3(plan.waves * kWave),
                       plan.lds_bytes, s, a.X, a.n, a.M, a.labels_in, a.K, a.part_sums,
                       a.part_counts, a.ctl, a.fixed);
    return hipGetLastError();
}

}  // namespace lloyd
