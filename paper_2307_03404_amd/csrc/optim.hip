// Mapping update: one sparse RMSProp step over the vertex records (Sec. 5.4
// names RMSProp for the mapping).  A record is touched when any of its
// gradient entries is non-zero; only touched records change (values and
// running averages), so vertices no ray reached keep their state, as in the
// Plenoxel optimiser this method builds on.  The gradient is zeroed after it
// is read, so one call ends a mapping iteration.
//
// A group of L lanes per record (L = 8, 4, 1 for records of 7, 4, 1 float4:
// SH degree 2, 1, 0), lane q < Q holding float4 q of it: the record's
// "touched" bit comes from a wave ballot over its group, and every load and
// store is a contiguous run.  Bound by HBM: at degree 2, 112 B read per
// record, plus 112 B written (gradient zeroed) and 2 x 224 B
// read-modify-write (values, averages) per touched record.
#include "internal.hpp"

namespace pxm {

template <int Q, int L>
__global__ void __launch_bounds__(256) k_rmsprop(int64_t n, float4* __restrict__ data,
                                                 float4* __restrict__ grad,
                                                 float4* __restrict__ avg, float lr_d, float lr_sh,
                                                 float alpha, float eps) {
    static_assert(Q <= L && (L & (L - 1)) == 0 && L <= 8, "a record's lanes form one ballot group");
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t rec = t / L;
    const int q = (int)(t % L);
    const bool act = rec < n && q < Q;
    const int64_t i = rec * Q + q;
    const float4 g = act ? grad[i] : make_float4(0.f, 0.f, 0.f, 0.f);
    const bool nz = g.x != 0.f || g.y != 0.f || g.z != 0.f || g.w != 0.f;
    const unsigned long long m = __ballot(nz);
    const bool touched = ((m >> (lane_id() & ~(L - 1))) & ((1ull << L) - 1ull)) != 0ull;
    if (!act || !touched) return;
    float4 v = avg[i];
    float4 x = data[i];
    const float a1 = 1.f - alpha;
    v.x = alpha * v.x + a1 * g.x * g.x;
    v.y = alpha * v.y + a1 * g.y * g.y;
    v.z = alpha * v.z + a1 * g.z * g.z;
    v.w = alpha * v.w + a1 * g.w * g.w;
    x.x -= (q == 0 ? lr_d : lr_sh) * g.x / (sqrtf(v.x) + eps);   // entry 0 is the density
    x.y -= lr_sh * g.y / (sqrtf(v.y) + eps);
    x.z -= lr_sh * g.z / (sqrtf(v.z) + eps);
    x.w -= lr_sh * g.w / (sqrtf(v.w) + eps);
    avg[i] = v;
    data[i] = x;
    grad[i] = make_float4(0.f, 0.f, 0.f, 0.f);
}

template <int Q, int L>
static void rmsprop_go(int64_t n, float* data, float* grad, float* avg, float lr_d, float lr_sh,
                       float alpha, float eps, hipStream_t st) {
    const int64_t threads = n * L;
    const unsigned blocks = (unsigned)((threads + 255) / 256);
    hipLaunchKernelGGL((k_rmsprop<Q, L>), dim3(blocks), dim3(256), 0, st, n,
                       reinterpret_cast<float4*>(data), reinterpret_cast<float4*>(grad),
                       reinterpret_cast<float4*>(avg), lr_d, lr_sh, alpha, eps);
}

hipError_t launch_rmsprop(int64_t n, int deg, float* data, float* grad, float* avg, float lr_d,
                          float lr_sh, float alpha, float eps, hipStream_t st) {
    if (deg == 0) rmsprop_go<1, 1>(n, data, grad, avg, lr_d, lr_sh, alpha, eps, st);
    else if (deg == 1) rmsprop_go<4, 4>(n, data, grad, avg, lr_d, lr_sh, alpha, eps, st);
    else rmsprop_go<7, 8>(n, data, grad, avg, lr_d, lr_sh, alpha, eps, st);
    return hipGetLastError();
}

// Ray batch of a mapping iteration.  Up to GATHER_ONE rays in one launch: workgroup 0
// counts the valid target depths and finds the frames' offsets (the indices ascend, so
// frame f starts at the first index that is not below its keyframe offset); the others
// copy a ray per lane.  13 launches of elementwise and index kernels and a host
// synchronisation before.  That count is one workgroup's chain of dependent loads and
// grows with the batch; larger batches count where they copy, with one atomic per
// workgroup into frame_offsets[0], which a launch before clears and one after reads.
// us of one launch and of three, rays of 6.5 M: 2,048 6.8 and 12.5; 8,192 8.3 and 12.9;
// 16,384 22 and 13; 65,536 87 and 14; 1,048,576 642 and 35.
constexpr int COUNT_THREADS = 1024;
constexpr int64_t GATHER_ONE = 8192;

struct GatherIO {
    const int64_t* index;
    int64_t n, n_kf;
    int F;
    const int32_t* kf_off;
    const int32_t* kf_pix;
    const float* kf_rgb;
    const float* kf_depth;
    int32_t* pix;
    float* rgb;
    float* depth;
    int32_t* off;
    float* weight;
};

// Keyframe ray of ray r of the batch, inside the keyframes whatever the index says.
__device__ __forceinline__ int64_t gather_index(const GatherIO& io, int64_t r) {
    const int64_t i = io.index[r];
    return i < 0 ? 0 : i >= io.n_kf ? io.n_kf - 1 : i;
}

__device__ __forceinline__ bool gather_ray(const GatherIO& io, int64_t r) {
    const int64_t i = gather_index(io, r);
    // all loads before the first store: the arrays are not known to be apart
    const int32_t u = io.kf_pix[2 * i], v = io.kf_pix[2 * i + 1];
    const float c0 = io.kf_rgb[3 * i], c1 = io.kf_rgb[3 * i + 1], c2 = io.kf_rgb[3 * i + 2], d = io.kf_depth[i];
    io.pix[2 * r] = u;
    io.pix[2 * r + 1] = v;
    io.rgb[3 * r] = c0;
    io.rgb[3 * r + 1] = c1;
    io.rgb[3 * r + 2] = c2;
    io.depth[r] = d;
    return isfinite(d) && d > 0.f;
}

// Sum over the workgroup, returned to all of its threads.
__device__ __forceinline__ long long block_count(long long count) {
    __shared__ long long s_count[COUNT_THREADS / WAVE];
    count = wave_sum(count);
    if (lane_id() == 0) s_count[threadIdx.x / WAVE] = count;
    __syncthreads();
    count = 0;
    for (int w = 0; w < COUNT_THREADS / WAVE; ++w) count += s_count[w];
    return count;
}

// One workgroup: the frames' offsets and weights of a batch with `count` valid depths.
__device__ __forceinline__ void gather_frames(const GatherIO& io, long long count) {
    const float m = 1.0f / (float)(count < 1 ? 1 : count);
    for (int f = threadIdx.x; f <= io.F; f += COUNT_THREADS) {
        int64_t lo = 0, hi = io.n;                          // first r with an index >= kf_off[f]
        while (lo < hi) {
            const int64_t mid = (lo + hi) / 2;
            if (gather_index(io, mid) < io.kf_off[f]) lo = mid + 1; else hi = mid;
        }
        io.off[f] = (int32_t)(f == 0 ? 0 : f == io.F ? io.n : lo);
        if (f < io.F) io.weight[f] = m;
    }
}

__global__ void __launch_bounds__(COUNT_THREADS) k_gather_rays(GatherIO io) {
    if (blockIdx.x > 0) {
        const int64_t r = (int64_t)(blockIdx.x - 1) * COUNT_THREADS + threadIdx.x;
        if (r < io.n) gather_ray(io, r);
        return;
    }
    long long count = 0;
    for (int64_t r = threadIdx.x; r < io.n; r += COUNT_THREADS) {
        const float d = io.kf_depth[gather_index(io, r)];
        count += isfinite(d) && d > 0.f;
    }
    gather_frames(io, block_count(count));
}

__global__ void k_gather_clear(int32_t* count) { *count = 0; }

__global__ void __launch_bounds__(COUNT_THREADS) k_gather_copy(GatherIO io) {
    const int64_t r = (int64_t)blockIdx.x * COUNT_THREADS + threadIdx.x;
    const long long count = block_count(r < io.n && gather_ray(io, r));
    if (threadIdx.x == 0 && count > 0) atomicAdd(io.off, (int32_t)count);
}

__global__ void __launch_bounds__(COUNT_THREADS) k_gather_frames(GatherIO io) {
    const int32_t count = *io.off;
    __syncthreads();                                        // all have read it: it becomes the first offset
    gather_frames(io, count);
}

hipError_t launch_gather_rays(int64_t n, const int64_t* index, int64_t n_kf, int F, const int32_t* kf_off, const int32_t* kf_pix,
                              const float* kf_rgb, const float* kf_depth, int32_t* pix, float* rgb, float* depth,
                              int32_t* off, float* weight, hipStream_t st) {
    const GatherIO io = {index, n, n_kf, F, kf_off, kf_pix, kf_rgb, kf_depth, pix, rgb, depth, off, weight};
    const unsigned blocks = (unsigned)((n + COUNT_THREADS - 1) / COUNT_THREADS);
    if (n <= GATHER_ONE) {
        hipLaunchKernelGGL(k_gather_rays, dim3(1 + blocks), dim3(COUNT_THREADS), 0, st, io);
        return hipGetLastError();
    }
    hipLaunchKernelGGL(k_gather_clear, dim3(1), dim3(1), 0, st, off);
    hipLaunchKernelGGL(k_gather_copy, dim3(blocks), dim3(COUNT_THREADS), 0, st, io);
    hipLaunchKernelGGL(k_gather_frames, dim3(1), dim3(COUNT_THREADS), 0, st, io);
    return hipGetLastError();
}

}  // namespace pxm
