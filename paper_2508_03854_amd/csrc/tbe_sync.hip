// Replica synchronisation of Algorithm 1 (weight sync and moment sync) for replicas that live on ONE device:
// every replica's buffer is replaced by the element-wise mean over the replicas.  Across devices this step is
// an all-reduce; that is outside this library.
#include <hip/hip_fp16.h>
#include <hip/hip_runtime.h>

#include "tbe_device.h"
#include "tbe_internal.h"

namespace tbe {

__device__ __forceinline__ float elem_to_float(float x) { return x; }
__device__ __forceinline__ float elem_to_float(__half x) { return __half2float(x); }
__device__ __forceinline__ void elem_from_float(float* p, float x) { *p = x; }
__device__ __forceinline__ void elem_from_float(__half* p, float x) { *p = __float2half_rn(x); }

struct ReplicaPtrs {
    void* p[kMaxReplicas];
};

__device__ __forceinline__ uint4 pack(const float (&x)[4]) {
    return make_uint4(__float_as_uint(x[0]), __float_as_uint(x[1]), __float_as_uint(x[2]), __float_as_uint(x[3]));
}
__device__ __forceinline__ uint4 pack(const float (&x)[8]) {   // binary16, to nearest even
    uint32_t w[4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
        w[i] = (uint32_t)__half_as_ushort(__float2half_rn(x[2 * i])) | (uint32_t)__half_as_ushort(__float2half_rn(x[2 * i + 1])) << 16;
    return make_uint4(w[0], w[1], w[2], w[3]);
}

// 16 bytes per thread and replica, or two such pieces: the sum runs over the replicas in index order, in fp32, and is divided by M
// (a true division, so the result is the correctly rounded quotient of the fp32 sum).
// Bound: the stream, read once and written once.  The means are written past the caches, and replicas that together are much more than
// the Infinity Cache holds (LARGE) read past them too, two pieces in flight; smaller ones find part of themselves there, and have the
// workgroups to fill the chip at once instead.  Plain accesses / LARGE / the other, us: 4 x 60 M fp32 (960 MB) 378 / 354 / 379; 8 x
// 10 M fp32 (320 MB) 105 / 113 / 94; 2 x 40 M fp32 (320) 109 / 111 / 105; 4 x 20 M binary16 (160) 48 / 55 / 46.
// Many replicas that all fit the Infinity Cache are written to it (STREAM off), where they are next read; of a few replicas it makes no
// difference.  The mean, and with a reader of all replicas behind it, us, STREAM off / on: 5 x 8 M fp32 (160 MB) 48 100 / 48 101; 6 x
// 4.2 M (100) 31 67 / 31 71; 8 x 4 M (128) 38 85 / 40 91; 8 x 6.2 M (200) 59 125 / 62 136; 8 x 10.6 M (340) 123 241 / 101 226; 16 x 4.2 M
// (270) 87 197 / 97 207; 16 x 6.2 M (400) 177 323 / 146 294; 12 x 10.4 M binary16 (250) 74 175 / 82 177; 7 x 11.2 M (157) 48 107 / 49 111.
constexpr size_t kLargeReplicas = (size_t)512 << 20;   // bytes of all of them
static bool stream_means(const int M, const size_t bytes) { return M <= 5 || bytes > (size_t)(M > 8 ? 288 : 256) << 20; }
template <typename WT, bool LARGE, bool STREAM>
__global__ __launch_bounds__(256) void replica_mean_kernel(const ReplicaPtrs r, const int M, const size_t nvec,
                                                           const size_t count) {
    constexpr int V = RowIO<WT>::kVec;
    constexpr int U = LARGE ? 2 : 1;
    using raw_t = typename RowIO<WT>::raw_t;
    const float fm = (float)M;
    const size_t stride = (size_t)gridDim.x * blockDim.x * U;
    for (size_t i0 = (size_t)blockIdx.x * blockDim.x * U + threadIdx.x; i0 < nvec; i0 += stride) {
        float sum[U][V];
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int v = 0; v < V; ++v) sum[u][v] = 0.f;
        for (int m = 0; m < M; ++m) {
            raw_t raw[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const size_t i = i0 + u * blockDim.x < nvec ? i0 + u * blockDim.x : nvec - 1;
                const WT* const src = static_cast<const WT*>(r.p[m]) + i * V;
                if (LARGE) raw[u] = __builtin_bit_cast(raw_t, nt_load16(src));
                else raw[u] = RowIO<WT>::load_raw(src);
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                float x[V];
                RowIO<WT>::unpack(raw[u], x);
#pragma unroll
                for (int v = 0; v < V; ++v) sum[u][v] += x[v];
            }
        }
        uint4 mean[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
#pragma unroll
            for (int v = 0; v < V; ++v) sum[u][v] /= fm;
            mean[u] = pack(sum[u]);
        }
        for (int m = 0; m < M; ++m)
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (i0 + u * blockDim.x < nvec) {
                    WT* const dst = static_cast<WT*>(r.p[m]) + (i0 + u * blockDim.x) * V;
                    if (STREAM) nt_store16(dst, mean[u]);
                    else *reinterpret_cast<uint4*>(dst) = mean[u];
                }
    }
    // the last count % V elements, one thread each
    const size_t tail0 = nvec * V;
    if (blockIdx.x == 0 && tail0 + threadIdx.x < count) {
        const size_t e = tail0 + threadIdx.x;
        float s = 0.f;
        for (int m = 0; m < M; ++m) s += elem_to_float(static_cast<const WT*>(r.p[m])[e]);
        s /= fm;
        for (int m = 0; m < M; ++m) elem_from_float(static_cast<WT*>(r.p[m]) + e, s);
    }
}

template <typename WT>
static void launch_mean(const ReplicaPtrs& r, int M, size_t count, hipStream_t s) {
    const size_t nvec = count / RowIO<WT>::kVec, bytes = (size_t)M * count * sizeof(WT);
    if (bytes > kLargeReplicas) {
        replica_mean_kernel<WT, true, true><<<256 * 8, 256, 0, s>>>(r, M, nvec, count);
    } else {
        const size_t need = nvec / 256 + 1;   // (at least one workgroup, for the last few elements)
        const unsigned grid = (unsigned)(need < 16384 ? need : 16384);
        if (stream_means(M, bytes)) replica_mean_kernel<WT, false, true><<<grid, 256, 0, s>>>(r, M, nvec, count);
        else replica_mean_kernel<WT, false, false><<<grid, 256, 0, s>>>(r, M, nvec, count);
    }
}

hipError_t launch_replica_mean(const tbe_handle* h, void* const* replicas, int M, size_t count, bool f32, hipStream_t s) {
    ReplicaPtrs r;
    for (int m = 0; m < kMaxReplicas; ++m) r.p[m] = m < M ? replicas[m] : nullptr;
    LaunchTimer tm(h, s, "replica_mean");
    if (f32) launch_mean<float>(r, M, count, s);
    else launch_mean<__half>(r, M, count, s);
    tm.done();
    return hipGetLastError();
}

}  // namespace tbe
