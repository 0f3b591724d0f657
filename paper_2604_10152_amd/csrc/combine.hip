// Gate-weighted mix of the selected experts' outputs (SpecMoE Sec. 2.1, Fig. 1b) and the
// RMSNorm helper of the multi-layer benchmark configuration.
//
// combine is a gather, not a scatter: one workgroup per token reads its k expert rows through
// row_of and accumulates them in fp32 in slot order, so the result is deterministic and needs
// no atomics.  Both kernels are single HBM passes with 16-byte accesses.
#include "common.h"

namespace specmoe {
namespace {

constexpr int kRowThreads = 256;

template <typename T> struct RowVec;
template <> struct RowVec<float> {
    static constexpr int N = 4;
    __device__ static void widen(const U128& v, float (&o)[4]) {
#pragma unroll
        for (int i = 0; i < 4; ++i) o[i] = __uint_as_float(v[i]);
    }
    __device__ static void load(const float* p, float (&o)[4]) {
        widen(*reinterpret_cast<const U128*>(p), o);
    }
    __device__ static void store(float* p, const float (&o)[4]) {
        *reinterpret_cast<float4*>(p) = make_float4(o[0], o[1], o[2], o[3]);
    }
};
template <> struct RowVec<bf16_t> {
    static constexpr int N = 8;
    __device__ static void widen(const U128& v, float (&o)[8]) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            o[2 * i] = bf16_bits_to_float(v[i] & 0xffffu);
            o[2 * i + 1] = bf16_bits_to_float(v[i] >> 16);
        }
    }
    __device__ static void load(const bf16_t* p, float (&o)[8]) {
        widen(*reinterpret_cast<const U128*>(p), o);
    }
    __device__ static void store(bf16_t* p, const float (&o)[8]) {
        U128 v;
        v.x = pack_bf16x2(o[0], o[1]); v.y = pack_bf16x2(o[2], o[3]);
        v.z = pack_bf16x2(o[4], o[5]); v.w = pack_bf16x2(o[6], o[7]);
        *reinterpret_cast<U128*>(p) = v;
    }
};

template <typename T>
__global__ __launch_bounds__(kRowThreads) void combine_kernel(
    const T* __restrict__ y_perm, const int32_t* __restrict__ row_of,
    const float* __restrict__ w, const T* residual, int d, int k, int vec_ok, T* out) {
    const int t = blockIdx.x;
    constexpr int V = RowVec<T>::N;
    if (vec_ok) {                            // host checked: d % V == 0, 16-byte aligned bases
        for (int j = threadIdx.x * V; j < d; j += kRowThreads * V) {
            float acc[V];
            if (residual) RowVec<T>::load(residual + (size_t)t * d + j, acc);
            else {
#pragma unroll
                for (int i = 0; i < V; ++i) acc[i] = 0.f;
            }
            for (int s = 0; s < k; ++s) {
                const int r = row_of[(size_t)t * k + s];
                const float ws = w[(size_t)t * k + s];
                float v[V];
                RowVec<T>::load(y_perm + (size_t)r * d + j, v);
#pragma unroll
                for (int i = 0; i < V; ++i) acc[i] = fmaf(ws, v[i], acc[i]);
            }
            RowVec<T>::store(out + (size_t)t * d + j, acc);
        }
    } else {
        for (int j = threadIdx.x; j < d; j += kRowThreads) {
            float acc = residual ? load_as_float(residual + (size_t)t * d + j) : 0.f;
            for (int s = 0; s < k; ++s) {
                const int r = row_of[(size_t)t * k + s];
                acc = fmaf(w[(size_t)t * k + s], load_as_float(y_perm + (size_t)r * d + j), acc);
            }
            store_from_float(out + (size_t)t * d + j, acc);
        }
    }
}

// One workgroup per row.  NV > 0: 16-byte accesses, NV pieces per thread stay in registers between
// the sum of squares and the scaling, so x is read once.  Thread t sums the elements t, t + 256, ...
// in order in both forms (a piece's neighbours come through LDS), so the result does not depend on
// the alignment of the buffers.  NV = 0: any length and alignment, two passes of single elements; up
// to 256 elements that is one load per thread already (4096 x 64 bf16 3.4 us, a fifth more through LDS).
// 80 x 4096 bf16: 4.9 us in the general form, 2.8 in this one; 2048 x 4096 9.9 and 7.1.
template <typename T, int NV>
__global__ __launch_bounds__(kRowThreads) void rmsnorm_kernel(
    const T* __restrict__ x, const T* __restrict__ gain, int d, float eps, T* __restrict__ out) {
    __shared__ float part[kRowThreads / kWave];
    constexpr int V = RowVec<T>::N, N = NV > 0 ? NV : 1;
    const int t = blockIdx.x;
    const T* xt = x + (size_t)t * d;
    U128 raw[N];
    float ss = 0.f;
    if constexpr (NV > 0) {
        __shared__ __align__(16) T row[N * kRowThreads * V];
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const int p = i * kRowThreads + threadIdx.x;
            raw[i] = U128{0, 0, 0, 0};               // beyond the row: adds nothing to the sum
            if (p * V < d) raw[i] = *reinterpret_cast<const U128*>(xt + p * V);
        }
#pragma unroll
        for (int i = 0; i < N; ++i)
            *reinterpret_cast<U128*>(row + (i * kRowThreads + threadIdx.x) * V) = raw[i];
        __syncthreads();
#pragma unroll
        for (int i = 0; i < N * V; ++i) {
            const float e = load_as_float(row + i * kRowThreads + threadIdx.x);
            ss = fmaf(e, e, ss);
        }
    } else {
        for (int j = threadIdx.x; j < d; j += kRowThreads) {
            float e = load_as_float(xt + j);
            ss = fmaf(e, e, ss);
        }
    }
    ss = wave_sum(ss);
    if (threadIdx.x % kWave == 0) part[threadIdx.x / kWave] = ss;
    __syncthreads();
    float tot = 0.f;
#pragma unroll
    for (int i = 0; i < kRowThreads / kWave; ++i) tot += part[i];
    const float scale = 1.0f / sqrtf(tot / (float)d + eps);
    if constexpr (NV > 0) {
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const int j = (i * kRowThreads + threadIdx.x) * V;
            if (j < d) {
                float v[V], g[V], o[V];
                RowVec<T>::widen(raw[i], v);
                RowVec<T>::load(gain + j, g);
#pragma unroll
                for (int q = 0; q < V; ++q) o[q] = v[q] * scale * g[q];
                RowVec<T>::store(out + (size_t)t * d + j, o);
            }
        }
    } else {
        for (int j = threadIdx.x; j < d; j += kRowThreads)
            store_from_float(out + (size_t)t * d + j,
                             load_as_float(xt + j) * scale * load_as_float(gain + j));
    }
}

template <typename T>
void launch_rmsnorm_typed(const T* x, const T* gain, int T_, int d, float eps, T* out,
                          hipStream_t s) {
    constexpr int V = RowVec<T>::N;
    const bool vec = d > kRowThreads && d % V == 0 &&
                     (((uintptr_t)x | (uintptr_t)gain | (uintptr_t)out) & 15u) == 0;
    const int pieces = (d + kRowThreads * V - 1) / (kRowThreads * V);      // per thread
    if (vec && pieces <= 1)
        hipLaunchKernelGGL((rmsnorm_kernel<T, 1>), dim3(T_), dim3(kRowThreads), 0, s, x, gain, d, eps, out);
    else if (vec && pieces <= 2)
        hipLaunchKernelGGL((rmsnorm_kernel<T, 2>), dim3(T_), dim3(kRowThreads), 0, s, x, gain, d, eps, out);
    else if (vec && pieces <= 4)
        hipLaunchKernelGGL((rmsnorm_kernel<T, 4>), dim3(T_), dim3(kRowThreads), 0, s, x, gain, d, eps, out);
    else
        hipLaunchKernelGGL((rmsnorm_kernel<T, 0>), dim3(T_), dim3(kRowThreads), 0, s, x, gain, d, eps, out);
}

}  // namespace

hipError_t launch_combine(const void* y_perm, const int32_t* row_of, const float* w,
                          const void* residual, int T, int d, int k, int dtype, void* out,
                          hipStream_t s) {
    if (T == 0 || d == 0) return hipSuccess;
    const bool aligned = (((uintptr_t)y_perm | (uintptr_t)residual | (uintptr_t)out) & 15u) == 0;
    if (dtype == 0)
        hipLaunchKernelGGL(combine_kernel<float>, dim3(T), dim3(kRowThreads), 0, s,
                           (const float*)y_perm, row_of, w, (const float*)residual, d, k,
                           (int)(aligned && d % 4 == 0), (float*)out);
    else
        hipLaunchKernelGGL(combine_kernel<bf16_t>, dim3(T), dim3(kRowThreads), 0, s,
                           (const bf16_t*)y_perm, row_of, w, (const bf16_t*)residual, d, k,
                           (int)(aligned && d % 8 == 0), (bf16_t*)out);
    return hipGetLastError();
}

hipError_t launch_rmsnorm(const void* x, const void* gain, int T, int d, float eps, int dtype,
                          void* out, hipStream_t s) {
    if (T == 0 || d == 0) return hipSuccess;
    if (dtype == 0)
        launch_rmsnorm_typed((const float*)x, (const float*)gain, T, d, eps, (float*)out, s);
    else
        launch_rmsnorm_typed((const bf16_t*)x, (const bf16_t*)gain, T, d, eps, (bf16_t*)out, s);
    return hipGetLastError();
}

}  // namespace specmoe
