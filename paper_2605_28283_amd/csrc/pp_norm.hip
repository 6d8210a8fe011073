// Residual add + RMSNorm between stacked FFN layers (pre-norm wiring):
//   x_out = x + y,  u = bf16(x_out / sqrt(mean(x_out^2) + eps))  (norm weight 1).
// Not part of the paper's method; it chains the layers of the stacked decode
// workload.  One workgroup of 256 threads per row.  The sum of squares is
// taken in one fixed order (per-thread partials over its float4 columns in
// ascending order, then the wavefront scan, then wavefronts in order), so a
// row's result does not depend on T.
#include "pp_internal.h"

namespace pp {
namespace {

constexpr int kNormThreads = 256;

__device__ __forceinline__ float4 add4(float4 v, const float4 w) {
    v.x += w.x;
    v.y += w.y;
    v.z += w.z;
    v.w += w.w;
    return v;
}

__device__ __forceinline__ float add_squares(float ss, const float4 v) {
    ss += v.x * v.x;
    ss += v.y * v.y;
    ss += v.z * v.z;
    ss += v.w * v.w;
    return ss;
}

// 1 / rms of the row from the threads' partial sums.
__device__ __forceinline__ float row_scale(float ss, int d, float eps, float *wsum) {
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const float ws = lane_value(wave_scan_f32(ss), 63);
    if (lane == 0) wsum[wv] = ws;
    __syncthreads();
    float tot = wsum[0];
#pragma unroll
    for (int w = 1; w < kNormThreads / 64; ++w) tot += wsum[w];
    return 1.0f / sqrtf(tot / (float)d + eps);
}

__device__ __forceinline__ uint2 scaled_bf16(const float4 v, float r) {
    return make_uint2((uint32_t)f32_to_bf16(v.x * r) | ((uint32_t)f32_to_bf16(v.y * r) << 16),
                      (uint32_t)f32_to_bf16(v.z * r) | ((uint32_t)f32_to_bf16(v.w * r) << 16));
}

// N: float4 columns a thread holds in registers (rows of up to 1024 N values),
// or 0 for any row, read column by column and again for the scaling.  A
// decode batch's rows are one memory round trip: with N every load of a row is
// issued before its first store, which the compiler cannot do by itself as
// x_out may be x or y (16 x 4096: 3.7 us column by column, 2.6 us).  Columns
// past the row read its last one, whose value they do not use.
template <int N>
__global__ __launch_bounds__(kNormThreads) void residual_rmsnorm_k(const float *x, const float *y,
                                                                   float *x_out, int d, float eps,
                                                                   uint16_t *__restrict__ u) {
    __shared__ float wsum[kNormThreads / 64];
    const int t = blockIdx.x, tid = threadIdx.x;
    const size_t row = (size_t)t * d;
    const int n4 = d / 4;
    const float4 *x4 = reinterpret_cast<const float4 *>(x + row);
    const float4 *y4 = reinterpret_cast<const float4 *>(y + row);
    float4 *o4 = reinterpret_cast<float4 *>(x_out + row);
    uint2 *u2 = reinterpret_cast<uint2 *>(u + row);
    float ss = 0.0f;
    if constexpr (N > 0) {
        float4 v[N], w[N];
#pragma unroll
        for (int i = 0; i < N; ++i) v[i] = x4[min(tid + i * kNormThreads, n4 - 1)];
        if (y) {
#pragma unroll
            for (int i = 0; i < N; ++i) w[i] = y4[min(tid + i * kNormThreads, n4 - 1)];
#pragma unroll
            for (int i = 0; i < N; ++i) v[i] = add4(v[i], w[i]);
        }
#pragma unroll
        for (int i = 0; i < N; ++i)
            if (tid + i * kNormThreads < n4) {
                o4[tid + i * kNormThreads] = v[i];
                ss = add_squares(ss, v[i]);
            }
        if (!u) return;
        const float r = row_scale(ss, d, eps, wsum);
#pragma unroll
        for (int i = 0; i < N; ++i)
            if (tid + i * kNormThreads < n4) u2[tid + i * kNormThreads] = scaled_bf16(v[i], r);
    } else {
        for (int c = tid; c < n4; c += kNormThreads) {
            const float4 v = y ? add4(x4[c], y4[c]) : x4[c];
            o4[c] = v;
            ss = add_squares(ss, v);
        }
        if (!u) return;
        const float r = row_scale(ss, d, eps, wsum);
        // each thread rereads the columns it wrote itself
        for (int c = tid; c < n4; c += kNormThreads) u2[c] = scaled_bf16(o4[c], r);
    }
}

}  // namespace
}  // namespace pp

extern "C" pp_status prunepath_residual_rmsnorm(const float *x, const float *y, float *x_out,
                                                int32_t T, int32_t d, float eps, uint16_t *u,
                                                void *hip_stream) {
    if (!x || !x_out) return PP_EINVAL;
    if (T < 1 || T > 65536 || d < 4 || d % 4 != 0 || d > (1 << 20)) return PP_EINVAL;
    if (u && !(eps >= 0.0f)) return PP_EINVAL;  // also rejects NaN
    // rows are moved as float4 (x, y, x_out) and as 4 x bf16 (u)
    if (((uintptr_t)x | (uintptr_t)y | (uintptr_t)x_out) % 16 != 0 || (uintptr_t)u % 8 != 0)
        return PP_EINVAL;
    // every element of x and y is read by the thread that writes that element
    // of x_out, so x, y and x_out may be the same array
    hipStream_t s = static_cast<hipStream_t>(hip_stream);
    // the registers of 4 or 8 columns a thread, or memory past them
    const int cols = (d / 4 + pp::kNormThreads - 1) / pp::kNormThreads;
    if (cols <= 4)
        hipLaunchKernelGGL(pp::residual_rmsnorm_k<4>, dim3(T), dim3(pp::kNormThreads), 0, s, x, y,
                           x_out, d, eps, u);
    else if (cols <= 8)
        hipLaunchKernelGGL(pp::residual_rmsnorm_k<8>, dim3(T), dim3(pp::kNormThreads), 0, s, x, y,
                           x_out, d, eps, u);
    else
        hipLaunchKernelGGL(pp::residual_rmsnorm_k<0>, dim3(T), dim3(pp::kNormThreads), 0, s, x, y,
                           x_out, d, eps, u);
    return hipGetLastError() == hipSuccess ? PP_OK : PP_EHIP;
}
