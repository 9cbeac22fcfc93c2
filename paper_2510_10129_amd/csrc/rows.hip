// Row-wise HBM-bound kernels: gather + RMSNorm of the selected hidden rows,
// RMSNorm of the fp32 residual stream, and the rotary table.
#include "cc_internal.h"
#include "launch_plan.h"

__device__ __forceinline__ float wave_sum(float v) {
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
    return v;
}

// Sum over the WPR waves of a row (1, 2 or 4; a workgroup is four waves, and all of them come here).
template <int WPR>
__device__ __forceinline__ float row_sum(float v) {
    v = wave_sum(v);
    if constexpr (WPR > 1) {
        __shared__ float part[4];
        const int wave = threadIdx.x >> 6;
        if ((threadIdx.x & 63) == 0) part[wave] = v;
        __syncthreads();
        v = WPR == 4 ? (part[0] + part[1]) + (part[2] + part[3]) : part[wave & 2] + part[wave | 1];
    }
    return v;
}

// WPR waves per recomputed token, the whole row held in registers between the
// sum of squares and the scaled write (one pass over HBM): lane L of them owns the
// 16-byte chunks L, L + 64 WPR, ... of row gather_idx[i], so every load and store of a
// wave covers 1 KiB of contiguous row.  NCH = chunks per lane (d <= 512*NCH*WPR).
// Several waves a row hold the row and the weights' chunks in flight together, and a lane's share fits the
// registers of full occupancy; how many, by cc_norm_waves.
template <int NCH, int WPR>
__global__ __launch_bounds__(256) void gather_rmsnorm_kernel(
    const bf16_t* __restrict__ hidden, const int32_t* __restrict__ gather_idx, int M, int d,
    const bf16_t* __restrict__ w, float eps, bf16_t* __restrict__ xn) {
    const int lane = threadIdx.x % (64 * WPR);
    const int row_i = blockIdx.x * (4 / WPR) + threadIdx.x / (64 * WPR), i = min(row_i, M - 1);
    const int64_t src = gather_idx ? (int64_t)gather_idx[i] : (int64_t)i;
    const bf16x8* row = reinterpret_cast<const bf16x8*>(hidden + src * d);
    const bf16x8* wv = reinterpret_cast<const bf16x8*>(w);
    bf16x8* dst = reinterpret_cast<bf16x8*>(xn + (int64_t)i * d);
    const int nchunk = d >> 3;
    constexpr int ST = 64 * WPR;
    bf16x8 v[NCH], g[NCH];
    float ss = 0.0f;
#pragma unroll
    for (int c = 0; c < NCH; ++c)
        if (lane + ST * c < nchunk) v[c] = __builtin_nontemporal_load(row + lane + ST * c);
    if constexpr (WPR > 1) {
#pragma unroll
        for (int c = 0; c < NCH; ++c)
            if (lane + ST * c < nchunk) g[c] = wv[lane + ST * c];
    }
#pragma unroll
    for (int c = 0; c < NCH; ++c)
        if (lane + ST * c < nchunk) {
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                float f = (float)v[c][u];
                ss += f * f;
            }
        }
    const float r = 1.0f / sqrtf(row_sum<WPR>(ss) / (float)d + eps);
    if (row_i >= M) return;                       // repeats the last row
#pragma unroll
    for (int c = 0; c < NCH; ++c)
        if (lane + ST * c < nchunk) {
            bf16x8 o;
            if constexpr (WPR == 1) g[c] = wv[lane + ST * c];
#pragma unroll
            for (int u = 0; u < 8; ++u) o[u] = (bf16_t)((float)v[c][u] * r * (float)g[c][u]);
            dst[lane + ST * c] = o;
        }
}

void cc_launch_gather_rmsnorm(const bf16_t* hidden, const int32_t* gather_idx, int M, int d,
                              const bf16_t* w, float eps, bf16_t* xn, hipStream_t s) {
    if (M <= 0) return;
    const int waves = cc_norm_waves(cc_device_cus(), M, d, 2);
    dim3 grid(((int64_t)M * waves + 3) / 4), block(256);
#define CC_NORM(NCH, WPR) hipLaunchKernelGGL((gather_rmsnorm_kernel<NCH, WPR>), grid, block, 0, s, hidden, gather_idx, M, d, w, eps, xn)
    if (waves == 1) {                                // d <= 4096
        if (d <= 1024) CC_NORM(2, 1);
        else if (d <= 2048) CC_NORM(4, 1);
        else CC_NORM(8, 1);
    } else if (waves == 2) {                         // d <= 8192
        CC_NORM(8, 2);
    } else {
        if (d <= 4096) CC_NORM(2, 4);
        else if (d <= 8192) CC_NORM(4, 4);
        else CC_NORM(8, 4);
    }
#undef CC_NORM
}

// RMSNorm of the fp32 residual rows y [M, d] -> bf16, same scheme (lane owns
// 16-byte chunks of 4 floats; NCH chunks per lane, d <= 256*NCH*WPR).
template <int NCH, int WPR>
__global__ __launch_bounds__(256) void rmsnorm_f32_kernel(const float* __restrict__ y, int M, int d,
                                                          const bf16_t* __restrict__ w, float eps,
                                                          bf16_t* __restrict__ out) {
    const int lane = threadIdx.x % (64 * WPR);
    const int row_i = blockIdx.x * (4 / WPR) + threadIdx.x / (64 * WPR), i = min(row_i, M - 1);
    const f32x4* row = reinterpret_cast<const f32x4*>(y + (int64_t)i * d);
    const bf16x4* wv = reinterpret_cast<const bf16x4*>(w);
    bf16x4* dst = reinterpret_cast<bf16x4*>(out + (int64_t)i * d);
    const int nchunk = d >> 2;
    constexpr int ST = 64 * WPR;
    f32x4 v[NCH];
    bf16x4 g[NCH];
    float ss = 0.0f;
#pragma unroll
    for (int c = 0; c < NCH; ++c)
        if (lane + ST * c < nchunk) v[c] = row[lane + ST * c];
    if constexpr (WPR > 1) {
#pragma unroll
        for (int c = 0; c < NCH; ++c)
            if (lane + ST * c < nchunk) g[c] = wv[lane + ST * c];
    }
#pragma unroll
    for (int c = 0; c < NCH; ++c)
        if (lane + ST * c < nchunk) ss += v[c][0] * v[c][0] + v[c][1] * v[c][1] + v[c][2] * v[c][2] + v[c][3] * v[c][3];
    const float r = 1.0f / sqrtf(row_sum<WPR>(ss) / (float)d + eps);
    if (row_i >= M) return;                       // repeats the last row
#pragma unroll
    for (int c = 0; c < NCH; ++c)
        if (lane + ST * c < nchunk) {
            bf16x4 o;
            if constexpr (WPR == 1) g[c] = wv[lane + ST * c];
#pragma unroll
            for (int u = 0; u < 4; ++u) o[u] = (bf16_t)(v[c][u] * r * (float)g[c][u]);
            dst[lane + ST * c] = o;
        }
}

void cc_launch_rmsnorm_f32(const float* y, int M, int d, const bf16_t* w, float eps, bf16_t* out,
                           hipStream_t s) {
    if (M <= 0) return;
    const int waves = cc_norm_waves(cc_device_cus(), M, d, 4);
    dim3 grid(((int64_t)M * waves + 3) / 4), block(256);
#define CC_NORM(NCH, WPR) hipLaunchKernelGGL((rmsnorm_f32_kernel<NCH, WPR>), grid, block, 0, s, y, M, d, w, eps, out)
    if (waves == 1) {                                // d <= 1024
        if (d <= 512) CC_NORM(2, 1);
        else CC_NORM(4, 1);
    } else {
        if (d <= 4096) CC_NORM(4, 4);
        else if (d <= 8192) CC_NORM(8, 4);
        else CC_NORM(16, 4);
    }
#undef CC_NORM
}

// Rotary table: entry (p, j) = (cos, sin) of p * base^(-2j/d_h), evaluated in
// fp64 and stored as fp32.
__global__ void rope_table_kernel(float2* __restrict__ table, int n_pos, int half, double log2_base) {
    int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= (int64_t)n_pos * half) return;
    int p = (int)(e / half), j = (int)(e % half);
    double inv = exp2(-(double)j / (double)half * log2_base);   // base^(-2j/d_h), d_h = 2*half
    double ang = (double)p * inv;
    table[e] = make_float2((float)cos(ang), (float)sin(ang));
}

void cc_launch_rope_table(float2* table, int n_pos, int d_h, double base, hipStream_t s) {
    int half = d_h / 2;
    int64_t n = (int64_t)n_pos * half;
    hipLaunchKernelGGL(rope_table_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, table,
                       n_pos, half, log2(base));
}

// Plain copy, 16 bytes per lane, grid-stride: the known-traffic kernel that the
// HBM byte counters are calibrated against.
__global__ __launch_bounds__(256) void calib_copy_kernel(u32x4* __restrict__ dst,
                                                         const u32x4* __restrict__ src, int64_t n) {
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256)
        dst[i] = src[i];
}

void cc_launch_copy(void* dst, const void* src, int64_t bytes, hipStream_t s) {
    const int64_t n = bytes / 16;
    if (n <= 0) return;
    int64_t blocks = (n + 255) / 256;
    if (blocks > 256 * 64) blocks = 256 * 64;
    hipLaunchKernelGGL(calib_copy_kernel, dim3((unsigned)blocks), dim3(256), 0, s, (u32x4*)dst,
                       (const u32x4*)src, n);
}
