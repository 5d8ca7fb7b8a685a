// Elementwise and reduction kernels around the product: zero fill (k = 0),
// split-K partial reduction, operand conversion for the reduced-precision
// forms, and the binary64 comparison reduction.
#include "kernels.hpp"

// --------------------------------------------------------------------------
// C = 0 (the empty sum, k == 0).
__global__ void fill_zero_kernel(float *C, int64_t ldc, int m, int n) {
    const int64_t total = (int64_t)m * n;
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < total;
         i += (int64_t)gridDim.x * blockDim.x) {
        const int64_t r = i / n, c = i - r * n;
        C[r * ldc + c] = 0.f;
    }
}

static int grid_for(int64_t work, int per_block, int cap = 4096) {
    int64_t g = (work + per_block - 1) / per_block;
    if (g < 1) g = 1;
    if (g > cap) g = cap;
    return (int)g;
}

hipError_t launch_fill_zero(float *C, int64_t ldc, int m, int n, hipStream_t s) {
    hipLaunchKernelGGL(fill_zero_kernel, dim3(grid_for((int64_t)m * n, 256)), dim3(256), 0, s, C, ldc,
                       m, n);
    return hipGetLastError();
}

// --------------------------------------------------------------------------
// Split-K: C[i][j] = scale * sum_{p=0}^{S-1} ws[p][i][j], summed in ascending
// p so the result does not depend on which workgroup finished first.
__global__ void splitk_reduce_kernel(const float *__restrict__ ws, int64_t split_stride, int splits,
                                     float scale, float *__restrict__ C, int64_t ldc, int m, int n) {
    const int64_t total = (int64_t)m * n;
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < total;
         i += (int64_t)gridDim.x * blockDim.x) {
        float acc = ws[i];
        for (int p = 1; p < splits; ++p) acc += ws[p * split_stride + i];
        const int64_t r = i / n, c = i - r * n;
        C[r * ldc + c] = acc * scale;
    }
}

// Tuning operands: element i of a buffer of `count` elements gets a value in
// (-4, 4) from a hash of i (a 32-bit integer mix), so the timed products
// toggle the matrix cores and draw the power that real data draws (all-zero
// operands let the clock run higher than any real product would).  Element
// types: 4 = float32, 2 = the upper half of the float32 value (read as
// bfloat16 or as binary16, finite either way), 1 = E4M3 (random sign and
// mantissa, exponent field 4..8: no NaN code).
__device__ __forceinline__ uint32_t tune_hash(uint64_t i, uint32_t seed) {
    uint32_t h = (uint32_t)i * 0x9E3779B1u ^ (uint32_t)(i >> 32) * 0x85EBCA77u ^ seed;
    h ^= h >> 16;
    h *= 0x7FEB352Du;
    h ^= h >> 15;
    h *= 0x846CA68Bu;
    h ^= h >> 16;
    return h;
}

__global__ void fill_tuning_kernel(void *p, int64_t count, int elem_bytes, uint32_t seed) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < count;
         i += (int64_t)gridDim.x * blockDim.x) {
        const uint32_t h = tune_hash((uint64_t)i, seed);
        if (elem_bytes == 1) {
            static_cast<uint8_t *>(p)[i] = (uint8_t)((h & 0x80u) | ((4u + (h >> 8) % 5u) << 3) | ((h >> 16) & 7u));
        } else {
            const float v = ((float)(h >> 8) * (1.f / 8388608.f) - 1.f) * 4.f;
            if (elem_bytes == 4) static_cast<float *>(p)[i] = v;
            else static_cast<uint16_t *>(p)[i] = (uint16_t)(__float_as_uint(v) >> 16);
        }
    }
}

hipError_t launch_fill_tuning(void *p, int64_t count, int elem_bytes, uint32_t seed, hipStream_t s) {
    if (count <= 0) return hipSuccess;
    hipLaunchKernelGGL(fill_tuning_kernel, dim3(grid_for(count, 256, 8192)), dim3(256), 0, s, p, count, elem_bytes,
                       seed);
    return hipGetLastError();
}

// Plan upload: read over PCIe from the pinned staging buffer by a kernel.  In
// front of a kernel on the same stream this costs less than an asynchronous
// copy, whose engine the stream has to hand over to and wait for: 512 grouped
// bfloat16 problems (150 KB) 155 us a call with
// hipMemcpyAsync, 139 now.
__global__ __launch_bounds__(256) void upload_kernel(u32x4 *__restrict__ dst, const u32x4 *__restrict__ src,
                                                     int64_t count) {
    const int64_t i = blockIdx.x * (int64_t)256 + threadIdx.x;
    if (i < count) dst[i] = src[i];
}

hipError_t launch_upload(void *dst, const void *pinned, int64_t bytes, hipStream_t s) {
    const int64_t count = bytes / 16;
    hipLaunchKernelGGL(upload_kernel, dim3((uint32_t)((count + 255) / 256)), dim3(256), 0, s, static_cast<u32x4 *>(dst),
                       static_cast<const u32x4 *>(pinned), count);
    return hipGetLastError();
}

hipError_t launch_splitk_reduce(const float *ws, int64_t split_stride, int splits, float scale,
                                float *C, int64_t ldc, int m, int n, hipStream_t s) {
    hipLaunchKernelGGL(splitk_reduce_kernel, dim3(grid_for((int64_t)m * n, 256, 8192)), dim3(256), 0, s,
                       ws, split_stride, splits, scale, C, ldc, m, n);
    return hipGetLastError();
}

// --------------------------------------------------------------------------
// Four consecutive elements from index 4 * i of `count` (zero past the end);
// any alignment of x.
__device__ __forceinline__ f32x4 load4(const float *__restrict__ x, int64_t i, int64_t count) {
    f32x4 v = {0.f, 0.f, 0.f, 0.f};
    if (4 * i + 4 <= count) {
        __builtin_memcpy(&v, x + 4 * i, 16);
    } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (4 * i + e < count) v[e] = x[4 * i + e];
    }
    return v;
}

// The four groups i, i + step, i + 2 step, i + 3 step.  `whole` (uniform over
// the workgroup: all of its threads' groups lie before `count`) keeps the
// loads free of bounds branches, so the four are in flight together.
__device__ __forceinline__ void load4x4(const float *__restrict__ x, int64_t i, int64_t step, int64_t count, bool whole,
                                        f32x4 (&v)[4]) {
    if (whole) {
#pragma unroll
        for (int u = 0; u < 4; ++u) __builtin_memcpy(&v[u], x + 4 * (i + u * step), 16);
    } else {
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = load4(x, i + u * step, count);
    }
}

// --------------------------------------------------------------------------
// float32 -> bfloat16, round to nearest even: add half an ulp of the kept
// part (0x7FFF) plus the kept part's lowest bit, then truncate.  NaN stays a
// quiet NaN.
__device__ __forceinline__ uint16_t f32_to_bf16_rne(float x) {
    const uint32_t u = __float_as_uint(x);
    if ((u & 0x7FFFFFFFu) > 0x7F800000u) return (uint16_t)((u >> 16) | 0x40u);
    return (uint16_t)((u + 0x7FFFu + ((u >> 16) & 1u)) >> 16);
}

__device__ __forceinline__ uint16_t f32_to_f16_rne(float x) {
    // the hardware conversion rounds to nearest even (default mode)
    return __builtin_bit_cast(uint16_t, (_Float16)x);
}

// Bound by the read of x and the write of its codes: four 16-byte loads in
// flight and four 8-byte stores per thread.  8192^2 to bfloat16: 110.6 us
// with one element per thread and pass, 82.2 us now (4.9 TB/s, a large copy's
// rate).
template <bool BF16>
__global__ __launch_bounds__(256) void convert_kernel(const float *__restrict__ x, int64_t count,
                                                      uint16_t *__restrict__ out) {
    const int64_t groups = (count + 3) / 4, step = (int64_t)gridDim.x * 256;
    for (int64_t b = blockIdx.x * (int64_t)256; b < groups; b += 4 * step) {
        const int64_t i = b + threadIdx.x;
        f32x4 v[4];
        load4x4(x, i, step, count, 4 * (b + 256 + 3 * step) <= count, v);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int64_t at = 4 * (i + u * step);
            uint16_t h[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) h[e] = BF16 ? f32_to_bf16_rne(v[u][e]) : f32_to_f16_rne(v[u][e]);
            if (at + 4 <= count) {
                __builtin_memcpy(out + at, h, 8);
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (at + e < count) out[at + e] = h[e];
            }
        }
    }
}

hipError_t launch_convert_f32(const float *x, int64_t count, int to_mode, void *out, hipStream_t s) {
    const int g = grid_for(count, 256 * 16, 8192);
    if (to_mode == GEMM_MODE_BF16)
        hipLaunchKernelGGL(convert_kernel<true>, dim3(g), dim3(256), 0, s, x, count, (uint16_t *)out);
    else
        hipLaunchKernelGGL(convert_kernel<false>, dim3(g), dim3(256), 0, s, x, count, (uint16_t *)out);
    return hipGetLastError();
}

// --------------------------------------------------------------------------
// OCP E4M3 ("fn") encoding of a float32 value, round to nearest even with
// saturation to +-448.  Normal codes: value = 2^(E-7) * (1 + F/8), E in
// 1..15 (E = 15, F = 7 is NaN, so 448 = 2^8 * 1.75 is the largest);
// subnormals: value = F * 2^-9.
__device__ __forceinline__ uint8_t f32_to_e4m3_sat(float x) {
    const uint32_t sign = (__float_as_uint(x) >> 24) & 0x80u;
    const float a = fabsf(x);
    // below 448 the hardware conversion (round to nearest even, subnormal
    // codes included) needs no saturation
    const uint32_t code = (uint32_t)__builtin_amdgcn_cvt_pk_fp8_f32(a, 0.f, 0, false) & 0xFFu;
    return (uint8_t)(sign | (a < 448.f ? code : 0x7Eu));   // saturate (also NaN -> 448)
}

__device__ __forceinline__ uint32_t absmax4(uint32_t m, const f32x4 &v) {
#pragma unroll
    for (int e = 0; e < 4; ++e) m = max(m, __float_as_uint(v[e]) & 0x7FFFFFFFu);
    return m;
}

// Maximum of m over the workgroup's WAVES waves, in every thread.
template <int WAVES>
__device__ __forceinline__ uint32_t block_max(uint32_t m) {
    for (int off = 32; off > 0; off >>= 1) m = max(m, (uint32_t)__shfl_xor((int)m, off));
    __shared__ uint32_t wmax[WAVES];
    if ((threadIdx.x & 63) == 0) wmax[threadIdx.x >> 6] = m;
    __syncthreads();
    uint32_t b = wmax[0];
#pragma unroll
    for (int w = 1; w < WAVES; ++w) b = max(b, wmax[w]);
    return b;
}

// s = amax / 448 (IEEE division), 1 for an all-zero tensor.
__device__ __forceinline__ float e4m3_scale(uint32_t amax_bits) {
    const float amax = __uint_as_float(amax_bits);
    return (amax == 0.f) ? 1.f : amax / 448.f;
}

// Codes of elements 4 i .. 4 i + 3 (those before `count`).
__device__ __forceinline__ void quantize4(const f32x4 &v, float s, uint8_t *__restrict__ q, int64_t i, int64_t count) {
    uint32_t w = 0;
#pragma unroll
    for (int e = 0; e < 4; ++e) w |= (uint32_t)f32_to_e4m3_sat(v[e] / s) << (8 * e);
    if (4 * i + 4 <= count) {
        __builtin_memcpy(q + 4 * i, &w, 4);
    } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (4 * i + e < count) q[4 * i + e] = (uint8_t)(w >> (8 * e));
    }
}

// amax via the bit patterns of |x|: for non-negative floats the unsigned
// order of the bits is the numeric order, so an integer max is exact.  One
// partial maximum per workgroup; the quantising kernel folds them (a maximum
// is the same in any order).  Bound by the read of x: four 16-byte loads in
// flight per thread.  4096^2: 55.5 us with one 4-byte load per thread
// and pass and an atomic per workgroup, 12.9 us now (5.2 TB/s).  The
// quantising kernel: 22.8 us, now 19.7 (its IEEE divisions cost 1.5 of them).
#define QUANT_PARTS 1024
__global__ __launch_bounds__(256) void amax_partial_kernel(const float *__restrict__ x, int64_t count,
                                                           uint32_t *__restrict__ parts) {
    uint32_t m = 0;
    const int64_t groups = (count + 3) / 4, step = (int64_t)gridDim.x * 256;
    for (int64_t b = blockIdx.x * (int64_t)256; b < groups; b += 4 * step) {
        const int64_t i = b + threadIdx.x;
        f32x4 v[4];
        load4x4(x, i, step, count, 4 * (b + 256 + 3 * step) <= count, v);
#pragma unroll
        for (int u = 0; u < 4; ++u) m = absmax4(m, v[u]);
    }
    m = block_max<4>(m);
    if (threadIdx.x == 0) parts[blockIdx.x] = m;
}

__global__ __launch_bounds__(256) void quantize_e4m3_kernel(const float *__restrict__ x, int64_t count,
                                                            uint8_t *__restrict__ q,
                                                            const uint32_t *__restrict__ parts, int nparts,
                                                            float *scale_out) {
    uint32_t m = 0;
    for (int i = threadIdx.x; i < nparts; i += 256) m = max(m, parts[i]);
    const float s = e4m3_scale(block_max<4>(m));
    if (blockIdx.x == 0 && threadIdx.x == 0) *scale_out = s;
    const int64_t groups = (count + 3) / 4, step = (int64_t)gridDim.x * 256;
    for (int64_t b = blockIdx.x * (int64_t)256; b < groups; b += 4 * step) {
        const int64_t i = b + threadIdx.x;
        f32x4 v[4];
        load4x4(x, i, step, count, 4 * (b + 256 + 3 * step) <= count, v);
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (i + u * step < groups) quantize4(v[u], s, q, i + u * step, count);
    }
}

// A tensor that one workgroup of 1024 threads holds in its registers (4 VEC
// elements per thread): maximum and codes in one launch, one read of x.
template <int VEC>
__global__ __launch_bounds__(1024) void quantize_e4m3_one_kernel(const float *__restrict__ x, int64_t count,
                                                                 uint8_t *__restrict__ q, float *scale_out) {
    f32x4 v[VEC];
    uint32_t m = 0;
#pragma unroll
    for (int u = 0; u < VEC; ++u) v[u] = load4(x, u * 1024 + (int)threadIdx.x, count);
#pragma unroll
    for (int u = 0; u < VEC; ++u) m = absmax4(m, v[u]);
    const float s = e4m3_scale(block_max<16>(m));
    if (threadIdx.x == 0) *scale_out = s;
#pragma unroll
    for (int u = 0; u < VEC; ++u) {
        const int64_t i = u * 1024 + (int)threadIdx.x;
        if (4 * i < count) quantize4(v[u], s, q, i, count);
    }
}

hipError_t launch_quantize_e4m3(const float *x, int64_t count, uint8_t *q, float *scale_out,
                                uint32_t *amax_scratch, hipStream_t s) {
    // up to 32768 elements (what 1024 threads hold without spilling) one launch:
    // 7.5 us a call at 32768 elements, 8.2 in two launches at 32769
    if (count <= 4 * 1024 * 4) {
        hipLaunchKernelGGL(quantize_e4m3_one_kernel<4>, dim3(1), dim3(1024), 0, s, x, count, q, scale_out);
        return hipGetLastError();
    }
    if (count <= 8 * 1024 * 4) {
        hipLaunchKernelGGL(quantize_e4m3_one_kernel<8>, dim3(1), dim3(1024), 0, s, x, count, q, scale_out);
        return hipGetLastError();
    }
    const int parts = grid_for(count, 256 * 16, QUANT_PARTS);
    hipLaunchKernelGGL(amax_partial_kernel, dim3(parts), dim3(256), 0, s, x, count, amax_scratch);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(quantize_e4m3_kernel, dim3(grid_for(count, 256 * 16, 4096)), dim3(256), 0, s, x, count, q,
                       amax_scratch, parts, scale_out);
    return hipGetLastError();
}

// --------------------------------------------------------------------------
// Comparison reduction in binary64: per-block partial (sum d^2, sum R^2,
// max |d|) over a grid-stride walk, then one block folds the partials in
// index order, so the result is independent of scheduling.
__device__ __forceinline__ void reduce3_block(double &a, double &b, double &c, double *sh) {
    for (int off = 32; off > 0; off >>= 1) {
        a += __shfl_xor(a, off);
        b += __shfl_xor(b, off);
        c = fmax(c, __shfl_xor(c, off));
    }
    const int w = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) {
        sh[3 * w] = a;
        sh[3 * w + 1] = b;
        sh[3 * w + 2] = c;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int i = 1; i < (int)(blockDim.x >> 6); ++i) {
            a += sh[3 * i];
            b += sh[3 * i + 1];
            c = fmax(c, sh[3 * i + 2]);
        }
    }
}

__global__ void errnorm_partial_kernel(const float *__restrict__ C, int64_t ldc, const double *__restrict__ R,
                                       int64_t ldr, int64_t m, int64_t n, double *partials) {
    double sd = 0.0, sr = 0.0, mx = 0.0;
    const int64_t total = m * n;
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < total;
         i += (int64_t)gridDim.x * blockDim.x) {
        const int64_t r = i / n, c = i - r * n;
        const double ref = R[r * ldr + c];
        const double d = (double)C[r * ldc + c] - ref;
        sd = fma(d, d, sd);
        sr = fma(ref, ref, sr);
        mx = fmax(mx, fabs(d));
    }
    __shared__ double sh[3 * 4];
    reduce3_block(sd, sr, mx, sh);
    if (threadIdx.x == 0) {
        partials[3 * blockIdx.x] = sd;
        partials[3 * blockIdx.x + 1] = sr;
        partials[3 * blockIdx.x + 2] = mx;
    }
}

__global__ void errnorm_final_kernel(const double *partials, int nparts, double *out3) {
    double sd = 0.0, sr = 0.0, mx = 0.0;
    for (int i = threadIdx.x; i < nparts; i += blockDim.x) {
        sd += partials[3 * i];
        sr += partials[3 * i + 1];
        mx = fmax(mx, partials[3 * i + 2]);
    }
    __shared__ double sh[3 * 4];
    reduce3_block(sd, sr, mx, sh);
    if (threadIdx.x == 0) {
        out3[0] = sd;
        out3[1] = sr;
        out3[2] = mx;
    }
}

hipError_t launch_errnorm(const float *C, int64_t ldc, const double *R, int64_t ldr, int64_t m, int64_t n,
                          double *out3, double *partials, int nparts, hipStream_t s) {
    const int g = grid_for(m * n, 256, nparts);
    hipLaunchKernelGGL(errnorm_partial_kernel, dim3(g), dim3(256), 0, s, C, ldc, R, ldr, m, n, partials);
    hipLaunchKernelGGL(errnorm_final_kernel, dim3(1), dim3(256), 0, s, partials, g, out3);
    return hipGetLastError();
}
