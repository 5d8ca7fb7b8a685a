// Operand preparation of the pre-split split-BF16x3 path: each float32
// operand becomes a bfloat16 copy in which every block of 16 consecutive k
// holds the 16 hi and then the 16 lo parts (of A's row: 32 elements; of B:
// 32 rows).  The product (Lp2Cfg's split form) reads each part once per tile
// and issues, per 16 k, lo_A hi_B, then hi_A lo_B, then hi_A hi_B: the three
// products of the compensated form in the order the register-staged split
// tile issues them (same bits).  hi = RNE_bf16(x), lo = RNE_bf16(x - hi), as
// at that tile's staging.
#include "kernels.hpp"
#include "tile_lp.hpp"

// Eight consecutive floats of row r from column c, zero at and beyond `cols`.
__device__ __forceinline__ void load8(const float *__restrict__ P, int64_t ld, int r, int c, int cols, float (&v)[8]) {
    const float *p = P + (int64_t)r * ld + c;
    if (c + 8 <= cols) {
        const u32x4 x = ld16(p), y = ld16(p + 4);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            v[e] = __uint_as_float(x[e]);
            v[4 + e] = __uint_as_float(y[e]);
        }
    } else {
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = c + e < cols ? p[e] : 0.f;
    }
}

__device__ __forceinline__ void split8(const float (&v)[8], u32x4 &hi, u32x4 &lo) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        uint32_t h, l;
        split_bf16_pair(v[2 * e], v[2 * e + 1], h, l);
        hi[e] = h;
        lo[e] = l;
    }
}

// One launch for both operands: the first `a_blocks` workgroups take A, the
// others B, one thread per eight consecutive elements.
//   A, row i, k group j: A[i][8j..8j+7] -> the hi and lo slots of its 16-k
//   block b = j/2, half h = j%2;
//   B, k row r, column group c: B[r][8c..8c+7] -> rows 32 (r/16) + r%16 (hi)
//   and +16 (lo) of Bp, whose rows are n8 columns (n rounded up to
//   8; the padding and the rows r >= k are zero).
// Bound by the read and the two writes: 2048^2 of each 12.3 us (5.5 TB/s).
__global__ __launch_bounds__(256) void presplit_kernel(const float *__restrict__ A, int64_t lda, int m, int k, int k16,
                                                       uint16_t *__restrict__ Ap, const float *__restrict__ B,
                                                       int64_t ldb, int n, int n8, uint16_t *__restrict__ Bp,
                                                       int a_blocks) {
    if ((int)blockIdx.x < a_blocks) {
        const int groups = k16 / 8;
        const int64_t total = (int64_t)m * groups;
        for (int64_t t = blockIdx.x * (int64_t)256 + threadIdx.x; t < total; t += (int64_t)a_blocks * 256) {
            const int i = (int)(t / groups), j = (int)(t % groups);
            float v[8];
            load8(A, lda, i, 8 * j, k, v);
            u32x4 hi, lo;
            split8(v, hi, lo);
            uint16_t *row = Ap + (int64_t)i * 2 * k16 + (int64_t)32 * (j / 2) + 8 * (j % 2);
            *reinterpret_cast<u32x4 *>(row) = hi;
            *reinterpret_cast<u32x4 *>(row + 16) = lo;
        }
        return;
    }
    const int groups = n8 / 8;
    const int64_t total = (int64_t)k16 * groups;
    const int64_t step = (int64_t)(gridDim.x - a_blocks) * 256;
    for (int64_t t = (blockIdx.x - a_blocks) * (int64_t)256 + threadIdx.x; t < total; t += step) {
        const int r = (int)(t / groups), c = (int)(t % groups);
        float v[8];
        if (r < k) {
            load8(B, ldb, r, 8 * c, n, v);
        } else {
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] = 0.f;
        }
        u32x4 hi, lo;
        split8(v, hi, lo);
        uint16_t *base = Bp + ((int64_t)32 * (r / 16) + r % 16) * n8 + 8 * c;
        *reinterpret_cast<u32x4 *>(base) = hi;
        *reinterpret_cast<u32x4 *>(base + (int64_t)16 * n8) = lo;
    }
}

hipError_t launch_presplit(const float *A, int64_t lda, const float *B, int64_t ldb, int m, int n, int k,
                           uint16_t *Ap, uint16_t *Bp, hipStream_t s) {
    const int k16 = (k + 15) / 16 * 16, n8 = (n + 7) / 8 * 8;
    auto grid = [](int64_t work) {
        int64_t g = (work + 255) / 256;
        return (int)(g < 1 ? 1 : (g > 16384 ? 16384 : g));
    };
    const int a_blocks = grid((int64_t)m * (k16 / 8)), b_blocks = grid((int64_t)k16 * (n8 / 8));
    hipLaunchKernelGGL(presplit_kernel, dim3(a_blocks + b_blocks), dim3(256), 0, s, A, lda, m, k, k16, Ap, B, ldb, n,
                       n8, Bp, a_blocks);
    return hipGetLastError();
}
