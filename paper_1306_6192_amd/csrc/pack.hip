// Aligned copies of operands for the asynchronous-copy tiles, which move whole
// 16-byte chunks: each row of a matrix whose rows are not whole chunks (or do
// not start on one) is copied to a row of the next whole number of chunks,
// zeros behind its last element.  One launch copies A, B or both.
// Bound by the read and the write: one thread per four chunks, each read from
// any byte address with one 16-byte load and written aligned; a row's last,
// partial chunk is read as the row's last 16 bytes and shifted into place.
#include "kernels.hpp"
#include "tile_common.hpp"

struct PackMat {
    const uint8_t *src;
    uint8_t *dst;
    int64_t ld;          // bytes between source rows
    uint32_t row_bytes;  // bytes of a source row
    uint32_t chunks;     // 16-byte chunks of a copied row
    int64_t total;       // chunks of the copy (0: this matrix is not copied)
    int64_t blocks;      // workgroups that copy it
};

__device__ __forceinline__ u32x4 pack_chunk(const uint8_t *row, uint32_t row_bytes, uint32_t c) {
    const int have = (int)row_bytes - 16 * (int)c;
    if (have >= 16) return ld16(row + 16 * (int64_t)c);
    if (row_bytes >= 16) {
        // the row's last 16 bytes, its last `have` bytes moved to the front
        return shift_down16(ld16(row + row_bytes - 16), 16 - have);
    }
    uint8_t b[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) b[i] = i < have ? row[i] : 0;
    u32x4 r;
    __builtin_memcpy(&r, b, 16);
    return r;
}

__global__ __launch_bounds__(256) void pack_kernel(PackMat A, PackMat B) {
    const bool second = (int64_t)blockIdx.x >= A.blocks;
    const PackMat &M = second ? B : A;
    const int64_t base = ((int64_t)blockIdx.x - (second ? A.blocks : 0)) * 1024 + threadIdx.x;
    u32x4 v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int64_t t = base + 256 * u;
        if (t < M.total) {
            const int64_t r = M.total <= UINT32_MAX ? (int64_t)((uint32_t)t / M.chunks) : t / M.chunks;
            v[u] = pack_chunk(M.src + r * M.ld, M.row_bytes, (uint32_t)(t - r * M.chunks));
        }
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int64_t t = base + 256 * u;
        if (t < M.total) *reinterpret_cast<u32x4 *>(M.dst + 16 * t) = v[u];
    }
}

static PackMat pack_mat(const void *src, int64_t ld_bytes, int64_t rows, int64_t row_bytes, void *dst) {
    PackMat M;
    M.src = static_cast<const uint8_t *>(src);
    M.dst = static_cast<uint8_t *>(dst);
    M.ld = ld_bytes;
    M.row_bytes = (uint32_t)row_bytes;
    M.chunks = (uint32_t)((row_bytes + 15) / 16);
    M.total = dst ? rows * M.chunks : 0;
    M.blocks = (M.total + 1023) / 1024;
    return M;
}

hipError_t launch_pack(const void *A, int64_t lda_bytes, int64_t a_rows, int64_t a_row_bytes, void *Ap, const void *B,
                       int64_t ldb_bytes, int64_t b_rows, int64_t b_row_bytes, void *Bp, hipStream_t s) {
    const PackMat a = pack_mat(A, lda_bytes, a_rows, a_row_bytes, Ap);
    const PackMat b = pack_mat(B, ldb_bytes, b_rows, b_row_bytes, Bp);
    const int64_t blocks = a.blocks + b.blocks;
    if (blocks == 0) return hipSuccess;
    hipLaunchKernelGGL(pack_kernel, dim3((uint32_t)blocks), dim3(256), 0, s, a, b);
    return hipGetLastError();
}
