// Reduced-precision output tile of C = A*B on gfx950 matrix cores:
//   BF16 / F16        v_mfma_f32_32x32x16_{bf16,f16}, k-tile 64
//   FP8 E4M3          v_mfma_f32_32x32x64_f8f6f4 (no block scaling), k-tile 128
//   split-BF16x3      three v_mfma_f32_32x32x16_bf16 per step on float32
//                     inputs split at staging into hi = RNE_bf16(x) and
//                     lo = RNE_bf16(x - hi): acc += hiA hiB + hiA loB + loA hiB
// All accumulate in float32.
//
// Structure (same as the FP32 tile): 256-lane workgroup, 2 x 2 waves, two LDS
// stages, the next k-tile's global loads in flight during the current k-tile's
// MFMAs, one barrier per k-tile.
//
// Operand layout.  These MFMAs take, per lane, several consecutive-k values of
// one A row (lane l: row l%32) and of one B column (lane l: column l%32); the
// two lane halves (l/32) hold two disjoint k-groups, A and B alike.  A is
// row-major (k contiguous) in HBM, so an A row is staged as is.  B is
// row-major k x n (n contiguous):
//   * BF16, F16, FP8: its rows are staged as they are too, and each lane's
//     consecutive k are gathered by the transposing LDS reads.  Consecutive
//     lanes load consecutive 16-byte chunks of a row, so one load instruction
//     touches a few rows.  (Transposing in registers at staging, as below, had
//     every lane of a load on another row, one address cycle and one cache
//     line each, and the address units bound the kernels: 512 grouped bfloat16
//     problems 145 us against 131 now, 48 grouped E4M3 problems of 64..4096
//     156 against 112, binary16 2047 x 1999 x 2501 112 against 105.)
//   * split-BF16x3: the staging transposes it in registers while it splits:
//     each thread loads TKB rows of 16 bytes (VN columns) and writes VN LDS
//     rows of TKB consecutive-k elements ("B^T" rows); lanes of one LDS write
//     cover one B^T row, so those writes are free of bank conflicts.
//
// Column permutation (split-BF16x3): as in the FP32 tile, lane jj of
// accumulator block cb computes output column CB*jj + cb of the wave's columns,
// so the epilogue stores CB consecutive floats per lane.  The B^T row of
// wave-local column n = CB*jj + cb is stored at LDS row 32*cb + jj, which makes
// every fragment read a run of consecutive LDS rows (conflict-free with the
// padded stride).  The other forms' columns are in natural order.
#pragma once

#include "tile_common.hpp"

typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef int i32x2 __attribute__((ext_vector_type(2)));

// The MFMA B operand (consecutive k of one column per lane) of the 32 columns
// from n0 and the k-step from k0, gathered from row-major LDS rows of `rowb`
// bytes with the transposing reads (see tile_lp2.hpp for their lane layout);
// `swz` gives the chunk swizzle of a row.  16-bit: 16 k, 8-bit: 64 k.
template <class Swz>
__device__ __forceinline__ u32x4 lp_b_fragment16(const uint8_t *Bs, int rowb, int k0, int n0, Swz swz) {
    const int lane = threadIdx.x & 63;
    const int p16 = lane & 15, G = lane >> 4;
    const int n = n0 + 16 * (G & 1) + 4 * (p16 & 3);
    s16x4 hv[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int k = k0 + 8 * (G >> 1) + 4 * h + (p16 >> 2);
        const uint8_t *a = Bs + k * rowb + 16 * ((n >> 3) ^ swz(k)) + 2 * (n & 7);
        hv[h] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4 *)a);
    }
    const i32x2 lo = __builtin_bit_cast(i32x2, hv[0]);
    const i32x2 hi = __builtin_bit_cast(i32x2, hv[1]);
    return (u32x4){(uint32_t)lo[0], (uint32_t)lo[1], (uint32_t)hi[0], (uint32_t)hi[1]};
}

template <class Swz>
__device__ __forceinline__ i32x8 lp_b_fragment8(const uint8_t *Bs, int rowb, int k0, int n0, Swz swz) {
    const int lane = threadIdx.x & 63;
    const int p16 = lane & 15, G = lane >> 4;
    // (the swizzle repeats every 8 rows: one address, the four reads 8 rows apart)
    const int k = k0 + 32 * (G >> 1) + (p16 >> 1);
    const uint8_t *a = Bs + k * rowb + 16 * (((n0 >> 4) + (G & 1)) ^ swz(p16 >> 1)) + 8 * (p16 & 1);
    i32x2 q[4];
#pragma unroll
    for (int h = 0; h < 4; ++h)
        q[h] = __builtin_amdgcn_ds_read_tr8_b64_v2i32((__attribute__((address_space(3))) i32x2 *)(a + 8 * h * rowb));
    return (i32x8){q[0][0], q[0][1], q[1][0], q[1][1], q[2][0], q[2][1], q[3][0], q[3][1]};
}

// Natural-column epilogue: lane l%32 of accumulator block cb holds output
// column 32*cb + l%32 of the wave's columns.
template <class Cfg>
__device__ __forceinline__ void lp2_epilogue(float *__restrict__ C, int64_t ldc, int M, int N, int m0, int n0,
                                             float scale, const f32x16 (&acc)[Cfg::RB][Cfg::CB]) {
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    const int wm = wave / Cfg::WN, wn = wave % Cfg::WN;
    const int l32 = lane & 31, g = lane >> 5;
#pragma unroll
    for (int rb = 0; rb < Cfg::RB; ++rb)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int row = m0 + wm * Cfg::TM + rb * 32 + 8 * (r >> 2) + 4 * g + (r & 3);
            if (row >= M) continue;
            float *p = C + (int64_t)row * ldc;
#pragma unroll
            for (int cb = 0; cb < Cfg::CB; ++cb) {
                const int col = n0 + wn * Cfg::TN + cb * 32 + l32;
                if (col < N) p[col] = acc[rb][cb][r] * scale;
            }
        }
}

template <int MODE> struct LpTraits;
template <> struct LpTraits<GEMM_MODE_BF16> {
    static constexpr int IN_ESZ = 2, BK = 64, PLANES = 1, ROW = 128, KCH = 16, VB = 16;
};
template <> struct LpTraits<GEMM_MODE_F16> {
    static constexpr int IN_ESZ = 2, BK = 64, PLANES = 1, ROW = 128, KCH = 16, VB = 16;
};
template <> struct LpTraits<GEMM_MODE_F8E4M3> {
    static constexpr int IN_ESZ = 1, BK = 128, PLANES = 1, ROW = 128, KCH = 64, VB = 32;
};
template <> struct LpTraits<GEMM_MODE_F32_SPLIT_BF16X3> {
    static constexpr int IN_ESZ = 4, BK = 32, PLANES = 2, ROW = 64, KCH = 16, VB = 16;
};

// BK_ may halve the mode's k-tile (half the LDS, for more resident
// workgroups); the MFMA k-steps and their order are the same.
template <int MODE_, int BM_, int BN_, int BK_ = LpTraits<MODE_>::BK>
struct LpCfg {
    typedef LpTraits<MODE_> T;
    static constexpr int MODE = MODE_;
    static constexpr int BM = BM_, BN = BN_, BK = BK_;
    static constexpr int ROW = T::ROW / (T::BK / BK);   // bytes of a staged LDS row per plane
    static_assert(BK == T::BK || 2 * BK == T::BK, "the mode's k-tile or half of it");
    static constexpr int WM = 2, WN = 2;
    static constexpr int THREADS = GEMM_THREADS;
    static constexpr int TM = BM / WM, TN = BN / WN;
    static constexpr int RB = TM / 32, CB = TN / 32;
    static constexpr int RS = ROW + 16;          // padded LDS row stride in bytes (odd multiple of 16)
    // BF16 / F16 / FP8: A rows unpadded, their 16-byte chunks XOR-swizzled
    // by row (a_swz), so that the staging writes (several chunks of a few
    // rows per 16-lane phase) and the fragment reads (one chunk of each of
    // 16 rows per read) both hit 64 distinct banks; the padded stride puts
    // the rows of one staging phase on overlapping banks.  Split-BF16x3
    // (two planes of 8-byte pieces) keeps RS.
    static constexpr bool SWZ_A = T::PLANES == 1;
    static constexpr int RSA = SWZ_A ? ROW : RS;  // LDS row stride of A in bytes
    __device__ static __forceinline__ int a_swz(int r) {
        if constexpr (ROW / 16 == 8) return (r >> 1) & 7;
        return ((r >> 1) ^ (r >> 2)) & 3;
    }
    // row-major B in LDS, its 16-byte chunks XOR-swizzled by row
    static constexpr bool ROW_B = T::PLANES == 1;
    static constexpr int B_ROWB = BN * T::IN_ESZ, B_CPR = B_ROWB / 16;
    __device__ static __forceinline__ int b_swz(int k) {
        return (T::IN_ESZ == 2 ? 4 * (k & 3) : 2 * (k & 7)) & (B_CPR - 1);
    }
    static constexpr int PLANE_A = BM * RSA, PLANE_B = ROW_B ? BK * B_ROWB : BN * RS;
    static constexpr int A_BYTES = T::PLANES * PLANE_A, B_BYTES = T::PLANES * PLANE_B;
    static constexpr int STAGE = A_BYTES + B_BYTES;
    static constexpr int LDS_BYTES = 2 * STAGE;
    static constexpr int VPR = BK * T::IN_ESZ / 16;        // 16-B global vectors per A row
    static constexpr int AV = BM * VPR / GEMM_THREADS;     // A vectors per thread
    static constexpr int VN = 16 / T::IN_ESZ;              // B columns per 16-B global vector
    static constexpr int NBLK = BN / VN;                   // column blocks of B per k-tile
    static constexpr int TKB = BK * NBLK / GEMM_THREADS;   // k rows per thread's B block
    static constexpr int KBLK = BK / TKB;                  // k blocks per k-tile
    static constexpr int MFMA_K = T::KCH;
    // B vector q of this thread: k row kr of the k-tile, column c
    __device__ static __forceinline__ void b_pos(int q, int &kr, int &c) {
        if constexpr (ROW_B) {
            const int idx = threadIdx.x + q * GEMM_THREADS;
            kr = idx / NBLK;
            c = (idx % NBLK) * VN;
        } else {
            kr = (threadIdx.x % KBLK) * TKB + q;
            c = (threadIdx.x / KBLK) * VN;
        }
    }
    static_assert((RS / 16) % 2 == 1, "row stride must be an odd multiple of 16 bytes");
    static_assert(RB >= 1 && (CB == 1 || CB == 2 || CB == 4), "wave tile");
    static_assert(AV >= 1 && AV * GEMM_THREADS == BM * VPR, "A staging");
    static_assert(TKB >= 2 && TKB * KBLK == BK && KBLK * NBLK == GEMM_THREADS, "B staging");
    static_assert(LDS_BYTES <= 160 * 1024, "LDS");
    __device__ static void run(const TileProblem &P, int tm, int tn, int split, uint8_t *lds);
};

// ---------------------------------------------------------------------------
// Global loads (zero outside the matrix).  Elements of ESZ bytes; a row
// segment of 16 bytes starting at element column c of row r.
template <int ESZ>
__device__ __forceinline__ u32x4 lp_load16(const uint8_t *__restrict__ base, int64_t ld, int r, int c, int R,
                                           int Cn) {
    constexpr int N = 16 / ESZ;
    u32x4 v = {0u, 0u, 0u, 0u};
    if (r < R) {
        const uint8_t *p = base + ((int64_t)r * ld + c) * ESZ;
        if (c + N <= Cn) {
            v = ld16(p);
        } else if (ESZ < 4 && Cn >= N) {
            // the row's last 16 bytes, its last Cn - c elements moved to the
            // front: one load where 8 or 16 are behind as many branches, which
            // every wave of a tile at the matrices' ends takes (E4M3
            // 1502x1350x461 14.8 -> 9.3 us, 172 drawn ragged products 1.09 times
            // faster, bfloat16 1.04; four float32 loads are not slower)
            if (c < Cn) v = shift_down16(ld16(p - (c + N - Cn) * ESZ), (c + N - Cn) * ESZ);
        } else {
            uint8_t b[16];
#pragma unroll
            for (int i = 0; i < 16; ++i) b[i] = 0;
#pragma unroll
            for (int e = 0; e < N; ++e)
                if (c + e < Cn) {
#pragma unroll
                    for (int i = 0; i < ESZ; ++i) b[e * ESZ + i] = p[e * ESZ + i];
                }
            __builtin_memcpy(&v, b, 16);
        }
    }
    return v;
}

// hi = RNE_bf16(x), lo = RNE_bf16(x - hi) of two floats, each pair packed (x0
// in the low half); x - hi is exact in float32.  The hardware conversion of
// pairs (v_cvt_pk_bf16_f32: round to nearest even, denormals kept; a NaN stays
// a NaN), 7 instructions per pair where rounding by integer arithmetic took
// about 20: the register-staged split tiles are bound by them, since every
// output tile splits its operands again (128x4096x4096 35.8 -> 32.5 us,
// 2000x300x4000 52.4 -> 47.7, 512 grouped problems of 32..1024 240 -> 218).
// Equal to that rounding for every finite input; of infinities and NaN only the
// bits of NaN parts differ (the integer form wrapped the largest ones to zero).
__device__ __forceinline__ void split_bf16_pair(float x0, float x1, uint32_t &hi, uint32_t &lo) {
    typedef __bf16 Pair __attribute__((ext_vector_type(2)));
    const f32x2 x = {x0, x1};
    hi = __builtin_bit_cast(uint32_t, __builtin_convertvector(x, Pair));
    const f32x2 r = {x0 - __uint_as_float(hi << 16), x1 - __uint_as_float(hi & 0xFFFF0000u)};
    lo = __builtin_bit_cast(uint32_t, __builtin_convertvector(r, Pair));
}

// LDS row of the B^T row holding wave-tile-local column n (see the column
// permutation above).
template <class Cfg>
__device__ __forceinline__ int bt_row(int n) {
    const int wn = n / Cfg::TN, nn = n % Cfg::TN;
    return wn * Cfg::TN + (nn % Cfg::CB) * 32 + nn / Cfg::CB;
}

template <class Cfg>
struct LpStage {
    u32x4 a[Cfg::AV];
    u32x4 b[Cfg::TKB];
};

template <class Cfg>
__device__ __forceinline__ void lp_load_tiles(const TileProblem &P, int m0, int n0, int k0, LpStage<Cfg> &R) {
    constexpr int ESZ = Cfg::T::IN_ESZ;
    const int tid = threadIdx.x;
    const uint8_t *A = static_cast<const uint8_t *>(P.A);
    const uint8_t *B = static_cast<const uint8_t *>(P.B);
#pragma unroll
    for (int q = 0; q < Cfg::AV; ++q) {
        const int idx = tid + q * GEMM_THREADS;
        const int r = idx / Cfg::VPR;
        const int c = (idx % Cfg::VPR) * (16 / ESZ);
        R.a[q] = lp_load16<ESZ>(A, P.lda, m0 + r, k0 + c, P.m, P.k);
    }
#pragma unroll
    for (int e = 0; e < Cfg::TKB; ++e) {
        int kr, c;
        Cfg::b_pos(e, kr, c);
        R.b[e] = lp_load16<ESZ>(B, P.ldb, k0 + kr, n0 + c, P.k, P.n);
    }
}

// Element c (of width W bits) of a 16-byte row vector.
template <int W>
__device__ __forceinline__ uint32_t lane_elem(const u32x4 &v, int c) {
    constexpr int PER = 32 / W;
    return (v[c / PER] >> ((c % PER) * W)) & ((1u << W) - 1u);
}

template <class Cfg>
__device__ __forceinline__ void lp_store_tiles(uint8_t *stage, const LpStage<Cfg> &R) {
    constexpr int MODE = Cfg::MODE;
    const int tid = threadIdx.x;
    uint8_t *As = stage;
    uint8_t *Bs = stage + Cfg::A_BYTES;
    // ---- A: row segments as they are (split: converted to two planes)
#pragma unroll
    for (int q = 0; q < Cfg::AV; ++q) {
        const int idx = tid + q * GEMM_THREADS;
        const int r = idx / Cfg::VPR;
        const int v = idx % Cfg::VPR;
        if constexpr (MODE == GEMM_MODE_F32_SPLIT_BF16X3) {
            uint32_t h[2], l[2];
#pragma unroll
            for (int e = 0; e < 2; ++e)
                split_bf16_pair(__uint_as_float(R.a[q][2 * e]), __uint_as_float(R.a[q][2 * e + 1]), h[e], l[e]);
            const u32x2 hv = {h[0], h[1]}, lv = {l[0], l[1]};
            *reinterpret_cast<u32x2 *>(As + r * Cfg::RSA + v * 8) = hv;
            *reinterpret_cast<u32x2 *>(As + Cfg::PLANE_A + r * Cfg::RSA + v * 8) = lv;
        } else if constexpr (Cfg::SWZ_A) {
            *reinterpret_cast<u32x4 *>(As + r * Cfg::RSA + 16 * (v ^ Cfg::a_swz(r))) = R.a[q];
        } else {
            *reinterpret_cast<u32x4 *>(As + r * Cfg::RSA + v * 16) = R.a[q];
        }
    }
    if constexpr (Cfg::ROW_B) {
        // ---- B: row chunks as they are
#pragma unroll
        for (int q = 0; q < Cfg::TKB; ++q) {
            int kr, c;
            Cfg::b_pos(q, kr, c);
            *reinterpret_cast<u32x4 *>(Bs + kr * Cfg::B_ROWB + 16 * ((c / Cfg::VN) ^ Cfg::b_swz(kr))) = R.b[q];
        }
        return;
    }
    // ---- B: transpose the thread's TKB x VN block into VN B^T rows
    const int kb = tid % Cfg::KBLK, nb = tid / Cfg::KBLK;
    constexpr int TKB = Cfg::TKB;
#pragma unroll
    for (int c = 0; c < Cfg::VN; ++c) {
        const int row = bt_row<Cfg>(nb * Cfg::VN + c);
        if constexpr (MODE == GEMM_MODE_F32_SPLIT_BF16X3) {
            uint32_t hw[TKB / 2], lw[TKB / 2];
#pragma unroll
            for (int p = 0; p < TKB / 2; ++p)
                split_bf16_pair(__uint_as_float(R.b[2 * p][c]), __uint_as_float(R.b[2 * p + 1][c]), hw[p], lw[p]);
            uint8_t *dh = Bs + row * Cfg::RS + kb * TKB * 2;
            __builtin_memcpy(dh, hw, sizeof(hw));
            __builtin_memcpy(dh + Cfg::PLANE_B, lw, sizeof(lw));
        } else if constexpr (Cfg::T::IN_ESZ == 2) {
            uint32_t w[TKB / 2];
#pragma unroll
            for (int p = 0; p < TKB / 2; ++p)
                w[p] = lane_elem<16>(R.b[2 * p], c) | (lane_elem<16>(R.b[2 * p + 1], c) << 16);
            __builtin_memcpy(Bs + row * Cfg::RS + kb * TKB * 2, w, sizeof(w));
        } else {  // bytes
            uint8_t w[TKB];
#pragma unroll
            for (int e = 0; e < TKB; ++e) w[e] = (uint8_t)lane_elem<8>(R.b[e], c);
            __builtin_memcpy(Bs + row * Cfg::RS + kb * TKB, w, sizeof(w));
        }
    }
}

template <class Cfg>
__device__ __forceinline__ void lp_compute_stage(const uint8_t *stage, f32x16 (&acc)[Cfg::RB][Cfg::CB]) {
    constexpr int MODE = Cfg::MODE;
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    const int wm = wave / Cfg::WN, wn = wave % Cfg::WN;
    const int l32 = lane & 31, g = lane >> 5;
    const int ar = wm * Cfg::TM + l32;             // A row of row block 0
    const uint8_t *As = stage + ar * Cfg::RSA + (Cfg::SWZ_A ? 0 : g * Cfg::T::VB);
    const uint8_t *Bs = stage + Cfg::A_BYTES + (wn * Cfg::TN + l32) * Cfg::RS + g * Cfg::T::VB;
    constexpr int CHUNK_BYTES = 2 * Cfg::T::VB;   // bytes of one MFMA k-step in a row
#pragma unroll
    for (int kc = 0; kc < Cfg::ROW / CHUNK_BYTES; ++kc) {
        if constexpr (MODE == GEMM_MODE_F8E4M3) {
            i32x8 af[Cfg::RB];
#pragma unroll
            for (int rb = 0; rb < Cfg::RB; ++rb) {
                // the lane's two chunks: 4 kc + 2 g and the next
                const uint8_t *p = As + rb * 32 * Cfg::RSA;
                const int c0 = 4 * kc + 2 * g;
                const u32x4 lo = *reinterpret_cast<const u32x4 *>(
                    p + (Cfg::SWZ_A ? 16 * (c0 ^ Cfg::a_swz(ar)) : kc * CHUNK_BYTES));
                const u32x4 hi = *reinterpret_cast<const u32x4 *>(
                    p + (Cfg::SWZ_A ? 16 * ((c0 + 1) ^ Cfg::a_swz(ar)) : kc * CHUNK_BYTES + 16));
                af[rb] = (i32x8){(int)lo[0], (int)lo[1], (int)lo[2], (int)lo[3],
                                 (int)hi[0], (int)hi[1], (int)hi[2], (int)hi[3]};
            }
            // (one B fragment at a time: the grouped kernel's registers)
#pragma unroll
            for (int cb = 0; cb < Cfg::CB; ++cb) {
                const i32x8 bf = lp_b_fragment8(stage + Cfg::A_BYTES, Cfg::B_ROWB, 64 * kc, wn * Cfg::TN + cb * 32,
                                                [](int k) { return Cfg::b_swz(k); });
#pragma unroll
                for (int rb = 0; rb < Cfg::RB; ++rb)
                    acc[rb][cb] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(af[rb], bf, acc[rb][cb], 0, 0, 0, 0,
                                                                                 0, 0);
            }
        } else {
            u32x4 af[Cfg::RB], bf[Cfg::CB];
#pragma unroll
            for (int rb = 0; rb < Cfg::RB; ++rb)
                af[rb] = *reinterpret_cast<const u32x4 *>(
                    As + rb * 32 * Cfg::RSA +
                    (Cfg::SWZ_A ? 16 * ((2 * kc + g) ^ Cfg::a_swz(ar)) : kc * CHUNK_BYTES));
#pragma unroll
            for (int cb = 0; cb < Cfg::CB; ++cb) {
                if constexpr (Cfg::ROW_B)
                    bf[cb] = lp_b_fragment16(stage + Cfg::A_BYTES, Cfg::B_ROWB, 16 * kc, wn * Cfg::TN + cb * 32,
                                             [](int k) { return Cfg::b_swz(k); });
                else
                    bf[cb] = *reinterpret_cast<const u32x4 *>(Bs + cb * 32 * Cfg::RS + kc * CHUNK_BYTES);
            }
            if constexpr (MODE == GEMM_MODE_F32_SPLIT_BF16X3) {
                u32x4 al[Cfg::RB], bl[Cfg::CB];
#pragma unroll
                for (int rb = 0; rb < Cfg::RB; ++rb)
                    al[rb] = *reinterpret_cast<const u32x4 *>(As + Cfg::PLANE_A + rb * 32 * Cfg::RSA +
                                                              kc * CHUNK_BYTES);
#pragma unroll
                for (int cb = 0; cb < Cfg::CB; ++cb)
                    bl[cb] = *reinterpret_cast<const u32x4 *>(Bs + Cfg::PLANE_B + cb * 32 * Cfg::RS +
                                                              kc * CHUNK_BYTES);
#pragma unroll
                for (int rb = 0; rb < Cfg::RB; ++rb)
#pragma unroll
                    for (int cb = 0; cb < Cfg::CB; ++cb) {
                        const bf16x8 ah = __builtin_bit_cast(bf16x8, af[rb]);
                        const bf16x8 alo = __builtin_bit_cast(bf16x8, al[rb]);
                        const bf16x8 bh = __builtin_bit_cast(bf16x8, bf[cb]);
                        const bf16x8 blo = __builtin_bit_cast(bf16x8, bl[cb]);
                        f32x16 c = acc[rb][cb];
                        c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(alo, bh, c, 0, 0, 0);
                        c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah, blo, c, 0, 0, 0);
                        c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah, bh, c, 0, 0, 0);
                        acc[rb][cb] = c;
                    }
            } else if constexpr (MODE == GEMM_MODE_BF16) {
#pragma unroll
                for (int rb = 0; rb < Cfg::RB; ++rb)
#pragma unroll
                    for (int cb = 0; cb < Cfg::CB; ++cb)
                        acc[rb][cb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                            __builtin_bit_cast(bf16x8, af[rb]), __builtin_bit_cast(bf16x8, bf[cb]), acc[rb][cb], 0,
                            0, 0);
            } else {
#pragma unroll
                for (int rb = 0; rb < Cfg::RB; ++rb)
#pragma unroll
                    for (int cb = 0; cb < Cfg::CB; ++cb)
                        acc[rb][cb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(
                            __builtin_bit_cast(f16x8, af[rb]), __builtin_bit_cast(f16x8, bf[cb]), acc[rb][cb], 0,
                            0, 0);
            }
        }
    }
}

// One BM x BN output tile over the k-tiles of split `split`.
template <class Cfg>
__device__ __forceinline__ void lp_tile(const TileProblem &P, int tm, int tn, int split, uint8_t *lds) {
    const int m0 = tm * Cfg::BM, n0 = tn * Cfg::BN;
    const int nkt = (P.k + Cfg::BK - 1) / Cfg::BK;
    const int kt0 = split * P.kt_per_split;
    const int kt1 = min(kt0 + P.kt_per_split, nkt);

    f32x16 acc[Cfg::RB][Cfg::CB];
#pragma unroll
    for (int rb = 0; rb < Cfg::RB; ++rb)
#pragma unroll
        for (int cb = 0; cb < Cfg::CB; ++cb)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[rb][cb][r] = 0.f;

    LpStage<Cfg> R;
    if (kt0 < kt1) {
        lp_load_tiles<Cfg>(P, m0, n0, kt0 * Cfg::BK, R);
        lp_store_tiles<Cfg>(lds, R);
    }
    __syncthreads();
    for (int kt = kt0; kt < kt1; ++kt) {
        const int cur = (kt - kt0) & 1;
        const bool more = kt + 1 < kt1;
        if (more) lp_load_tiles<Cfg>(P, m0, n0, (kt + 1) * Cfg::BK, R);
        lp_compute_stage<Cfg>(lds + cur * Cfg::STAGE, acc);
        if (more) lp_store_tiles<Cfg>(lds + (cur ^ 1) * Cfg::STAGE, R);
        __syncthreads();
    }
    float *C;
    int64_t ldc;
    float scale;
    epilogue_target(P, split, C, ldc, scale);
    if constexpr (Cfg::ROW_B) lp2_epilogue<Cfg>(C, ldc, P.m, P.n, m0, n0, scale, acc);
    else tile_epilogue<Cfg>(C, ldc, P.m, P.n, m0, n0, scale, acc);
}

template <int MODE, int BM, int BN, int BK>
__device__ __forceinline__ void LpCfg<MODE, BM, BN, BK>::run(const TileProblem &P, int tm, int tn, int split,
                                                         uint8_t *lds) {
    lp_tile<LpCfg<MODE, BM, BN, BK>>(P, tm, tn, split, lds);
}
