// Kernel templates shared by every mode: the plain launch (one output tile
// per workgroup, XCD-aware tile order) and the grouped persistent launch
// (tile_gs.hpp: workgroups walk host-scheduled tile lists over many
// problems, each problem with one of two tile configurations).
#pragma once

#include "kernels.hpp"
#include "tile_gs.hpp"

template <class Cfg, int OCC>
__global__ __launch_bounds__(Cfg::THREADS, OCC) void gemm_plain_kernel(TileProblem P) {
    __shared__ __attribute__((aligned(16))) uint8_t lds[Cfg::LDS_BYTES];
    const int per_split = P.tiles_m * P.tiles_n;
    int t = xcd_remap(blockIdx.x, gridDim.x);
    const int split = t / per_split;
    t -= split * per_split;
    int tm, tn;
    tile_coords(t, P.tiles_m, P.tiles_n, 8, tm, tn);
    Cfg::run(P, tm, tn, split, lds);
}

template <int A, int B> struct cmax { static constexpr int v = A > B ? A : B; };

// The two grouped kernels of a mode (the autotuner picks one per mode on a
// mixed batch; variant 0 unless measured otherwise): resident workgroups per
// CU and depth of the register ring (k-tiles in flight: DEPTH - 1).
//   0: one 128x128 tile, three workgroups per CU, one k-tile in flight;
//   1: two tiles (128x128 and 64x64, the cost model choosing per problem),
//      two workgroups per CU, three k-tiles in flight (FP32: one in flight).
// On the 512-problem workload variant 0 measured faster: the stream is bound
// by its per-step instructions, which more resident waves overlap, and the
// second tile's registers or a deeper ring do not fit three workgroups.
// Variant 0 keeps one k-tile in flight per workgroup where the workgroups have
// several output tiles each (512 problems of 32..1024 in bfloat16: 127 us
// against 137 with two), and two where a launch has about as many tiles as
// resident workgroups and ends with its longest k loop, whose loads nothing
// else covers: 40 problems 36 -> 30 us, 151 (1.3 tiles per workgroup) 42 -> 38,
// 200 (1.6) 48 -> 43, level at 2.5; split-BF16x3 40 problems 72 -> 59; E4M3
// 25.6 -> 22.3, level at 1.6.  FP32, bound by its matrix pipe, gains nothing.
constexpr int GROUPED_ONE_OCC = 3, GROUPED_ONE_DEPTH = 2;
constexpr double GROUPED_DEEP_16 = 2.0, GROUPED_DEEP_8 = 1.5;
// A launch of few 128x128 tiles runs on 64x64 tiles instead (four workgroups
// per CU, two k-tiles in flight): one workgroup per CU cannot cover a step's
// own chain of loads, LDS and MFMAs, four smaller ones do.  The lines are in
// 128x128 tiles per CU, where a call's time stops gaining; a fuller launch
// loses to the padding it saves less of and to the host's four times as many
// schedule entries.  A call (us), 128x128 / 64x64: FP32 29 tiles 80 / 34, 324
// tiles 95 / 48, 1266 tiles 153 / 128, level near 1900; split-BF16x3 29 tiles
// 56 / 29, 464 tiles 63 / 38, level near 1000; bfloat16 29 tiles 27 / 16, 238
// tiles 32 / 25, 464 tiles 33 / 35; E4M3 125 tiles 39 / 28, 238 tiles 22 / 25.
constexpr int GROUPED_SMALL_OCC = 4, GROUPED_SMALL_DEPTH = 3;
constexpr double GROUPED_SMALL_F32 = 5.0, GROUPED_SMALL_SPLIT = 2.5, GROUPED_SMALL_16 = 1.0, GROUPED_SMALL_8 = 0.6;
constexpr int GROUPED_TWO_OCC = 2, GROUPED_TWO_DEPTH = 4;

template <class Cfg, int OCC>
static hipError_t launch_plain_t(const TileProblem &P, int nwg, hipStream_t s) {
    hipLaunchKernelGGL((gemm_plain_kernel<Cfg, OCC>), dim3(nwg), dim3(Cfg::THREADS), 0, s, P);
    return hipGetLastError();
}

template <class Cfg0, class Cfg1, int OCC, int DEPTH>
static hipError_t launch_grouped_t(const GroupedArgs &G, int nwg, hipStream_t s) {
    hipLaunchKernelGGL((gemm_grouped_stream_kernel<Cfg0, Cfg1, OCC, DEPTH>), dim3(nwg), dim3(GEMM_THREADS), 0, s,
                       G.descs, G.tiles, G.wg_first);
    return hipGetLastError();
}

// A grouped kernel's table entry: its resident workgroups per CU are the
// launch bound, capped by what fits in the CU's 160 KiB of LDS (two stages
// of the larger tile); alone0 / alone1 are the larger and the smaller plain
// configuration a problem launched on its own may take.
template <class Cfg0, class Cfg1, int OCC, int DEPTH>
constexpr GroupedKernel make_grouped(int cfg0, int cfg1, int alone0, int alone1) {
    return GroupedKernel{{cfg0, cfg1},
                         {alone0, alone1},
                         (160 * 1024 / (2 * GsRing<Cfg0, Cfg1>::STAGE)) < OCC
                             ? (160 * 1024 / (2 * GsRing<Cfg0, Cfg1>::STAGE))
                             : OCC,
                         2 * GsRing<Cfg0, Cfg1>::STAGE,
                         launch_grouped_t<Cfg0, Cfg1, OCC, DEPTH>,
                         nullptr,
                         0.0,
                         nullptr,
                         0,
                         0,
                         0.0};
}

// A one-tile grouped kernel with its deeper form (see GROUPED_ONE_DEPTH;
// deep_below 0: none) and its smaller tile's kernel; `alone1` is that tile's
// index in the plain table.
template <class Cfg, class Small>
constexpr GroupedKernel make_grouped_one(int cfg, int alone0, int alone1, double deep_below, double small_below) {
    GroupedKernel g = make_grouped<Cfg, Cfg, GROUPED_ONE_OCC, GROUPED_ONE_DEPTH>(cfg, cfg, alone0, alone1);
    if (deep_below > 0.0) g.launch_deep = launch_grouped_t<Cfg, Cfg, GROUPED_ONE_OCC, GROUPED_ONE_DEPTH + 1>;
    g.deep_below = deep_below;
    g.launch_small = launch_grouped_t<Small, Small, GROUPED_SMALL_OCC, GROUPED_SMALL_DEPTH>;
    g.small_idx = alone1;
    g.small_per_cu = (160 * 1024 / (2 * GsRing<Small, Small>::STAGE)) < GROUPED_SMALL_OCC
                         ? (160 * 1024 / (2 * GsRing<Small, Small>::STAGE))
                         : GROUPED_SMALL_OCC;
    g.small_below = small_below;
    return g;
}

template <class Cfg, int OCC, int CHUNK = 0, int PRESPLIT = 0>
constexpr KernelCfg make_cfg() {
    return KernelCfg{Cfg::BM, Cfg::BN, Cfg::BK, Cfg::THREADS / 64, Cfg::LDS_BYTES, Cfg::MFMA_K,
                     (160 * 1024 / Cfg::LDS_BYTES) < OCC ? (160 * 1024 / Cfg::LDS_BYTES) : OCC,
                     launch_plain_t<Cfg, OCC>, CHUNK, PRESPLIT, 0};
}

// The table entry of a tile whose waves run the k ranges of the split factor
// (Lp2Cfg with WK).  OCC: waves per SIMD.
template <class Cfg, int OCC, int CHUNK = 0>
constexpr KernelCfg make_fused() {
    return KernelCfg{Cfg::BM, Cfg::BN, Cfg::BK, Cfg::WK, Cfg::LDS_BYTES, Cfg::MFMA_K,
                     (160 * 1024 / Cfg::LDS_BYTES) < 4 * OCC / Cfg::WK ? (160 * 1024 / Cfg::LDS_BYTES)
                                                                       : (4 * OCC / Cfg::WK),
                     launch_plain_t<Cfg, OCC>, CHUNK, 0, Cfg::WK};
}
