// Split-BF16x3 product kernels: float32 operands split into bfloat16 hi/lo
// planes at staging (two planes per operand in LDS, so the largest tile is
// 256 x 128), and tiles on operands split once beforehand.
#include <iterator>
#include <vector>

#include "kernels_impl.hpp"
#include "tile_lp.hpp"
#include "tile_lp2.hpp"

static const KernelCfg kTable[] = {
    make_cfg<LpCfg<GEMM_MODE_F32_SPLIT_BF16X3, 256, 128>, 1>(), make_cfg<LpCfg<GEMM_MODE_F32_SPLIT_BF16X3, 128, 256>, 1>(),
    make_cfg<LpCfg<GEMM_MODE_F32_SPLIT_BF16X3, 128, 128>, 2>(), make_cfg<LpCfg<GEMM_MODE_F32_SPLIT_BF16X3, 128, 64>, 2>(),
    make_cfg<LpCfg<GEMM_MODE_F32_SPLIT_BF16X3, 64, 128>, 2>(),  make_cfg<LpCfg<GEMM_MODE_F32_SPLIT_BF16X3, 64, 64>, 4>(),
};

// The table entry of an asynchronous-copy tile on the operand copies (any
// shape: the copies are padded); its k-tile is half as many k as elements.
template <class Cfg, int OCC>
static KernelCfg presplit() {
    KernelCfg k = make_cfg<Cfg, OCC, 0, 1>();
    k.bk /= 2;
    return k;
}
template <class Cfg, int OCC>
static KernelCfg presplit_fused() {
    KernelCfg k = make_fused<Cfg, OCC>();
    k.bk /= 2;
    k.presplit = 1;
    return k;
}

// (BM, BN, LDS stages, waves along m and n, bytes of an A row: 64 = 16 k, 128 =
// 32 k; waves along k)
template <int BM, int BN, int STAGES, int WM = 2, int WN = 2, int AROWB = 64, int WK = 0>
using Spl = Lp2Cfg<GEMM_MODE_F32_SPLIT_BF16X3, BM, BN, STAGES, WM, WN, AROWB, 16, 32, WK>;

template <int BM, int BN, int WK>
static KernelCfg fused_reg() {
    KernelCfg k = make_fused<Lp2Cfg<GEMM_MODE_F32_SPLIT_BF16X3, BM, BN, 2, 1, 1, 64, 0, 32, WK>, 2>();
    k.bk /= 2;
    return k;
}

static const KernelCfg kPresplit[] = {
    presplit<Spl<256, 256, 4>, 1>(),
    presplit<Spl<256, 128, 4>, 1>(),
    presplit<Spl<128, 256, 4>, 1>(),
    presplit<Spl<128, 128, 4>, 2>(),
    // eight waves (two per SIMD)
    presplit<Spl<256, 256, 4, 2, 4>, 2>(),
    presplit<Spl<256, 256, 4, 4, 2>, 2>(),
    // k-tiles of 32 in two stages
    presplit<Spl<256, 128, 2, 2, 2, 128>, 1>(),
    presplit<Spl<128, 256, 2, 2, 2, 128>, 1>(),
    presplit<Spl<128, 128, 2, 2, 2, 128>, 2>(),
    // the register-staged 128 x 128 tile with k-tiles of 16 (the grouped
    // launch's large tile)
    make_cfg<LpCfg<GEMM_MODE_F32_SPLIT_BF16X3, 128, 128, 16>, 3>(),
    // waves along k
    presplit_fused<Spl<32, 64, 2, 1, 1, 64, 8>, 2>(),
    presplit_fused<Spl<64, 64, 2, 1, 1, 64, 8>, 2>(),
    // waves along k on the float32 operands themselves, split on their way into
    // LDS (any shape; no copies, one launch)
    fused_reg<32, 32, 4>(),
    fused_reg<32, 32, 8>(),
    fused_reg<32, 64, 8>(),
    fused_reg<64, 64, 8>(),
};

// The register-staged tiles (any shape), then the tiles on operand copies that
// are split once (presplit.hip); the same products in the same order, so the
// same bits.
const KernelCfg *lp_configs_split(int *count) {
    static const std::vector<KernelCfg> table = [] {
        std::vector<KernelCfg> t(std::begin(kTable), std::end(kTable));
        t.insert(t.end(), std::begin(kPresplit), std::end(kPresplit));
        return t;
    }();
    *count = (int)table.size();
    return table.data();
}

// The register-staged 128 x 128 tile with k-tiles of 16 in the table.
static int index_bk16() {
    int n = 0, at = 0;
    const KernelCfg *t = lp_configs_split(&n);
    for (int c = 0; c < n; ++c)
        if (t[c].bk == 16 && !t[c].presplit && !t[c].fused) at = c;
    return at;
}

// The grouped launches' tiles: 128 x 128 with k-tiles of 16 (in the table
// above) and, in variant 1, 64 x 64; a problem launched on its
// own takes either.
const GroupedKernel *lp_grouped_split(int variant) {
    static const GroupedKernel k[2] = {
        [] {
            GroupedKernel g =
                make_grouped_one<LpCfg<GEMM_MODE_F32_SPLIT_BF16X3, 128, 128, 16>, LpCfg<GEMM_MODE_F32_SPLIT_BF16X3, 64, 64>>(0, 0, 5, GROUPED_DEEP_16,
                                                                                     GROUPED_SMALL_SPLIT);
            g.cfg_idx[0] = g.cfg_idx[1] = g.alone_idx[0] = index_bk16();
            return g;
        }(),
        [] {
            GroupedKernel g = make_grouped<LpCfg<GEMM_MODE_F32_SPLIT_BF16X3, 128, 128, 16>,
                                           LpCfg<GEMM_MODE_F32_SPLIT_BF16X3, 64, 64>, GROUPED_TWO_OCC,
                                           GROUPED_TWO_DEPTH>(0, 5, 0, 5);
            g.cfg_idx[0] = g.alone_idx[0] = index_bk16();
            return g;
        }()};
    return &k[variant];
}
