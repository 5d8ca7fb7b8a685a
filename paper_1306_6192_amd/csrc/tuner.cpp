// Tile-configuration autotuner: tables of (config, split-K) choices for plain
// launches and of tile choices for grouped launches, filled by measurement on
// the device (gemm_tune, gemm_tune_bucket, gemm_tune_grouped) and consulted
// before a cost model.  Plain choices are keyed by the exact (mode, m, n, k)
// or, failing that, by its log2 bucket (floor(log2) of each dimension), so
// shapes never measured still get a measured choice of a neighbouring shape;
// grouped choices are keyed by bucket.  Every choice depends on (mode, m, n,
// k) only, never on load, so a shape gets the same configuration -- and
// therefore the same summation order -- on every path.
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <tuple>
#include <vector>

#include "host.hpp"

namespace mg {

typedef std::tuple<int, int64_t, int64_t, int64_t> Key;
typedef std::tuple<int, int, int, int> BKey;   // mode, log2 buckets of m, n, k

static std::mutex g_mu;
static std::map<Key, std::pair<int, int>> g_table;          // exact shape -> (cfg, split)
static std::map<BKey, std::pair<int, int>> g_plain_bucket;  // bucket -> (cfg, split)
static std::map<BKey, int> g_grouped;                       // bucket -> option alone
static double g_grouped_eff[GEMM_NUM_MODES] = {-1, -1, -1, -1, -1};   // small-tile efficiency (< 0: unset)
static int g_grouped_variant[GEMM_NUM_MODES] = {-1, -1, -1, -1, -1};  // grouped kernel variant (< 0: unset)
static bool g_env_loaded = false;

// The measured grid: the choice at every combination of the points 32, 48, 64,
// 96, ... 8192 (2^b and 1.5 2^b) of m, n and k, for shapes of whole 16-byte
// chunks (split-BF16x3: n a multiple of 8) and for ragged ones.  A shape takes
// the choice of the nearest points (in log distance; dimensions beyond the
// ends take the end).  Measured per point because the best tile turns with
// each factor of 1.4: on 5000 drawn shapes the choices by log2 bucket and cost
// model were 1.3 to 2.1 times slower (geometric means by mode) than the best
// configuration, those of the nearest of 500 measured shapes 1.02 to 1.08.
constexpr int GRID_POINTS = 17;
struct GridChoice {
    int16_t cfg = -1, split = 1;
};
static GridChoice g_grid[GEMM_NUM_MODES][2][GRID_POINTS][GRID_POINTS][GRID_POINTS];

int dim_bucket(int64_t d) {
    int b = 0;
    while (d > 1) {
        d >>= 1;
        ++b;
    }
    return b;
}

// Index of the grid point nearest to d: 2^b up to sqrt(1.5) 2^b, 1.5 2^b up to
// sqrt(3) 2^b, then 2^(b+1).
static int grid_point(int64_t d) {
    if (d <= 32) return 0;
    const int b = dim_bucket(d);
    if (b >= 13) return GRID_POINTS - 1;
    const int64_t sq = d * d, base = (int64_t)1 << (2 * b);
    return 2 * (b - 5) + (2 * sq < 3 * base ? 0 : sq < 3 * base ? 1 : 2);
}

static int64_t point_dim(int i) { return (int64_t)(i % 2 ? 3 : 2) << (4 + i / 2); }

// Whether k and n are whole 16-byte chunks of the mode's asynchronous-copy
// tiles (split-BF16x3: whether n is, for its operand copies).
static int grid_class(int mode, int64_t n, int64_t k) {
    if (mode == GEMM_MODE_F32_SPLIT_BF16X3) return n % 8 == 0;
    const int64_t c = 16 / (int64_t)elem_size(mode);
    return k % c == 0 && n % c == 0;
}

static BKey bucket_of(int mode, int64_t m, int64_t n, int64_t k) {
    return BKey(mode, dim_bucket(m), dim_bucket(n), dim_bucket(k));
}

static int load_file_locked(const char *path);

// Relative sustained efficiency of a workgroup tile (larger tiles reuse each
// staged operand more often and hide the per-k-tile barrier better).
static double tile_eff(const KernelCfg &kc) {
    const double area = (double)kc.bm * kc.bn;
    if (area >= 65536) return 1.00;
    if (area >= 32768) return 0.92;
    if (area >= 16384) return 0.82;
    if (area >= 8192) return 0.62;
    return 0.45;
}

void heuristic_choose(int mode, int64_t m, int64_t n, int64_t k, int *cfg_out, int *split_out) {
    int count = 0;
    const KernelCfg *t = configs(mode, &count);
    *cfg_out = 0;
    *split_out = 1;
    if (!t || count == 0 || m == 0 || n == 0 || k == 0) return;
    const double cus = (double)num_cus();
    double best = 1e300;
    for (int c = 0; c < count; ++c) {
        const KernelCfg &kc = t[c];
        // chunked (asynchronous-copy) tiles need k and n in whole 16-byte
        // chunks; where they apply they sustain 1.4x (16-bit) to 3.5x (FP8),
        // and 1.1x (FP32) the register-staged tile's rate at 8192^3
        // the tiles with waves along k are chosen by measurement only
        if (kc.fused) continue;
        if (kc.chunk && (k % kc.chunk || n % kc.chunk)) continue;
        if (kc.presplit && !presplit_shape_ok(n, k)) continue;
        // the pre-split split-BF16x3 path runs at about 1.8x the register-
        // staged split tile at 8192^3 (its operands are split once, not once
        // per output tile)
        double bonus = kc.presplit ? 1.8 : 1.0;
        if (kc.chunk) bonus = mode == GEMM_MODE_F32 ? 1.1 : 1.7;
        const int64_t tiles = ((m + kc.bm - 1) / kc.bm) * ((n + kc.bn - 1) / kc.bn);
        const int64_t nkt = (k + split_grain(mode) - 1) / split_grain(mode) * (split_grain(mode) / kc.bk);
        for (int split = 1; split <= 16; split *= 2) {
            if (split > 1 && nkt / split < 4) break;
            const int64_t per = (nkt + split - 1) / split;
            const int64_t wgs = tiles * split;
            const double slots = cus * std::max(1, kc.wg_per_cu);
            const double rounds = std::ceil((double)wgs / slots);
            // time ~ rounds * (work of one CU slot-set) / efficiency
            const double per_round = (double)std::max(1, kc.wg_per_cu) * kc.bm * kc.bn * (double)(per * kc.bk);
            double cost = rounds * per_round / (tile_eff(kc) * bonus);
            // split-K pays for writing and re-reading the partial slabs
            if (split > 1) cost += (double)(split + 1) * (double)m * n * 64.0 / cus;
            // a launch that cannot reach every CU also leaves HBM bandwidth idle
            if ((double)wgs < cus) cost *= 1.0 + 0.25 * (1.0 - (double)wgs / cus);
            if (cost < best * 0.999) {
                best = cost;
                *cfg_out = c;
                *split_out = split;
            }
        }
    }
}

static void load_env_locked() {
    if (g_env_loaded) return;
    g_env_loaded = true;
    const char *env = getenv("MI355GEMM_TUNE_FILE");
    if (env && *env) (void)load_file_locked(env);
}

static GridChoice grid_at(int mode, int cl, int im, int in, int ik) {
    GridChoice c = g_grid[mode][cl][im][in][ik];
    // binary16 runs on the same tiles as bfloat16, at the same rates
    if (c.cfg < 0 && mode == GEMM_MODE_F16) c = g_grid[GEMM_MODE_BF16][cl][im][in][ik];
    return c;
}

// The k ranges that a split factor gives (make_launch), with slabs of at most
// 64 MB, as at the measured points: larger products of a point's range take
// fewer ranges (147x7866x7815 in split-BF16x3 with 14 of its point's 16: 186 us;
// with one, 606).
static int bounded_split(const KernelCfg &kc, int64_t m, int64_t n, int split) {
    const int in_wg = std::max(1, kc.fused);
    const int64_t slab = ((m * n + 3) / 4 * 4) * 4;
    return split > in_wg && split * slab > 67108864 ? std::max(in_wg, (int)(67108864 / slab)) : split;
}

static int64_t k_ranges(int mode, int64_t k, int split) {
    const int64_t grains = std::max<int64_t>(1, (k + split_grain(mode) - 1) / split_grain(mode));
    const int64_t per = (grains + std::min<int64_t>(split, grains) - 1) / std::min<int64_t>(split, grains);
    return (grains + per - 1) / per;
}

// Workgroups over those that are resident at once.
static double rounds_of(const KernelCfg &kc, int64_t m, int64_t n, int64_t ranges) {
    const double tiles = (double)((m + kc.bm - 1) / kc.bm) * (double)((n + kc.bn - 1) / kc.bn);
    return tiles * (double)(kc.fused ? (ranges + kc.fused - 1) / kc.fused : ranges) /
           ((double)num_cus() * std::max(1, kc.wg_per_cu));
}

void tuner_choose(int mode, int64_t m, int64_t n, int64_t k, int *cfg, int *split) {
    {
        std::lock_guard<std::mutex> lk(g_mu);
        load_env_locked();
        auto it = g_table.find(Key(mode, m, n, k));
        if (it != g_table.end()) {
            *cfg = it->second.first;
            *split = it->second.second;
            return;
        }
        auto ib = g_plain_bucket.find(bucket_of(mode, m, n, k));
        if (ib != g_plain_bucket.end()) {
            *cfg = ib->second.first;
            *split = ib->second.second;
            return;
        }
        if (mode_known(mode)) {
            const int cl = grid_class(mode, n, k), im = grid_point(m), in = grid_point(n), ik = grid_point(k);
            const GridChoice c = grid_at(mode, cl, im, in, ik);
            if (c.cfg >= 0) {
                int count = 0;
                const KernelCfg *t = configs(mode, &count);
                *cfg = c.cfg;
                *split = bounded_split(t[c.cfg], m, n, c.split);
                // A shape just above its point may need one more, mostly empty
                // round of workgroups than the point did (up to 1.6 rounds; 2 and
                // more gain nothing).  It takes the configuration of the next
                // point along the dimension in which it is further above, if
                // that has fewer rounds here, the same k ranges (so the same
                // bits) and another tile.  119 of 9000 drawn shapes (m, n, k of
                // 32..4096, and 1..256 by 1024..8192) do: 0.80 of their time on
                // average, one more than 1.07 (E4M3 3046x147x115 10.5 -> 6.2 us,
                // FP32 2305x3990x3498 846 -> 651; 572x580x2397 29.4 -> 35.8).
                // With other ranges or along both dimensions: up
                // to 1.4 and 2.9 times slower.  Split-BF16x3's points stay level.
                const int64_t ranges = k_ranges(mode, k, *split);
                const double here = rounds_of(t[c.cfg], m, n, ranges);
                const double above_m = (double)m / point_dim(im), above_n = (double)n / point_dim(in);
                const bool by_m = above_m >= above_n;
                if (mode != GEMM_MODE_F32_SPLIT_BF16X3 && here <= 1.6 && std::max(above_m, above_n) > 1.0 &&
                    (by_m ? im : in) + 1 < GRID_POINTS &&
                    std::ceil(here) > std::ceil(rounds_of(t[c.cfg], point_dim(im), point_dim(in), ranges))) {
                    const GridChoice up = grid_at(mode, cl, im + by_m, in + !by_m, ik);
                    const int up_split = up.cfg >= 0 ? bounded_split(t[up.cfg], m, n, up.split) : 0;
                    if (up.cfg >= 0 && rounds_of(t[up.cfg], m, n, ranges) < here && k_ranges(mode, k, up_split) == ranges &&
                        (t[up.cfg].bm != t[c.cfg].bm || t[up.cfg].bn != t[c.cfg].bn || t[up.cfg].waves != t[c.cfg].waves)) {
                        *cfg = up.cfg;
                        *split = up_split;
                    }
                }
                return;
            }
        }
    }
    heuristic_choose(mode, m, n, k, cfg, split);
}

bool tuner_grouped_alone(int mode, int64_t m, int64_t n, int64_t k, int *alone) {
    std::lock_guard<std::mutex> lk(g_mu);
    load_env_locked();
    auto it = g_grouped.find(bucket_of(mode, m, n, k));
    if (it == g_grouped.end()) return false;
    *alone = it->second;
    return true;
}

void tuner_record_grouped(int mode, int64_t m, int64_t n, int64_t k, int alone) {
    std::lock_guard<std::mutex> lk(g_mu);
    g_grouped[bucket_of(mode, m, n, k)] = alone;
}

double tuner_grouped_eff(int mode) {
    std::lock_guard<std::mutex> lk(g_mu);
    load_env_locked();
    return mode_known(mode) ? g_grouped_eff[mode] : -1.0;
}

void tuner_record_grouped_eff(int mode, double eff, int variant) {
    std::lock_guard<std::mutex> lk(g_mu);
    if (!mode_known(mode)) return;
    g_grouped_eff[mode] = eff;
    g_grouped_variant[mode] = variant;
}

int tuner_grouped_variant(int mode) {
    std::lock_guard<std::mutex> lk(g_mu);
    load_env_locked();
    return mode_known(mode) && g_grouped_variant[mode] >= 0 ? g_grouped_variant[mode] : 0;
}

// One JSON object per line, in one of five forms (the forms gemm_tuner_save
// writes; lines in any other form are skipped):
//   {"mode": M, "m": m, "n": n, "k": k, "cfg": C, "split": S}
//   {"bucket": "plain", "mode": M, "bm": a, "bn": b, "bk": c, "cfg": C, "split": S}
//   {"bucket": "grouped", "mode": M, "bm": a, "bn": b, "bk": c, "alone": U}
//   {"grouped_eff": M, "eff": E, "variant": V}  (", variant" optional: 0)
//   {"grid": M, "whole": W, "m": i, "n": j, "choices": "C:S C:S ..."}
//     (grid point indices i of m and j of n; one choice per point of k)
static int load_file_locked(const char *path) {
    FILE *f = fopen(path, "r");
    if (!f) return fail(GEMM_ENOTFOUND, "cannot open tuning file %s", path);
    char line[512];
    int n_ok = 0;
    while (fgets(line, sizeof(line), f)) {
        int mode, cfg, split, bm, bn, bk;
        long long m, n, k;
        int count = 0;
        int at = 0;
        if (sscanf(line, " {\"grid\": %d, \"whole\": %d, \"m\": %d, \"n\": %d, \"choices\": \"%n", &mode, &split, &bm, &bn,
                   &at) == 4 &&
            at > 0) {
            if (!mode_known(mode) || split < 0 || split > 1 || bm < 0 || bm >= GRID_POINTS || bn < 0 || bn >= GRID_POINTS)
                continue;
            configs(mode, &count);
            const char *c = line + at;
            for (int i = 0; i < GRID_POINTS; ++i) {
                char *end = nullptr;
                const long cf = strtol(c, &end, 10);
                if (end == c || *end != ':') break;
                c = end + 1;
                const long sp = strtol(c, &end, 10);
                if (end == c) break;
                c = end;
                if (cf < 0 || cf >= count || sp < 1 || sp > 4096) continue;
                g_grid[mode][split][bm][bn][i].cfg = (int16_t)cf;
                g_grid[mode][split][bm][bn][i].split = (int16_t)sp;
                ++n_ok;
            }
        } else if (sscanf(line, " {\"mode\": %d, \"m\": %lld, \"n\": %lld, \"k\": %lld, \"cfg\": %d, \"split\": %d",
                   &mode, &m, &n, &k, &cfg, &split) == 6) {
            if (!mode_known(mode)) continue;
            configs(mode, &count);
            if (cfg >= 0 && cfg < count && split >= 1) {
                g_table[Key(mode, m, n, k)] = {cfg, split};
                ++n_ok;
            }
        } else if (sscanf(line,
                          " {\"bucket\": \"plain\", \"mode\": %d, \"bm\": %d, \"bn\": %d, \"bk\": %d, "
                          "\"cfg\": %d, \"split\": %d",
                          &mode, &bm, &bn, &bk, &cfg, &split) == 6) {
            if (!mode_known(mode)) continue;
            configs(mode, &count);
            if (cfg >= 0 && cfg < count && split >= 1) {
                g_plain_bucket[BKey(mode, bm, bn, bk)] = {cfg, split};
                ++n_ok;
            }
        } else if (sscanf(line,
                          " {\"bucket\": \"grouped\", \"mode\": %d, \"bm\": %d, \"bn\": %d, \"bk\": %d, "
                          "\"alone\": %d",
                          &mode, &bm, &bn, &bk, &cfg) == 5 ||
                   sscanf(line,
                          " {\"bucket\": \"grouped\", \"mode\": %d, \"bm\": %d, \"bn\": %d, \"bk\": %d, "
                          "\"tile\": %d, \"alone\": %d",
                          &mode, &bm, &bn, &bk, &split, &cfg) == 6) {
            // (the second form also carries an in-batch tile, which the
            // calibrated cost model now decides; only the alone choice is kept)
            if (!mode_known(mode) || cfg < 0 || cfg > 1) continue;
            g_grouped[BKey(mode, bm, bn, bk)] = cfg;
            ++n_ok;
        } else {
            double eff = 0;
            int variant = 0;
            const int got = sscanf(line, " {\"grouped_eff\": %d, \"eff\": %lf, \"variant\": %d", &mode, &eff,
                                   &variant);
            if (got >= 2 && mode_known(mode) && eff > 0 && eff <= 4 && variant >= 0 && variant <= 1) {
                g_grouped_eff[mode] = eff;
                g_grouped_variant[mode] = got == 3 ? variant : 0;
                ++n_ok;
            }
        }
    }
    fclose(f);
    return n_ok;
}

// Time one (cfg, split) choice: median of `reps` event-timed launches.
static int time_choice(const gemm_problem_t &p, int cfg, int split, void *ws, hipStream_t s, float *ms_out) {
    hipEvent_t e0, e1;
    MG_HIP(hipEventCreate(&e0));
    MG_HIP(hipEventCreate(&e1));
    const int reps = 5;
    float ts[reps];
    int rc = enqueue_plain(p, cfg, split, ws, s, true);  // warm-up
    for (int r = 0; r < reps && rc == GEMM_OK; ++r) {
        (void)hipEventRecord(e0, s);
        rc = enqueue_plain(p, cfg, split, ws, s, true);
        (void)hipEventRecord(e1, s);
        if (hipEventSynchronize(e1) != hipSuccess) rc = fail(GEMM_EHIP, "event sync failed");
        (void)hipEventElapsedTime(&ts[r], e0, e1);
    }
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    if (rc != GEMM_OK) return rc;
    std::sort(ts, ts + reps);
    *ms_out = ts[reps / 2];
    return GEMM_OK;
}

}  // namespace mg

using namespace mg;

extern "C" {

int gemm_tuner_lookup(int32_t mode, int64_t m, int64_t n, int64_t k, int32_t *cfg, int32_t *split_k) {
    clear_error();
    if (!mode_known(mode)) return fail(GEMM_EINVAL, "unknown mode %d", mode);
    if (!cfg || !split_k) return fail(GEMM_EINVAL, "NULL output");
    if (m < 0 || n < 0 || k < 0) return fail(GEMM_EINVAL, "negative dimension");
    int c = 0, s = 1;
    tuner_choose(mode, m, n, k, &c, &s);
    *cfg = c;
    *split_k = s;
    return GEMM_OK;
}

int gemm_tuner_load(const char *path) {
    clear_error();
    if (!path) return fail(GEMM_EINVAL, "path is NULL");
    std::lock_guard<std::mutex> lk(g_mu);
    const int rc = load_file_locked(path);
    return rc < 0 ? rc : GEMM_OK;
}

int gemm_tuner_save(const char *path) {
    clear_error();
    if (!path) return fail(GEMM_EINVAL, "path is NULL");
    std::lock_guard<std::mutex> lk(g_mu);
    FILE *f = fopen(path, "w");
    if (!f) return fail(GEMM_ENOTFOUND, "cannot write %s", path);
    for (auto &kv : g_table) {
        fprintf(f, "{\"mode\": %d, \"m\": %lld, \"n\": %lld, \"k\": %lld, \"cfg\": %d, \"split\": %d}\n",
                std::get<0>(kv.first), (long long)std::get<1>(kv.first), (long long)std::get<2>(kv.first),
                (long long)std::get<3>(kv.first), kv.second.first, kv.second.second);
    }
    for (auto &kv : g_plain_bucket)
        fprintf(f,
                "{\"bucket\": \"plain\", \"mode\": %d, \"bm\": %d, \"bn\": %d, \"bk\": %d, \"cfg\": %d, "
                "\"split\": %d}\n",
                std::get<0>(kv.first), std::get<1>(kv.first), std::get<2>(kv.first), std::get<3>(kv.first),
                kv.second.first, kv.second.second);
    for (int mode = 0; mode < GEMM_NUM_MODES; ++mode)
        for (int whole = 0; whole < 2; ++whole)
            for (int i = 0; i < GRID_POINTS; ++i)
                for (int j = 0; j < GRID_POINTS; ++j) {
                    const GridChoice *row = g_grid[mode][whole][i][j];
                    int known = 0;
                    for (int q = 0; q < GRID_POINTS; ++q) known += row[q].cfg >= 0;
                    if (!known) continue;
                    fprintf(f, "{\"grid\": %d, \"whole\": %d, \"m\": %d, \"n\": %d, \"choices\": \"", mode, whole, i, j);
                    for (int q = 0; q < GRID_POINTS; ++q)   // (a point not measured: -1:1, skipped on loading)
                        fprintf(f, "%s%d:%d", q ? " " : "", row[q].cfg, row[q].split);
                    fprintf(f, "\"}\n");
                }
    for (auto &kv : g_grouped)
        fprintf(f, "{\"bucket\": \"grouped\", \"mode\": %d, \"bm\": %d, \"bn\": %d, \"bk\": %d, \"alone\": %d}\n",
                std::get<0>(kv.first), std::get<1>(kv.first), std::get<2>(kv.first), std::get<3>(kv.first),
                kv.second);
    for (int m = 0; m < GEMM_NUM_MODES; ++m)
        if (g_grouped_eff[m] > 0)
            fprintf(f, "{\"grouped_eff\": %d, \"eff\": %.3f, \"variant\": %d}\n", m, g_grouped_eff[m],
                    std::max(0, g_grouped_variant[m]));
    fclose(f);
    return GEMM_OK;
}

}  // extern "C"

namespace mg {

// Time every legal (configuration, split) of one shape; *cfg_out gets the
// fastest, *split_out its requested split factor and *norm_split_out the
// factor make_launch normalises it to for this shape.
static int tune_plain(int32_t mode, int64_t m, int64_t n, int64_t k, void *stream, int *cfg_out, int *split_out,
                      int *norm_split_out) {
    if (!mode_known(mode)) return fail(GEMM_EINVAL, "unknown mode %d", mode);
    if (m <= 0 || n <= 0 || k <= 0) return fail(GEMM_EINVAL, "tuning needs a non-empty product");
    int count = 0;
    const KernelCfg *t = configs(mode, &count);
    if (!t || count == 0) return fail(GEMM_EUNSUPPORTED, "mode %d has no kernels", mode);
    hipStream_t s = (hipStream_t)stream;
    const size_t es = elem_size(mode);
    void *A = nullptr, *B = nullptr, *C = nullptr, *ws = nullptr;
    int64_t ws_need = 0;
    gemm_problem_t p;
    memset(&p, 0, sizeof(p));
    p.mode = mode;
    p.m = m;
    p.n = n;
    p.k = k;
    p.lda = k;
    p.ldb = n;
    p.ldc = n;
    p.scale_a = p.scale_b = 1.f;
    for (int c = 0; c < count; ++c)
        for (int sp = 1; sp <= 16; sp *= 2) ws_need = std::max(ws_need, plain_ws_bytes(p, c, sp, true));
    int rc = GEMM_OK;
    if (hipMalloc(&A, (size_t)m * k * es) != hipSuccess || hipMalloc(&B, (size_t)k * n * es) != hipSuccess ||
        hipMalloc(&C, (size_t)m * n * 4) != hipSuccess ||
        (ws_need > 0 && hipMalloc(&ws, (size_t)ws_need) != hipSuccess)) {
        (void)hipGetLastError();
        rc = fail(GEMM_ENOMEM, "tuning buffers do not fit");
    }
    int best_c = 0, best_s = 1, best_req = 1;
    float best_ms = 1e30f;
    struct Cand {
        int cfg, split;
        float ms;
    };
    std::vector<Cand> cands;
    if (rc == GEMM_OK) {
        // non-zero operands: the clock under load depends on the data
        if (launch_fill_tuning(A, m * k, (int)es, 1u, s) != hipSuccess ||
            launch_fill_tuning(B, k * n, (int)es, 2u, s) != hipSuccess)
            rc = fail(GEMM_EHIP, "filling the tuning operands failed");
        p.A = A;
        p.B = B;
        p.C = static_cast<float *>(C);
        for (int c = 0; c < count && rc == GEMM_OK; ++c) {
            if (!cfg_runs(p, t[c])) continue;
            const int64_t nkt = (k + split_grain(mode) - 1) / split_grain(mode);
            int last_split = 0;
            for (int sp = 1; sp <= 16 && rc == GEMM_OK; sp *= 2) {
                if (sp > 1 && nkt / sp < (t[c].fused ? 1 : 4)) break;
                const int eff = make_launch(p, t[c], sp).splits;
                if (eff == last_split) continue;
                last_split = eff;
                float ms = 0.f;
                rc = time_choice(p, c, sp, ws, s, &ms);
                if (rc == GEMM_OK) cands.push_back({c, sp, ms});
            }
        }
    }
    // Candidates within 3 % of the fastest are timed again, three rounds in
    // turn, and the lowest sum of the four medians wins: a single median
    // cannot tell choices that close apart.
    if (rc == GEMM_OK && !cands.empty()) {
        float first = 1e30f;
        for (const Cand &c : cands) first = std::min(first, c.ms);
        std::vector<Cand> close;
        for (const Cand &c : cands)
            if (c.ms <= first * 1.03f) close.push_back(c);
        for (int round = 0; round < 3 && close.size() > 1 && rc == GEMM_OK; ++round)
            for (Cand &c : close) {
                float ms = 0.f;
                rc = time_choice(p, c.cfg, c.split, ws, s, &ms);
                c.ms += ms;
                if (rc != GEMM_OK) break;
            }
        for (const Cand &c : close)
            if (c.ms < best_ms) {
                best_ms = c.ms;
                best_c = c.cfg;
                best_req = c.split;
                best_s = make_launch(p, t[c.cfg], c.split).splits;
            }
    }
    if (A) (void)hipFree(A);
    if (B) (void)hipFree(B);
    if (C) (void)hipFree(C);
    if (ws) (void)hipFree(ws);
    if (rc != GEMM_OK) return rc;
    *cfg_out = best_c;
    *split_out = best_req;
    *norm_split_out = best_s;
    return GEMM_OK;
}

}  // namespace mg

extern "C" {

int gemm_tune(int32_t mode, int64_t m, int64_t n, int64_t k, void *stream) {
    clear_error();
    int cfg = 0, req = 1, split = 1;
    const int rc = tune_plain(mode, m, n, k, stream, &cfg, &req, &split);
    if (rc != GEMM_OK) return rc;
    std::lock_guard<std::mutex> lk(g_mu);
    g_table[Key(mode, m, n, k)] = {cfg, split};
    return GEMM_OK;
}

int gemm_tune_bucket(int32_t mode, int64_t m, int64_t n, int64_t k, void *stream) {
    clear_error();
    int cfg = 0, req = 1, split = 1;
    const int rc = tune_plain(mode, m, n, k, stream, &cfg, &req, &split);
    if (rc != GEMM_OK) return rc;
    std::lock_guard<std::mutex> lk(g_mu);
    g_plain_bucket[bucket_of(mode, m, n, k)] = {cfg, req};
    return GEMM_OK;
}

}  // extern "C"
