// C ABI of libdfk: argument validation, the profile-driven scheduler and its
// table, dispatch to the VALU / MFMA launchers.  Host code only.
#include <algorithm>
#include <cstdio>
#include <cstring>
#include <map>
#include <mutex>
#include <tuple>
#include <vector>

#include "dfk_big_plan.h"
#include "dfk_internal.h"

namespace dfk {
thread_local int g_stage_mask = 3;

namespace {

thread_local int g_last_hip_error = 0;
thread_local int g_tune_skipped = 0;                  // candidates the last dfk_tune on this thread left out
thread_local dfk_status_t g_tune_skip_status = DFK_OK;  // status of the last one

dfk_status_t hip_fail(hipError_t e) {
    g_last_hip_error = (int)e;
    return DFK_ERR_HIP;
}

struct Registered {
    void* ptr = nullptr;
    size_t bytes = 0;
};
Registered g_ws;
Registered g_trace;
std::mutex g_mu;

// A consistent copy of a registered buffer: the setters write under the same lock.
Registered snapshot(const Registered& r) {
    std::lock_guard<std::mutex> lk(g_mu);
    return r;
}

// ---------------------------------------------------------------- validation
size_t elt_bytes(dfk_dtype_t d) { return d == DFK_FP32 ? 4 : 2; }

bool overlaps(const void* a, size_t na, const void* b, size_t nb) {
    const uintptr_t a0 = (uintptr_t)a, b0 = (uintptr_t)b;
    return a0 < b0 + nb && b0 < a0 + na;
}

// The shapes a call accepts: every query below and the argument check agree on it.
bool shape_supported(int M, int d_model, int d_ff) {
    return M >= 1 && M <= DFK_MAX_M && d_model >= 8 && d_model <= kMaxDModel && d_ff >= 8 && d_model % 8 == 0 && d_ff % 8 == 0;
}

bool config_valid(const dfk_config_t& c, int M, int d_model, int d_ff, dfk_dtype_t dtype) {
    if (!shape_supported(M, d_model, d_ff)) return false;
    if (c.path == DFK_PATH_VALU) return valu_config_valid(c, M, d_model, d_ff, dtype);
    if (c.path == DFK_PATH_MFMA) return mfma_config_valid(c, M, d_model, d_ff, dtype);
    return false;
}

// configurations whose down kernel takes W_down as [d_model, d_ff]
bool wdt_layout(const dfk_config_t& c) { return c.kmajor == 5; }

dfk_status_t check(const void* X, const void* Wg, const void* Wu, const void* Wd, const void* Y,
                   int M, int d_model, int d_ff, dfk_dtype_t dtype, const dfk_config_t* cfg,
                   const void* ws, size_t ws_bytes, bool need_ws, bool y_may_be_x = false, bool wd_t = false) {
    if (!X || !Wg || !Wu || !Wd || !Y) return DFK_ERR_INVALID_ARG;
    if (M < 1 || d_model < 1 || d_ff < 1) return DFK_ERR_INVALID_ARG;
    if (dtype != DFK_BF16 && dtype != DFK_FP32 && dtype != DFK_FP16) return DFK_ERR_INVALID_ARG;
    if (!shape_supported(M, d_model, d_ff)) return DFK_ERR_UNSUPPORTED_SHAPE;
    const void* ptrs[5] = {X, Wg, Wu, Wd, Y};
    for (const void* p : ptrs)
        if ((uintptr_t)p % 16) return DFK_ERR_ALIGNMENT;
    const size_t eb = elt_bytes(dtype);
    const size_t nx = (size_t)M * d_model * eb, nw = (size_t)d_ff * d_model * eb;
    if ((!(y_may_be_x && Y == X) && overlaps(Y, nx, X, nx)) || overlaps(Y, nx, Wg, nw) || overlaps(Y, nx, Wu, nw) ||
        overlaps(Y, nx, Wd, nw))
        return DFK_ERR_ALIAS;
    if (cfg) {
        if (cfg->variant != DFK_VARIANT_FUSED && cfg->variant != DFK_VARIANT_TWO_KERNEL)
            return DFK_ERR_INVALID_ARG;
        if (cfg->path != DFK_PATH_VALU && cfg->path != DFK_PATH_MFMA) return DFK_ERR_INVALID_ARG;
        if (wdt_layout(*cfg) != wd_t) return DFK_ERR_INVALID_ARG;   // the configuration is for the other layout of W_down
        if (!config_valid(*cfg, M, d_model, d_ff, dtype)) return DFK_ERR_UNSUPPORTED_SHAPE;
    }
    if (need_ws || ws || ws_bytes) {
        if (!ws) return DFK_ERR_WORKSPACE;
        if ((uintptr_t)ws % 256) return DFK_ERR_ALIGNMENT;
        if (ws_bytes < ws_layout(M, d_model, d_ff).total) return DFK_ERR_WORKSPACE;
        if (overlaps(ws, ws_bytes, Y, nx) || overlaps(ws, ws_bytes, X, nx) ||
            overlaps(ws, ws_bytes, Wg, nw) || overlaps(ws, ws_bytes, Wu, nw) ||
            overlaps(ws, ws_bytes, Wd, nw))
            return DFK_ERR_ALIAS;
    }
    return DFK_OK;
}

// ---------------------------------------------------------------- candidates and heuristic
// the single launch that holds both kernels' workgroups: variant FUSED, but partial sums and stages of the pair
bool roles_launch(const dfk_config_t& c) { return c.variant == DFK_VARIANT_FUSED && c.path == DFK_PATH_MFMA && c.kmajor == 4; }

// d_ff splits of the 64-token pair's down kernels, untuned, with `k2c` column blocks: as a rule 16 at most, because the end of
// the kernel is a chain of round trips plus the sum of the splits' blocks (one token, counter reduction: 512 x 1536 with 64
// splits 16.2 us per call, with 12 to 16 10.4; 896 x 4864 with 36 splits 18.6 us, with 16 15.6; 64 tokens: 512 x 2816 with 64
// 45.8, with 16 25.1; atomic reduction, 1024 x 5632 at 64 tokens with 32 27.3, with 16 23.0).  Where d_ff is many times d_model,
// 16 splits are long and their few workgroups leave most of the chip's bandwidth unused: more of them, of as many rows as the
// layer is wide (of twice as many for the counter reduction of more than 16 tokens, whose blocks cost the most, of three quarters
// for the atomic one, whose cost the least).  512 x 28672, counter reduction: 1 token 33.8 us with 16, 27.0 with 48, 27.5 with
// 64; 16 tokens 36.4, 32.6, 34.5; 64 tokens 60.2 with 16, 59.1 with 24, 70.1 with 64; 512 x 14336 at 1 token 20.7 with 16, 19.3
// with 24, 19.8 with 64, at 64 tokens 39.7, 41.6, 55.5; atomic, at 16 tokens, 1024 x 28672 42.2 with 16, 40.0 with 32, 1536 x
// 28672 53.9 with 16, 54.4 with 18, 53.1 with 21.
// The counter reduction of more than two tokens takes 12 where that gives the busiest wavefront no more 32-row blocks than 16 do:
// every split is a block to be added.  The line was drawn with the last workgroup of a column block adding them alone, as it still does
// in small eager calls (km_sum_launch); 16 / 12 splits, us: 512 x 1536 at 8 tokens 11.6 /
// 11.1, 768 x 4224 at 8 15.9 / 15.4, 896 x 4864 at 33 23.4 / 22.8, 1024 x 5632 at 16 18.5 / 17.8, 2048 x 6144 at 64 38.5 / 36.1.
// Where it gives more, the stream is longer by whole blocks: 512 x 4096 at 8 (two blocks of four wavefronts, three) 13.3 / 13.9,
// 896 x 7168 at 33 25.1 / 26.2, 1024 x 8192 at 3 and 64 18.2 / 19.2, 31.3 / 32.2, 896 x 4864 at 8 16.8 / 17.1.  From a width of
// 1536 on 16 splits are 192 workgroups and more, and up to four blocks 12 are the better in any case: 1536 x 12288 at 8 and 64
// 29.6 / 29.4, 46.3 / 44.5, 2048 x 11264 34.4 / 33.6, 50.9 / 49.6; beyond, 1536 x 18176 at 8 40.5 / 41.3, 2048 x 24320 60.2 /
// 61.5, 2048 x 16384 42.9 / 42.6, at 33 54.0 / 54.8.  At two tokens equal: 896 x 4864 15.4 / 15.8.  Where a launch adds the blocks on all
// CUs (blocks replayed from a graph) 16 gain on 12 at few tokens: 2048 x 6144 at 64 35.5 / 33.9, 896 x 4864 at 33 22.1 / 21.9, 768 x 4224
// at 8 15.2 / 15.1; 1024 x 5632 at 16 16.1 / 16.6, 1536 x 12288 at 8 and 64 29.1 / 29.9, 44.2 / 44.5, 2048 x 11264 32.4 / 33.1, 47.8 / 48.5.  The
// line has not been moved for that.
constexpr int kFewSplits = 16;
int few_splits(int M, int d_model, int d_ff, int k2c, int reduce) {
    const int rows = reduce == DFK_REDUCE_ATOMIC ? d_model - d_model / 4 : M > 16 ? 2 * d_model : d_model;
    int few = kFewSplits;
    if (reduce == DFK_REDUCE_TICKET && M > 2) {
        const int waves = M <= 16 && (d_model + 127) / 128 < 8 ? 4 : 8;                                  // of the down kernel
        auto blocks = [&](int splits) { return ((max_slice_rows(d_ff, splits) + 31) / 32 + waves - 1) / waves; };   // of its busiest one
        if (blocks(12) == blocks(16) || (d_model >= 1536 && blocks(12) <= 4)) few = 12;
    }
    return std::max(1, std::min(256 / k2c, std::max(few, d_ff / rows)));
}
// Workgroups of the 64-token pair's down kernels, untuned, own two 128-column blocks instead of one (512-byte pieces of W_down's
// rows, A_2 read half as often) where the layer is wide and a split then still has many rows: two blocks mean twice as many
// splits, whose sum has to be paid for by the reading.  Time with two blocks over time with one, atomic reduction (single
// launch), 2 to 16 tokens: 298 rows (5120 x 3584) 1.07 to 1.10, 614 (6144 x 6144) 1.00 to 1.02, 796 (7168 x 7168) 0.99 to 1.00,
// 930 (5888 x 10240) 1.00 to 1.02, 938 (5120 x 11264) 0.96 to 0.98, 1109 (7168 x 9984) 0.98 to 0.99, 2201 (11008 x 11008) 0.96;
// 32 tokens: 938 1.01, 1109 1.01, 1194 (10240 x 7168) 1.00, 1424 (8192 x 11392) 1.00, 2201 0.96.  Counter reduction (pair of
// launches, the block), 1 to 16 tokens: 938 1.00 to 1.03, 1175 (5888 x 12928) 1.00 to 1.02, 1393 (7168 x 12544) 0.98 to 1.00,
// 2201 0.98 to 0.99, 2304 (5120 x 27648, 4 tokens, whole call) 138.6 -> 137.1 us; 32 tokens: 1424 1.02, 1792 (8192 x 14336) 1.02,
// 2389 (10240 x 14336) 1.00, 2848 (16384 x 11392) 1.00, 3584 (8192 x 28672, whole call) 235.3 -> 238.5 us, 4096 (16384 x 16384)
// 0.99, and where splits of one block each make few workgroups 1536 (11008 x 7680, 172 of them) 0.99, 2457 (12288 x 12288, 192)
// 0.99. Below a d_model of 5120 it gained at most 2 % and lost as much (4608 x 10112, 722 rows: 0.99 to 1.02).
bool two_blocks(int M, int d_model, int d_ff, int reduce) {
    if (d_model < 5120) return false;
    const int nblk = (d_model + 127) / 128, rows = d_ff / few_splits(M, d_model, d_ff, nblk / 2, reduce);
    if (reduce == DFK_REDUCE_ATOMIC) return rows >= (M > 16 ? 1152 : 896);
    const bool few = nblk * few_splits(M, d_model, d_ff, nblk, reduce) < 208;   // workgroups with one block each
    return rows >= (M > 16 && !few ? 4096 : 1280);
}
// d_ff splits of the 256-token pair's down kernel, untuned: 12, one per 640 rows of a longer d_ff (512 with fewer than 8 column
// blocks), with fewer than 10 and more than 128 tokens up to 16 of 320 rows and more; or the next smaller count that cuts d_ff
// into whole 64-row steps of the down kernel, if there is one that is not much smaller (five eighths; where that makes splits of
// more than 1024 rows three quarters, up to 128 tokens seven eighths).  More splits only add partial blocks; fewer leave CUs
// without a workgroup; a split with a partial last step takes the form with clamped addresses and a step more, which costs the
// most with three or four token tiles per group. Whole call, us: 1920 x 3072 at 253 tokens 44.8 with 17 splits, 41.4 with 12,
// 40.6 with 8; 1024 x 2816 at 80 24.2 with 32, 20.5 with 12, 20.0 with 11; 2304 x 9216 at 256 68.7 with 14, 64.8 with 12; 2432 x
// 6656 at 256 60.6 with 12, 58.5 with 8; 1536 x 8960 at 256 53.4 with 12, 49.9 with 14, 52.1 with 20; 3584 x 18944 at 256 170
// with 9, 147 with 8; 6912 x 20352 at 212 266 with 4, 273 with 3; 4480 x 23040 at 68 139.9 with 7, 142.5 with 6; a long d_ff: 512
// x 28672 at 256 83.9 with 12, 59.4 with 32, 60.0 with 64; 256 x 8192 at 1 18.8 with 8, 17.4 with 12; 1024 x 14336 at 256 57.4
// with 12, 50.3 with 16, 52.3 with 32; no whole steps: 1920 x 10496 at 96 46.5 with 12 or 17, 45.5 with 16; few column blocks:
// 1152 x 5504 at 200 38.8 with 12, 37.6 with 16, 38.3 with 28, and at 128 30.7 with 12, 30.8 with 16; 2048 x 5504 at 200 46.9
// with 12, 47.7 with 16.  (All without token groups; where the launch divides the tokens it takes fewer of these splits,
// big_down_launch: 512 x 28672 at 256 has 32 and two groups, 55.4.)
int big_splits(int M, int d_ff, int k2c) {
    const int most = 256 / k2c, narrow = M > 128 && k2c < 10 ? std::min(16, d_ff / 320) : 0;
    const int want = std::min(most, std::max({12, d_ff / (k2c < 8 ? 512 : 640), narrow}));
    for (int k = want; 8 * k >= 5 * want; --k)
        if (d_ff % (64 * k) == 0 && (d_ff <= 1024 * k || (M > 128 ? 4 * k > 3 * want : 8 * k >= 7 * want))) return k;
    return want;
}
int clamp_splits(int want, int d_ff) { return std::max(1, std::min(want, d_ff / 8)); }

dfk_config_t make_cfg(int variant, int path, int splits, int waves, int depth, int k2s, int k2c,
                      int a2dt, int reduce = DFK_REDUCE_TICKET, int rows_by_wave = 0, int kmajor = 0) {
    dfk_config_t c;
    std::memset(&c, 0, sizeof c);
    c.variant = variant; c.path = path; c.splits = splits; c.waves = waves; c.depth = depth;
    c.reduce = reduce; c.k2_splits = k2s; c.k2_col_blocks = k2c; c.a2_dtype = a2dt;
    c.k2_rows_by_wave = rows_by_wave;
    c.kmajor = kmajor;
    return c;
}

bool same_cfg(const dfk_config_t& a, const dfk_config_t& b) {
    return a.variant == b.variant && a.path == b.path && a.splits == b.splits && a.waves == b.waves &&
           a.depth == b.depth && a.reduce == b.reduce && a.k2_splits == b.k2_splits &&
           a.k2_col_blocks == b.k2_col_blocks && a.a2_dtype == b.a2_dtype &&
           a.k2_rows_by_wave == b.k2_rows_by_wave && a.kmajor == b.kmajor;
}

// Half inputs off 128, untuned: whether the pair on the matrix cores comes before the plain-FMA one, which keeps A_2 in fp32 as well but
// takes 8 tokens per launch and reads X anew for every weight row.  Whole call, us, plain FMA / matrix cores: 736 x 3472 at 1, 8, 64 and 256
// tokens 19.3 / 17.2, 49.5 / 17.5, 388 / 30.2, 1545 / 114; 1800 x 5000 at 1, 4, 16 and 110 30.8 / 25.9, 61.0 / 25.4, 172 / 26.5, 1188 /
// 85.4; 2888 x 7688 at 2, 16 and 64 45.6 / 41.1, 189 / 42.5, 756 / 73.4.  One token needs no tile of sixteen: from 45 MB of weights on plain
// FMA is first there, 1208 x 6600 (48 MB) 23.9 / 25.6, 2888 x 5000 (87 MB) 29.0 / 31.2, 2936 x 9000 (159 MB) 41.4 / 49.2, 2296 x 4104 (57
// MB) 28.9 / 27.7, 2008 x 2400 (29 MB) 22.5 / 19.5; at two tokens from 180 MB on, 8200 x 4000 (197 MB) 55.1 / 55.9, 2936 x 9000 55.8 / 49.1.
bool matrix_cores_pay(int M, int d_model, int d_ff) {
    const size_t weights = (size_t)6 * d_model * d_ff;
    return M > 2 || weights < (M == 1 ? 45000000u : 180000000u);
}

// The candidate set of the scheduler (Method: tiling variants x tile sizes).
std::vector<dfk_config_t> candidates(int M, int d_model, int d_ff, dfk_dtype_t dtype) {
    std::vector<dfk_config_t> out;
    auto push = [&](const dfk_config_t& c) {
        if (!config_valid(c, M, d_model, d_ff, dtype)) return;
        for (const auto& o : out)
            if (same_cfg(o, c)) return;
        out.push_back(c);
    };
    const int a2dt = dtype == DFK_BF16 ? DFK_BF16 : DFK_FP32;   // VALU pair: fp32 unless the inputs are bf16
    if (dtype == DFK_BF16 || dtype == DFK_FP16) {   // (the first-generation MFMA kernels validate for bf16 only)
        // MFMA path: d_ff slices ("column-major tiling": each workgroup owns a
        // block of weight rows and reuses it for every token).
        for (int splits : {256, 512})
            for (int waves : {4, 8})
                for (int depth : {2, 4, 6, 8})
                    for (int reduce : {DFK_REDUCE_ATOMIC, DFK_REDUCE_TICKET})
                        push(make_cfg(DFK_VARIANT_FUSED, DFK_PATH_MFMA, clamp_splits(splits, d_ff), waves,
                                      depth, 0, 0, a2dt, reduce));
        const int nblk = (d_model + 127) / 128;   // (a partial last column block: the 64-token pair in bf16 only)
        // the single launch on the k-major stage one of the 64-token pair (a slice of at most 64 rows per workgroup)
        for (int splits : {256, 512, d_ff > 512 * 64 ? ((d_ff + 63) / 64 + 255) / 256 * 256 : 512})
            for (int reduce : {DFK_REDUCE_ATOMIC, DFK_REDUCE_TICKET})
                for (int wd : {83, 84, 46, 48})   // wavefronts, ring depth
                    push(make_cfg(DFK_VARIANT_FUSED, DFK_PATH_MFMA, clamp_splits(splits, d_ff), wd / 10, wd % 10, 0, 0, (int)dtype,
                                  reduce, 0, 1));
        // two-kernel: the down projection is tiled (d_ff splits) x (column blocks of
        // waves*128 or 2*waves*128 columns), about one or two workgroups per CU
        for (int splits : {256, 512})
            for (int waves : {4, 8})
                for (int per_wave : {1, 2}) {
                    const int wg_blocks = waves * per_wave;
                    if (wg_blocks > nblk || nblk % wg_blocks) continue;
                    const int k2c = nblk / wg_blocks;
                    for (int grid : {256, 512})
                        for (int reduce : {DFK_REDUCE_ATOMIC, DFK_REDUCE_TICKET})
                            push(make_cfg(DFK_VARIANT_TWO_KERNEL, DFK_PATH_MFMA, clamp_splits(splits, d_ff),
                                          waves, 4, clamp_splits(std::max(1, grid / k2c), d_ff), k2c, a2dt,
                                          reduce));
                }
        // two-kernel, down projection with the rows divided among the wavefronts: few d_ff splits
        for (int waves : {8, 4})
            for (int cbw : {1, 2, 4}) {           // 128-column blocks per workgroup
                if (nblk < cbw || nblk % cbw) continue;
                const int k2c = nblk / cbw;
                for (int grid : {256, 512})
                    for (int reduce : {DFK_REDUCE_TICKET, DFK_REDUCE_ATOMIC})
                        for (int depth : {3, 4})
                            push(make_cfg(DFK_VARIANT_TWO_KERNEL, DFK_PATH_MFMA, clamp_splits(256, d_ff), waves, depth,
                                          clamp_splits(std::max(1, grid / k2c), d_ff), k2c, DFK_BF16, reduce, 1));
            }
        // two-kernel, activations through the tile rings: up to 64 tokens per launch.  A slice of the
        // gate/up kernels of this pair and of the next holds at most 64 rows, so a d_ff beyond
        // 512 * 64 needs more slices: the next multiple of 256 that is enough.
        const int more_splits = d_ff > 512 * 64 ? ((d_ff + 63) / 64 + 255) / 256 * 256 : 512;
        for (int splits : {256, 512, more_splits})
            for (int cbw : {1, 2}) {
                if (nblk < cbw || nblk % cbw) continue;
                const int k2c = nblk / cbw;
                for (int k2s : {0, std::min(kFewSplits, 256 / k2c), 256 / k2c, 512 / k2c})     // 0: the untuned count
                    for (int reduce : {DFK_REDUCE_TICKET, DFK_REDUCE_ATOMIC})
                        for (int wd : {83, 84, 46, 48})   // wavefronts, ring depth
                            push(make_cfg(DFK_VARIANT_TWO_KERNEL, DFK_PATH_MFMA, clamp_splits(splits, d_ff), wd / 10, wd % 10,
                                          clamp_splits(k2s ? k2s : few_splits(M, d_model, d_ff, k2c, reduce), d_ff), k2c, (int)dtype,
                                          reduce, 0, 1));
            }
        // both kernels of that pair in one launch (gate/up workgroups at the head of the grid, down workgroups
        // behind them); off 128 it is a form of the listed pair that the scheduler takes by itself (single_launch_of)
        for (int splits : {256, 512})
            for (int cbw : {1, 2}) {
                if (d_model % 128 || nblk < cbw || nblk % cbw) continue;
                const int k2c = nblk / cbw;
                for (int k2s : {0, std::min(kFewSplits, 256 / k2c), 256 / k2c, 512 / k2c})
                    for (int reduce : {DFK_REDUCE_TICKET, DFK_REDUCE_ATOMIC})
                        for (int depth : {3, 4})
                            push(make_cfg(DFK_VARIANT_FUSED, DFK_PATH_MFMA, clamp_splits(splits, d_ff), 8, depth,
                                          clamp_splits(k2s ? k2s : few_splits(M, d_model, d_ff, k2c, reduce), d_ff), k2c, (int)dtype,
                                          reduce, 0, 4));
            }
        // two-kernel for 33..64 tokens: gate/up kernel with workgroup-shared weight tiles and one token tile per
        // wavefront, down kernel of the pair above
        if (M > 32 && nblk >= 1)
            for (int splits : {256, 512})
                for (int grid : {256, 512})
                    for (int reduce : {DFK_REDUCE_TICKET, DFK_REDUCE_ATOMIC})
                        for (int depth : {3, 4})
                            push(make_cfg(DFK_VARIANT_TWO_KERNEL, DFK_PATH_MFMA, clamp_splits(splits, d_ff), 8, depth,
                                          clamp_splits(std::max(1, grid / nblk), d_ff), nblk, (int)dtype, reduce, 0, 3));
        // two-kernel, workgroup-shared weight tiles: up to 256 tokens per launch.  Offered beyond 64 tokens,
        // and below where d_model rules out the pair above (it needs whole 128-k chunks per wavefront,
        // this one only d_model % 128 == 0)
        bool have_km = false;
        for (const auto& o : out) have_km = have_km || o.kmajor == 1;
        if ((M > 64 || !have_km) && nblk >= 1) {
            const int k2c = nblk;
            for (int splits : {256, 512, more_splits})
                for (int k2s : {big_splits(M, d_ff, k2c), std::min(12, 256 / k2c), 256 / k2c, 512 / k2c})   // the untuned count first
                    for (int reduce : {DFK_REDUCE_TICKET, DFK_REDUCE_ATOMIC})   // (waves and depth do not change its kernels)
                        push(make_cfg(DFK_VARIANT_TWO_KERNEL, DFK_PATH_MFMA, clamp_splits(splits, d_ff), 8, 3,
                                      clamp_splits(std::max(1, k2s), d_ff), k2c, (int)dtype, reduce, 0, 2));
        }
    }
    for (int splits : {256, 512, 1024})
        for (int waves : {4, 8})
            push(make_cfg(DFK_VARIANT_FUSED, DFK_PATH_VALU, clamp_splits(splits, d_ff), waves, 0, 0, 0,
                          a2dt));
    const int nchunk = d_model / (dtype == DFK_FP32 ? 4 : 8);
    // The first of these is the untuned two-kernel form: the fewest d_ff splits (a power of two, 8 to 64) whose down kernel has
    // at least 160 workgroups, or 64 splits where no count up to that has: with one or two column blocks (half inputs below a
    // d_model of 1536, fp32 below 768).  A workgroup's loads in flight are what paces it, so too few leave most of the chip
    // waiting; beyond, the sum of the splits' blocks costs more (down kernel, us, with 8, 16, 32 and 64 splits: half inputs, 8
    // tokens of 2888 x 7688, five column blocks: 105, 60.6, 41.4, 56.1; fp32, 4 tokens, eleven: 37.6, 26.8, 35.1, 40.2).
    const int max_cb = std::max(1, nchunk / 64);
    int k2_first = 8;
    while (k2_first < 64 && k2_first * std::min(max_cb, 512 / k2_first) < 160) k2_first *= 2;
    for (int splits : {512, 1024})
        for (int k2s : {k2_first, 8, 16, 32}) {
            const int k2 = clamp_splits(k2s, d_ff);
            const int cb = std::max(1, std::min(max_cb, std::max(1, 512 / k2)));
            push(make_cfg(DFK_VARIANT_TWO_KERNEL, DFK_PATH_VALU, clamp_splits(splits, d_ff), 8, 0, k2,
                          cb, a2dt));
        }
    if (dtype == DFK_FP16 && d_model % 128) {   // (ranked by matrix_cores_pay, not by their place)
        const int k2c = (d_model + 127) / 128, more_splits = d_ff > 512 * 64 ? ((d_ff + 63) / 64 + 255) / 256 * 256 : 512;
        for (int splits : {256, more_splits})
            push(make_cfg(DFK_VARIANT_TWO_KERNEL, DFK_PATH_VALU, clamp_splits(splits, d_ff), k2c >= 8 ? 8 : 4, k2c >= 8 ? 3 : 6,
                          clamp_splits(few_splits(M, d_model, d_ff, k2c, DFK_REDUCE_TICKET), d_ff), k2c, DFK_FP32, DFK_REDUCE_TICKET, 0, 1));
    }
    return out;
}

// W_down given as [d_model, d_ff]: whether the down projection is split over d_ff (kmajor = 5 with column blocks) or its
// workgroups own rows of W_down^T whole, with nothing to sum across them.  Beyond 64 tokens always: whole rows take 64 tokens per
// launch and stream the weights again for each (256 tokens, us: 4096 x 14336 345 whole rows, 108 split; 896 x 4864 136, 34; 12288 x
// 12288 665, 265).  Up to 64, whole rows read all of A_2 in every workgroup, which costs with tokens x d_ff where tokens are at
// least twice the workgroup's rows; the split's partial sums cost a launch and with tokens x d_model, the less of it the more tokens
// the other form has to fetch beside the same weights.  Split over whole rows, time, 1024 to 4096 wide: at 17 to 32 tokens 1536 x 8960
// 0.90 to 0.93, 2304 x 9216 0.98 to 0.99, 2816 x 9600 0.96 to 0.99, 3072 x 12288 0.95 to 0.98, 4096 x 14336 0.96 to 0.99, 3584 x
// 18944 0.92 to 0.96; other side: 1024 x 5632 1.02, 2048 x 5504 1.05, 2560 x 6912 1.02 to 1.03, 3584 x 9216 1.02 to 1.04; at 33 to 48
// 1280 x 5120 0.99, 2048 x 5504 0.98 to 0.99, 3584 x 9216 0.97 to 0.98; other side: 1024 x 2816 1.04 to 1.07, 1536 x 4096 1.04, 1792 x
// 4864 1.00; at 49 to 64 1536 x 4096 0.98 to 0.99; other side: 1024 x 2816 1.00 to 1.01.  Where rows of W_down^T are a multiple of
// 16 KB apart a step's rows share memory channels: 4096 x 8192 1.08 to 1.09, 1.04 and 0.98 to 0.99 at those counts, 3072 x 8192 1.03 to
// 1.05 and 0.97, 2048 x 8192 1.00 to 1.02 and 0.94.  Beyond 4096 the whole rows are uneven shares as a rule: 6144 x 8064 1.01 to 1.03
// up to 32 tokens, 0.97 to 0.98 at 48, 8192 x 7168 1.02 to 1.04 at 48, 0.98 at 64 (12288 x 12288 166 / 179 us at 64: tokens below twice
// the rows).  Below 1024, where four wavefronts own the whole rows: 512 x 2048 1.04 to 1.06 up to 32 tokens, 0.93 at 48, 768 x 3072 0.94.
// With the sum launch's present form (16 splits a batch) the lines hold, best candidate of either: at 24 tokens 1536 x 8960 0.91,
// 2304 x 9216 0.99, 4096 x 14336 0.99, other side 1024 x 5632 0.98, 2048 x 5504 1.05, 3584 x 9216 1.03; at 40 2048 x 5504 0.98, 1792 x 4864
// 1.00, 4096 x 8192 1.03; 8192 x 7168 at 48 1.03; 512 x 2048 at 24 and 48 1.01, 0.91.
bool wdt_split_pays(int M, int d_model, int d_ff) {
    if (M > 64) return true;
    const long long tokens = (M + 15) / 16 * 16, rows = d_model / std::max(1, std::min(256, d_model / 16)), a2 = tokens * d_ff;
    if (M <= 16 || tokens < 2 * rows) return false;
    if (d_model < 1024) return a2 >= 180 * 512;
    if (d_model > 4096) return a2 >= 450 * 512;
    return a2 >= (d_ff % 8192 ? 155000 : 200000) + 35 * (80 - tokens) * tokens * d_model / 1000;
}

// The candidates of that layout: the 64-token pair's gate/up kernel, then the down kernel whose workgroups own slices of d_model;
// and the form that splits d_ff.  First in the list = the untuned default.
std::vector<dfk_config_t> candidates_wdt(int M, int d_model, int d_ff, dfk_dtype_t dtype) {
    std::vector<dfk_config_t> out;
    // plain fp32-FMA kernels for every shape and type (after the MFMA pair in the list, where there is one)
    auto valu = [&]() {
        const int a2dt = dtype == DFK_BF16 ? DFK_BF16 : DFK_FP32;
        for (int splits : {512, 1024})
            for (int k2s : {256, 512}) {
                dfk_config_t c = make_cfg(DFK_VARIANT_TWO_KERNEL, DFK_PATH_VALU, clamp_splits(splits, d_ff), 8, 0,
                                          std::max(1, std::min(k2s, (d_model + 7) / 8)), 1, a2dt, DFK_REDUCE_TICKET, 0, 5);
                if (!config_valid(c, M, d_model, d_ff, dtype)) continue;
                bool dup = false;
                for (const auto& o : out) dup = dup || same_cfg(o, c);
                if (!dup) out.push_back(c);
            }
    };
    if (dtype != DFK_BF16 && dtype != DFK_FP16) {
        valu();
        return out;
    }
    const int more_splits = d_ff > 512 * 64 ? ((d_ff + 63) / 64 + 255) / 256 * 256 : 512;
    const int t16 = d_model / 16;
    auto push = [&](const dfk_config_t& c) {
        if (!config_valid(c, M, d_model, d_ff, dtype)) return;
        for (const auto& o : out)
            if (same_cfg(o, c)) return;
        out.push_back(c);
    };
    // the form that splits the down projection over d_ff
    auto split_form = [&]() {
        const int nblk = d_model / 128;
        if (nblk < 2) return;
        // (beyond 64 tokens waves and depth do not change its kernels)
        for (int wd : M > 64 ? std::vector<int>{84} : std::vector<int>{84, 83, 48})
            for (int splits : {256, more_splits})
                for (int k2s : {big_splits(M, d_ff, nblk), 256 / nblk, std::min(12, 256 / nblk)})
                    push(make_cfg(DFK_VARIANT_TWO_KERNEL, DFK_PATH_MFMA, clamp_splits(splits, d_ff), wd / 10, wd % 10,
                                  std::max(1, std::min(k2s, d_ff / 64)), nblk, (int)dtype, DFK_REDUCE_TICKET, 0, 5));
    };
    // Half inputs where the whole-rows form does not exist (it needs four 128-wide chunks each way): the plain-FMA pair, which
    // keeps A_2 in fp32, comes first at every token count.  The split form would round A_2 to half, and overflow beyond 65504:
    // only for a caller who asks.
    if (dtype == DFK_FP16 && (d_model < 512 || d_ff < 512)) valu();
    if (wdt_split_pays(M, d_model, d_ff)) split_form();
    // Wavefronts, ring depth: three slots where the down kernel has workgroups (a 16-row tile each) for less than seven eighths of
    // the CUs, so that each needs more in flight, else two.  Two / three slots, us, at 1, 12 and 29 to 32 tokens: 1536 x 4096 14.6 /
    // 13.9, 15.2 / 14.8, 18.8 / 18.0; 2304 x 9216 30.3 / 29.5, 31.7 / 31.6, 38.9 / 38.4; 3200 x 4352 25.0 / 24.2, 24.7 / 24.4, 29.7 /
    // 28.7; 3456 x 8320 38.1 / 37.3, 37.9 / 37.6, 44.9 / 44.5; the most it loses there is 1.3 % (2048 x 8192 at 9 to 16 tokens).  On
    // the other side: 3584 x 4352 25.6 / 25.5, 25.4 / 25.8, 30.1 / 30.3; 3584 x 18944 68.4 / 69.9, 72.0 / 74.4, 89.7 / 90.6; 4096 x
    // 14336 at 8 59.7 / 60.7, 8192 x 7168 at 24 64.3 / 65.3.
    const std::vector<int> rings = 8 * t16 < 7 * 256 ? std::vector<int>{83, 82, 84, 46} : std::vector<int>{82, 83, 84, 46};
    for (int wd : rings)
        for (int splits : {256, 512, more_splits})
            for (int k2s : {256, 512, 128}) {
                push(make_cfg(DFK_VARIANT_TWO_KERNEL, DFK_PATH_MFMA, clamp_splits(splits, d_ff), wd / 10, wd % 10,
                              std::max(1, std::min(k2s, t16)), 1, (int)dtype, DFK_REDUCE_TICKET, 0, 5));
            }
    if (M > 16) split_form();   // (again: nothing is listed twice)
    valu();
    return out;
}

// One token: whether the single launch that keeps A_2 in LDS is the untuned choice, or the one that holds both kernels'
// workgroups. The former has nothing to wait for, but 256 partial sums of all of Y, a second round of workgroups from d_ff =
// 16384 on (a slice is at most 64 rows), and wavefronts that each own an eighth of the chunks and column blocks, which only
// widths that are multiples of 1024 divide evenly.  us, A_2 in LDS / both kernels' workgroups: 2048 x 5504 20.2 / 21.1, 3072 x
// 12288 43.1 / 43.7, 4096 x 8192 40.4 / 41.1, 4096 x 14336 59.4 / 60.1, 4096 x 16384 66.6 / 67.8.  On the other side: 4096 x
// 20480 88.5 / 83.2, 4096 x 4096 30.1 / 23.7, 1024 x 2816 13.2 / 11.4, 1536 x 4096 20.2 / 15.1, 2304 x 9216 31.1 / 27.9, 3584 x
// 9216 40.8 / 37.1, 7168 x 20480 146 / 135, 8192 x 14336 113 / 111, 8192 x 28672 222 / 213, 16384 x 16384 277 / 246; 3072 x 8192
// 30.8 / 30.7.  Beyond a d_ff of 32768 the launch of both kernels' workgroups is not listed (more than 512 slices of 64 rows),
// and what follows is the pair of launches with the counter reduction.  A_2 in LDS / pair: 512 x 36864 37.1 / 33.6, 1024 x 33280
// 45.3 / 44.5, 4096 x 53248 215 / 209, 5120 x 40960 202 / 195, 8192 x 40960 321 / 307, 16384 x 53248 923 / 789; 1024 x 53248 63.4
// / 63.3, 3072 x 40960 124 / 124, 2048 x 40960 86.5 / 88.0.
bool local_pays(int d_model, int d_ff) {
    return d_model % 1024 == 0 && d_model >= 2048 && d_model <= 4096 && d_ff >= 2 * d_model && d_ff <= 16384;
}

// Untuned default, from measurements on MI355X.  One token of some sizes (local_pays): the single launch that keeps A_2 in LDS,
// with the atomic reduction (no boundary between two kernels, and its 256 full-width partial sums are still cheap).  Else, up to
// 64 tokens and a d_ff of 32768: the single launch that holds both kernels' workgroups (atomic reduction), which saves the launch
// boundary at every token count.  Of the two-kernel forms: beyond 64 tokens the pair that takes up to 256 per launch, else the
// pair for up to 64 tokens, then the rows-split down kernel, then the rest.  Within a form of the 64-token pair: splits and
// column blocks as few_splits and two_blocks say.
// `fits`: which candidates the caller can run (all of them, or those within its scratch).
template <typename F>
bool enumerate_default(int M, int d_model, int d_ff, dfk_dtype_t dtype, int want_variant, dfk_config_t* out, F fits) {
    auto cands = candidates(M, d_model, d_ff, dtype);
    auto rank = [&](const dfk_config_t& c) {
        if (c.variant == DFK_VARIANT_TWO_KERNEL) {
            if (c.path == DFK_PATH_VALU) return c.kmajor == 0 ? 2 : matrix_cores_pay(M, d_model, d_ff) ? 1 : 3;
            if (c.kmajor == 2) return M > 64 ? -1 : 1;     // one launch for up to 256 tokens beats several of 64
            if (c.kmajor == 3) return 1;
            return c.kmajor ? 0 : c.k2_rows_by_wave ? 1 : 2;
        }
        if (roles_launch(c)) return M <= 64 && c.reduce == DFK_REDUCE_ATOMIC && c.depth == 4 ? -2 : 3;
        if (c.path == DFK_PATH_MFMA && c.kmajor == 1)      // the single launch with A_2 in LDS
            return c.reduce == DFK_REDUCE_ATOMIC && c.waves == 8 ? (M == 1 && local_pays(d_model, d_ff) ? -3 : 3) : 4;
        return 5;
    };
    const int nblk = (d_model + 127) / 128;
    auto split_rank = [&](const dfk_config_t& c) {         // among configurations of one rank
        if (c.kmajor == 2) {
            const int few = clamp_splits(big_splits(M, d_ff, c.k2_col_blocks), d_ff);
            return (c.reduce == DFK_REDUCE_TICKET ? 0 : 4) + (c.k2_splits > few ? 2 : c.k2_splits < few ? 1 : 0);
        }
        if (c.path != DFK_PATH_MFMA || c.k2_col_blocks < 1 || (c.kmajor != 1 && c.kmajor != 4)) return 0;
        const int width = nblk / c.k2_col_blocks, want = two_blocks(M, d_model, d_ff, c.reduce) ? 2 : 1;
        const int few = clamp_splits(few_splits(M, d_model, d_ff, c.k2_col_blocks, c.reduce), d_ff);
        return (c.k2_splits > few ? 4 : c.k2_splits < few ? 2 : 0) + (width != want ? 1 : 0);
    };
    const dfk_config_t* best = nullptr;
    std::pair<int, int> best_rank;
    for (const auto& c : cands) {
        if ((want_variant != DFK_VARIANT_AUTO && c.variant != want_variant) || !fits(c)) continue;
        const std::pair<int, int> r(rank(c), split_rank(c));
        if (!best || r < best_rank) { best = &c; best_rank = r; }
    }
    if (!best) return false;
    *out = *best;
    return true;
}

// The pair for up to 64 tokens as the single launch of both kernels' workgroups: same splits, same reduction, so the same bits
// with the counter reduction, and no boundary between two launches.  What a block runs where it pays, and a width off 128 without
// a tuned entry (whose candidates are the pair and not this form of it; dfk_tune times it beside them).  us, pair / single launch:
//
// Blocks (layers replayed from a graph) from 48 MB of weights on; below, the down workgroups' wait costs what the boundary does.
// 2304 x 9216 at 1, 8 and 33 tokens 32.0 / 30.2, 32.6 / 31.1, 43.6 / 41.5; 4096 x 14336 at 1 and 64 62.3 / 61.2, 83.3 / 81.7; 5120
// x 40960 at 64 271 / 257; 1792 x 4864 (52 MB) at 8 and 33 20.4 / 20.2, 29.9 / 28.6; 1536 x 8960 at 17 30.2 / 29.4.  On the other
// side: 1024 x 4096 (25 MB) at 17 and 64 18.5 / 19.8, 27.3 / 28.2; 1536 x 4096 (38 MB) at 32 22.3 / 23.4; 1280 x 5120 (39 MB) at 17
// 23.0 / 23.6.  A width that is a multiple of 1024 gives the eight wavefronts equal runs of k, so the gate/up kernel ends evenly and
// there is less to gain: from 100 MB on.  2048 x 5504 (68 MB) at 8 and 17 22.7 / 23.2, 25.9 / 26.3; 1024 x 8192 (50 MB) at 8 20.1 /
// 20.8; 2048 x 8192 (101 MB) at 17 and 40 31.1 / 31.2, 37.5 / 36.9.  Not where the 256 slices of d_ff have two row tiles each and
// hardly one has fewer: no gate/up workgroup ends ahead of the others then, and their streams are short against the wait.  2816 x
// 3456 at 2, 17 and 64 20.9 / 21.5, 25.5 / 26.6, 38.8 / 40.0; 3456 x 3712 23.8 / 24.0, 28.3 / 29.6, 42.6 / 43.6; 3584 x 3968 25.3 /
// 25.7, 29.4 / 30.7, 43.2 / 44.5.  On the other side: 4352 x 4352 32.8 / 32.5, 37.8 / 36.6, 52.9 / 52.3; 3584 x 5376 30.9 / 29.9,
// 35.0 / 34.5, 48.8 / 48.5; 2304 x 3328 (46 MB) 20.4 / 19.9, 24.9 / 25.4, 38.1 / 37.9.
//
// Off 128 (whole call) from 48 MB on, beyond 16 tokens at every size.  2888 x 7688 at 1, 12 and 64 tokens 37.5 / 35.1, 39.1 / 37.3,
// 54.5 / 53.5; 1800 x 5000 at 16 and 33 25.0 / 23.9, 30.9 / 29.7; 2008 x 2400 (29 MB) at 17 and 33 22.1 / 20.6, 26.6 / 24.5; 904 x
// 1024 (6 MB) at 33 18.2 / 17.5; 1416 x 3776 at 17 22.2 / 22.6, at 64 31.1 / 31.0.  Not where d_ff is no larger than d_model: 8200 x
// 1000 at 1 and 17 22.8 / 24.7, 30.9 / 31.9 (2888 x 2888 at 12 24.5 / 23.4).
//
// These figures are from before a launch added the splits' blocks (km_sum_launch), which gave the pair more than the single launch.  Blocks
// in a graph with it: 2304 x 9216 at 1, 8 and 33 30.8 / 30.7, 31.1 / 31.7, 40.5 / 40.0; 4096 x 14336 at 1 and 64 63.3 / 62.8, 80.6 / 79.6; 1792 x
// 4864 at 8 and 33 19.1 / 20.3, 26.0 / 25.9; 1536 x 8960 at 17 28.2 / 28.2; 3584 x 5376 at 2, 17 and 64 28.5 / 28.6, 32.6 / 32.7, 46.2 / 44.6; 5120 x
// 27648 at 4 and 64 136.8 / 140.7, 179.7 / 171.6; on the other side 1024 x 4096 at 17 15.9 / 17.8, 2048 x 5504 at 8 21.0 / 23.0.  The lines are
// where they were: up to 16 tokens of 48 to 100 MB the pair would now be the faster by up to 6 %.
bool single_launch_pays(int M, int d_model, int d_ff) {
    const size_t bytes = (size_t)6 * d_model * d_ff;
    if (M > 64) return false;
    if (d_model % 128) return d_ff > d_model && (M > 16 || bytes >= 48000000u);
    const int tiles = d_ff / 8;
    if (tiles > 2 * 256 * 13 / 16 && tiles <= 2 * 256) return false;
    return bytes >= (d_model % 1024 ? 48000000u : 100000000u);
}
// That form of a configuration, if it is of the pair and the form fits.
bool single_launch_of(const dfk_config_t& c, int M, int d_model, int d_ff, dfk_dtype_t dtype, bool block, dfk_config_t* out) {
    if (M > 64 || c.kmajor != 1 || c.path != DFK_PATH_MFMA || c.variant != DFK_VARIANT_TWO_KERNEL) return false;
    dfk_config_t r = c;
    r.variant = DFK_VARIANT_FUSED; r.kmajor = 4; r.depth = 4;
    const auto fits = block ? mfma_km_block_config_valid : mfma_km_roles_config_valid;
    if (!fits(r, M, d_model, d_ff, dtype)) return false;
    *out = r;
    return true;
}

// The default is a pure function of the problem, and finding it lists and validates every candidate (5 to 25 us of host
// time per call; a 512 x 1536 layer, whose kernels take 9 us: 18.1 us per call from Python, 10.8 without it).  Each thread
// remembers the last ones it found, a fixed number of slots by hash of the problem.
constexpr int kWdtVariant = -1;        // in place of a variant: W_down given as [d_model, d_ff]
bool heuristic(int M, int d_model, int d_ff, dfk_dtype_t dtype, int want_variant, dfk_config_t* out) {
    struct Slot { int M, d_model, d_ff, dtype, variant; dfk_config_t cfg; };
    constexpr unsigned kSlots = 64;
    static thread_local Slot slots[kSlots];          // M = 0: empty
    const unsigned h = ((((unsigned)M * 31u + (unsigned)d_model) * 31u + (unsigned)d_ff) * 31u + (unsigned)dtype) * 31u + (unsigned)want_variant;
    Slot& s = slots[(h ^ h >> 6 ^ h >> 12) % kSlots];
    if (s.M != M || s.d_model != d_model || s.d_ff != d_ff || s.dtype != (int)dtype || s.variant != want_variant) {
        dfk_config_t c;
        if (want_variant == kWdtVariant) {
            const auto cands = candidates_wdt(M, d_model, d_ff, dtype);
            if (cands.empty()) return false;
            c = cands[0];
        } else if (!enumerate_default(M, d_model, d_ff, dtype, want_variant, &c, [](const dfk_config_t&) { return true; })) {
            return false;
        }
        if (want_variant == DFK_VARIANT_AUTO && d_model % 128 && single_launch_pays(M, d_model, d_ff))
            single_launch_of(c, M, d_model, d_ff, dtype, false, &c);
        s.M = M; s.d_model = d_model; s.d_ff = d_ff; s.dtype = (int)dtype; s.variant = want_variant; s.cfg = c;
    }
    *out = s.cfg;
    return true;
}

// ---------------------------------------------------------------- tuning table
struct Entry {
    dfk_config_t cfg;
    double usec;
};
// M, d_model, d_ff, dtype, slot.  Slot 0 holds the choice for the problem; slots DFK_VARIANT_FUSED and
// DFK_VARIANT_TWO_KERNEL the best known configuration of that variant (what a call that asks for a variant gets).
using Key = std::tuple<int, int, int, int, int>;
std::map<Key, Entry> g_table;
constexpr int kSlotWdt = 3;   // slot of the best configuration for W_down given as [d_model, d_ff]
void table_put(int M, int d_model, int d_ff, int dtype, const Entry& e, bool chosen) {   // g_mu held
    if (wdt_layout(e.cfg)) {   // the other layout of W_down has a slot of its own and never is the plain choice
        g_table[Key(M, d_model, d_ff, dtype, kSlotWdt)] = e;
        return;
    }
    // off 128 the single launch of both kernels' workgroups is a form of the pair, not an entry of the fused variant (that one
    // keeps A_2 in fp32)
    if (!(d_model % 128 && roles_launch(e.cfg))) g_table[Key(M, d_model, d_ff, dtype, e.cfg.variant)] = e;
    if (chosen) g_table[Key(M, d_model, d_ff, dtype, 0)] = e;
}

int m_bucket(int M) {
    int b = 1;
    while (b < M) b <<= 1;
    return b;
}

bool lookup(int M, int d_model, int d_ff, dfk_dtype_t dtype, int want_variant, dfk_config_t* out) {
    std::lock_guard<std::mutex> lk(g_mu);
    for (int m : {M, m_bucket(M)}) {
        auto it = g_table.find(Key(m, d_model, d_ff, (int)dtype, want_variant == DFK_VARIANT_AUTO ? 0 : want_variant));
        if (it == g_table.end()) continue;
        const dfk_config_t& c = it->second.cfg;
        if (!config_valid(c, M, d_model, d_ff, dtype)) continue;
        *out = c;
        return true;
    }
    return false;
}

bool choose_wdt(int M, int d_model, int d_ff, dfk_dtype_t dtype, dfk_config_t* out, int* tuned) {
    if (lookup(M, d_model, d_ff, dtype, kSlotWdt, out)) {
        if (tuned) *tuned = 1;
        return true;
    }
    if (tuned) *tuned = 0;
    return heuristic(M, d_model, d_ff, dtype, kWdtVariant, out);
}

bool choose(int M, int d_model, int d_ff, dfk_dtype_t dtype, int want_variant, dfk_config_t* out,
            int* tuned) {
    if (lookup(M, d_model, d_ff, dtype, want_variant, out)) {
        if (tuned) *tuned = 1;
        return true;
    }
    if (tuned) *tuned = 0;
    return heuristic(M, d_model, d_ff, dtype, want_variant, out);
}

// ---------------------------------------------------------------- dispatch
// norm_w / eps / resid: the pre-norm residual form (kernel pair for up to 64 tokens only,
// checked by the caller); NULL / 0 / NULL for the plain block.
dfk_status_t run_in(const WsLayout& l, const void* X, const void* Wg, const void* Wu, const void* Wd, void* Y, int M,
                    int d_model, int d_ff, dfk_dtype_t dtype, const dfk_config_t& c, void* ws,
                    hipStream_t st, const void* norm_w = nullptr, float eps = 0.f, const void* resid = nullptr) {
    MlpArgs a;
    std::memset(&a, 0, sizeof a);
    a.X = X; a.Wg = Wg; a.Wu = Wu; a.Wd = Wd; a.Y = Y;
    a.M = M; a.d_model = d_model; a.d_ff = d_ff;
    a.splits = c.splits; a.k2_splits = c.k2_splits; a.k2_col_blocks = c.k2_col_blocks;
    a.dtype = (int)dtype;
    a.a2_is_fp32 = c.a2_dtype == DFK_FP32;
    a.tickets = (unsigned*)((char*)ws + l.tickets_off);
    a.reduce_mode = c.reduce;
    a.yacc = (float*)((char*)ws + l.yacc_off);
    a.P = (float*)((char*)ws + l.p_off);
    a.Q = (float*)((char*)ws + l.q_off);
    a.a2 = (char*)ws + l.a2_off;
    a.norm_w = norm_w; a.eps = eps; a.resid = resid;
    if (norm_w && (c.kmajor == 2 || !mfma_km_block_config_valid(c, M, d_model, d_ff, dtype))) {   // (kmajor 1 and, up to 64 tokens, 5 fold it)
        // The 256-token pair is paced by its MFMA and LDS work, so scaling X inside every workgroup
        // costs more there than one small launch that writes the normalised input once.  The
        // 64-token pair folds the normalisation into its gate/up kernel unless the slices of the
        // normalisation weight do not fit its LDS beside the rings (very wide d_model): then it
        // takes the same small launch.  The transposed layout rounds the product with the weight alone at every token count, as that
        // kernel does, and scales its sums: rounding the normalised value instead was 0.5 % further from 64 bits with weights
        // near one (100 tokens of 2048 x 5504, 2.231e-3 / 2.241e-3).  (The factors: in the group sums' place, which it does not use.)
        void* xn = (char*)ws + l.xn_off;
        if (wdt_split(c)) a.row_scale = a.Q;
        hipError_t e = launch_rmsnorm_weighted(X, norm_w, xn, wdt_split(c) ? a.Q : nullptr, M, d_model, eps, dtype, st);
        if (e != hipSuccess) return hip_fail(e);
        a.X = xn;
        a.norm_w = nullptr;
    }
    a.trace = nullptr;
    {
        size_t grid = (size_t)c.splits + (size_t)c.k2_splits * std::max(1, c.k2_col_blocks);   // covers every kernel's grid,
        if (c.kmajor == 2 || (wdt_split(c) && M > mfma_km_tokens_per_launch()))                 // but for those of token groups
            grid = std::max(grid, mfma_big_workgroups(c, M, d_ff));
        const Registered tr = snapshot(g_trace);
        if (tr.ptr && tr.bytes >= grid * 8 * sizeof(unsigned long long))
            a.trace = (unsigned long long*)tr.ptr;
    }
    // Token chunking on the host: a launch handles at most `per` tokens; further
    // chunks are further launches on the same stream (they re-stream the weights).
    const int per = c.path == DFK_PATH_MFMA ? mfma_max_tokens_per_launch(c, d_model) : valu_max_tokens_per_launch(c, M, d_model, d_ff, dtype);
    for (int m0 = 0; m0 < M; m0 += per) {
        a.m_base = m0;
        a.m_count = std::min(per, M - m0);
        hipError_t e = c.path == DFK_PATH_MFMA ? launch_mfma(a, c, st) : launch_valu(a, c, dtype, st);
        if (e != hipSuccess) return hip_fail(e);
    }
    return DFK_OK;
}

dfk_status_t run(const void* X, const void* Wg, const void* Wu, const void* Wd, void* Y, int M,
                 int d_model, int d_ff, dfk_dtype_t dtype, const dfk_config_t& c, void* ws,
                 hipStream_t st, const void* norm_w = nullptr, float eps = 0.f, const void* resid = nullptr) {
    return run_in(ws_layout(M, d_model, d_ff), X, Wg, Wu, Wd, Y, M, d_model, d_ff, dtype, c, ws, st, norm_w, eps, resid);
}

dfk_status_t call(const void* X, const void* Wg, const void* Wu, const void* Wd, void* Y, int M,
                  int d_model, int d_ff, dfk_dtype_t dtype, const dfk_config_t* cfg, int want_variant,
                  void* ws, size_t ws_bytes, void* stream, bool wd_t = false) {
    dfk_status_t s = check(X, Wg, Wu, Wd, Y, M, d_model, d_ff, dtype, cfg, ws, ws_bytes, true, false, wd_t);
    if (s != DFK_OK) return s;
    dfk_config_t c;
    if (cfg) c = *cfg;
    else if (wd_t ? !choose_wdt(M, d_model, d_ff, dtype, &c, nullptr)
                  : !choose(M, d_model, d_ff, dtype, want_variant, &c, nullptr)) return DFK_ERR_UNSUPPORTED_SHAPE;
    return run(X, Wg, Wu, Wd, Y, M, d_model, d_ff, dtype, c, ws, (hipStream_t)stream);
}

// ---------------------------------------------------------------- library-owned scratch (dfk_swiglu_mlp_static)
// One array per device, part of the code object, held until the process ends.  In host code its
// name is only a stand-in: the device address comes from hipGetSymbolAddress, once per device, and
// everything below uses that pointer.
constexpr size_t kStaticScratchBytes = (size_t)48 << 20;
constexpr size_t kStaticA2MaxBytes = (size_t)16 << 20;
}  // namespace
}  // namespace dfk

static __device__ __align__(256) unsigned char scratch[dfk::kStaticScratchBytes];

namespace dfk {
namespace {

constexpr int kStaticDevices = 32;
void* g_static_ptr[kStaticDevices];        // device address of `scratch` on each device, NULL until resolved
bool g_static_cleared[kStaticDevices];     // its counter / accumulator part has been zeroed once on that device

// The array's address on the current device (resolved at the first call on that device, with
// that device current), or an error.  *first is set where the caller must enqueue the one-time
// clearing of the part that has to be zero between calls.
hipError_t static_scratch(void** ptr, bool* first) {
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kStaticDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lk(g_mu);
    if (!g_static_ptr[dev]) {
        void* p = nullptr;
        e = hipGetSymbolAddress((void**)&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (!p || (uintptr_t)p % 256) return hipErrorInvalidSymbol;
        g_static_ptr[dev] = p;
    }
    *ptr = g_static_ptr[dev];
    *first = !g_static_cleared[dev];
    g_static_cleared[dev] = true;
    return hipSuccess;
}

// Layout inside the array: counters and accumulator first, as in a caller's workspace; then A_2
// at its exact size; what is left is divided 8 : 1 between the partial sums and the group sums.
bool static_layout(int M, int d_ff, WsLayout* l, size_t* p_bytes, size_t* q_bytes) {
    const size_t a2 = align_up((size_t)M * d_ff * 4, 256);
    if (a2 > kStaticA2MaxBytes) return false;
    l->tickets_off = 0;
    l->yacc_off = kWsHeaderBytes;
    l->a2_off = l->yacc_off + kYaccBytes;
    l->p_off = l->a2_off + a2;
    const size_t rest = kStaticScratchBytes - l->p_off;
    *q_bytes = rest / 9 / 256 * 256;
    *p_bytes = (rest - *q_bytes) / 256 * 256;
    l->q_off = l->p_off + *p_bytes;
    l->xn_off = l->total = kStaticScratchBytes;   // no normalised input: this entry point is the plain block
    return true;
}

// The partial-sum blocks a configuration writes in one launch fit p_bytes / q_bytes.
bool partials_fit_static(const dfk_config_t& c, int M, int d_model, int d_ff, dfk_dtype_t dtype, size_t p_bytes, size_t q_bytes) {
    if (c.reduce == DFK_REDUCE_ATOMIC) return true;   // accumulator only, already checked against its fixed size
    const int per = c.path == DFK_PATH_MFMA ? mfma_max_tokens_per_launch(c, d_model) : valu_max_tokens_per_launch(c, M, d_model, d_ff, dtype);
    const size_t tokens = (size_t)std::min(M, per);
    const bool fused = c.variant == DFK_VARIANT_FUSED && !roles_launch(c);
    const size_t blocks = fused ? (size_t)c.splits : (size_t)c.k2_splits;
    const size_t groups = fused ? (blocks + kGroupSize - 1) / kGroupSize : 0;
    return blocks * tokens * d_model * 4 <= p_bytes && groups * tokens * d_model * 4 <= q_bytes;
}

// ---------------------------------------------------------------- tuning scratch
struct Scratch {
    size_t w_bytes, x_bytes, ws_bytes, set_bytes, total;
};
Scratch scratch_layout(int M, int d_model, int d_ff, dfk_dtype_t dtype, int sets) {
    Scratch s;
    s.w_bytes = align_up((size_t)d_ff * d_model * elt_bytes(dtype), 256);
    s.x_bytes = align_up((size_t)M * d_model * elt_bytes(dtype), 256);
    s.ws_bytes = align_up(ws_layout(M, d_model, d_ff).total, 256);
    s.set_bytes = 3 * s.w_bytes;
    s.total = (size_t)sets * s.set_bytes + 2 * s.x_bytes + s.ws_bytes;
    return s;
}

dfk_status_t time_config(const dfk_config_t& c, int M, int d_model, int d_ff, dfk_dtype_t dtype,
                         void* scratch, int sets, int iters, hipStream_t st, bool fill, double* usec) {
    const Scratch s = scratch_layout(M, d_model, d_ff, dtype, sets);
    char* base = (char*)scratch;
    char* X = base + (size_t)sets * s.set_bytes;
    char* Y = X + s.x_bytes;
    char* ws = Y + s.x_bytes;
    hipError_t e;
    if (fill) {
        const float sg = sqrtf(3.0f / (float)d_model), sd = sqrtf(3.0f / (float)d_ff);
        for (int i = 0; i < sets; ++i) {
            char* w = base + (size_t)i * s.set_bytes;
            const size_t n = (size_t)d_ff * d_model;
            if ((e = launch_fill(w, n, dtype, sg, 11u + 3u * i, st)) != hipSuccess) return hip_fail(e);
            if ((e = launch_fill(w + s.w_bytes, n, dtype, sg, 12u + 3u * i, st)) != hipSuccess) return hip_fail(e);
            if ((e = launch_fill(w + 2 * s.w_bytes, n, dtype, sd, 13u + 3u * i, st)) != hipSuccess) return hip_fail(e);
        }
        if ((e = launch_fill(X, (size_t)M * d_model, dtype, 1.7320508f, 7u, st)) != hipSuccess) return hip_fail(e);
        if ((e = launch_zero(ws, s.ws_bytes, st)) != hipSuccess) return hip_fail(e);
    }
    hipEvent_t t0, t1;
    if ((e = hipEventCreate(&t0)) != hipSuccess) return hip_fail(e);
    if ((e = hipEventCreate(&t1)) != hipSuccess) { (void)hipEventDestroy(t0); return hip_fail(e); }
    dfk_status_t rc = DFK_OK;
    for (int it = -2; it < iters && rc == DFK_OK; ++it) {
        if (it == 0 && (e = hipEventRecord(t0, st)) != hipSuccess) { rc = hip_fail(e); break; }
        char* w = base + (size_t)((it + 2) % sets) * s.set_bytes;
        rc = run(X, w, w + s.w_bytes, w + 2 * s.w_bytes, Y, M, d_model, d_ff, dtype, c, ws, st);
    }
    if (rc == DFK_OK) {
        if ((e = hipEventRecord(t1, st)) != hipSuccess) rc = hip_fail(e);
        else if ((e = hipEventSynchronize(t1)) != hipSuccess) rc = hip_fail(e);
        else {
            float ms = 0.f;
            if ((e = hipEventElapsedTime(&ms, t0, t1)) != hipSuccess) rc = hip_fail(e);
            else *usec = (double)ms * 1000.0 / iters;
        }
    }
    (void)hipEventDestroy(t0);
    (void)hipEventDestroy(t1);
    return rc;
}

// Same protocol as time_config, for each launch of the call on its own: `iters` gate/up
// launches back to back between two events, then `iters` down launches (they read the A_2
// the last gate/up launch left; every launch leaves the workspace clean).
dfk_status_t time_kernels(const dfk_config_t& c, int M, int d_model, int d_ff, dfk_dtype_t dtype,
                          void* scratch, int sets, int iters, hipStream_t st, double* usec2) {
    double whole = 0.0;
    dfk_status_t rc = time_config(c, M, d_model, d_ff, dtype, scratch, sets, 1, st, true, &whole);   // fill + warm-up
    if (rc != DFK_OK) return rc;
    const Scratch s = scratch_layout(M, d_model, d_ff, dtype, sets);
    char* base = (char*)scratch;
    char* X = base + (size_t)sets * s.set_bytes;
    char* Y = X + s.x_bytes;
    char* ws = Y + s.x_bytes;
    hipEvent_t t0, t1;
    hipError_t e;
    if ((e = hipEventCreate(&t0)) != hipSuccess) return hip_fail(e);
    if ((e = hipEventCreate(&t1)) != hipSuccess) { (void)hipEventDestroy(t0); return hip_fail(e); }
    usec2[0] = usec2[1] = 0.0;
    const int stages = c.variant == DFK_VARIANT_FUSED && !roles_launch(c) ? 1 : 2;   // (head and tail of the launch with both roles)
    for (int k = 0; k < stages && rc == DFK_OK; ++k) {
        g_stage_mask = 1 << k;
        for (int it = -2; it < iters && rc == DFK_OK; ++it) {
            if (it == 0 && (e = hipEventRecord(t0, st)) != hipSuccess) { rc = hip_fail(e); break; }
            char* w = base + (size_t)((it + 2) % sets) * s.set_bytes;
            rc = run(X, w, w + s.w_bytes, w + 2 * s.w_bytes, Y, M, d_model, d_ff, dtype, c, ws, st);
        }
        g_stage_mask = 3;
        if (rc != DFK_OK) break;
        float ms = 0.f;
        if ((e = hipEventRecord(t1, st)) != hipSuccess || (e = hipEventSynchronize(t1)) != hipSuccess ||
            (e = hipEventElapsedTime(&ms, t0, t1)) != hipSuccess) { rc = hip_fail(e); break; }
        usec2[k] = (double)ms * 1000.0 / iters;
    }
    g_stage_mask = 3;
    (void)hipEventDestroy(t0);
    (void)hipEventDestroy(t1);
    return rc;
}

}  // namespace
}  // namespace dfk

using namespace dfk;

extern "C" {

dfk_status_t dfk_swiglu_mlp(const void* X, const void* Wg, const void* Wu, const void* Wd, void* Y,
                            int M, int d_model, int d_ff, void* stream) {
    const Registered ws = snapshot(g_ws);
    return call(X, Wg, Wu, Wd, Y, M, d_model, d_ff, DFK_BF16, nullptr, DFK_VARIANT_AUTO, ws.ptr, ws.bytes, stream);
}

dfk_status_t dfk_swiglu_mlp_fused(const void* X, const void* Wg, const void* Wu, const void* Wd,
                                  void* Y, int M, int d_model, int d_ff, void* stream) {
    const Registered ws = snapshot(g_ws);
    return call(X, Wg, Wu, Wd, Y, M, d_model, d_ff, DFK_BF16, nullptr, DFK_VARIANT_FUSED, ws.ptr, ws.bytes, stream);
}

dfk_status_t dfk_swiglu_mlp_unfused(const void* X, const void* Wg, const void* Wu, const void* Wd,
                                    void* Y, int M, int d_model, int d_ff, void* stream) {
    const Registered ws = snapshot(g_ws);
    return call(X, Wg, Wu, Wd, Y, M, d_model, d_ff, DFK_BF16, nullptr, DFK_VARIANT_TWO_KERNEL, ws.ptr, ws.bytes, stream);
}

dfk_status_t dfk_swiglu_mlp_ex(const void* X, const void* Wg, const void* Wu, const void* Wd, void* Y,
                               int M, int d_model, int d_ff, dfk_dtype_t dtype,
                               const dfk_config_t* cfg, void* workspace, size_t workspace_bytes,
                               void* stream) {
    return call(X, Wg, Wu, Wd, Y, M, d_model, d_ff, dtype, cfg, DFK_VARIANT_AUTO, workspace,
                workspace_bytes, stream);
}

dfk_status_t dfk_swiglu_mlp_wdt(const void* X, const void* Wg, const void* Wu, const void* Wd_t, void* Y,
                                int M, int d_model, int d_ff, dfk_dtype_t dtype,
                                const dfk_config_t* cfg, void* workspace, size_t workspace_bytes,
                                void* stream) {
    return call(X, Wg, Wu, Wd_t, Y, M, d_model, d_ff, dtype, cfg, DFK_VARIANT_AUTO, workspace,
                workspace_bytes, stream, true);
}

dfk_status_t dfk_swiglu_mlp_static(const void* X, const void* Wg, const void* Wu, const void* Wd, void* Y,
                                   int M, int d_model, int d_ff, dfk_dtype_t dtype, const dfk_config_t* cfg,
                                   void* stream) {
    dfk_status_t s = check(X, Wg, Wu, Wd, Y, M, d_model, d_ff, dtype, cfg, nullptr, 0, false);
    if (s != DFK_OK) return s;
    WsLayout l;
    size_t p_bytes = 0, q_bytes = 0;
    if (!static_layout(M, d_ff, &l, &p_bytes, &q_bytes)) return DFK_ERR_WORKSPACE;   // A_2 beyond the array's share
    dfk_config_t c;
    if (cfg) {
        c = *cfg;
        if (!partials_fit_static(c, M, d_model, d_ff, dtype, p_bytes, q_bytes)) return DFK_ERR_WORKSPACE;
    } else {
        if (!choose(M, d_model, d_ff, dtype, DFK_VARIANT_AUTO, &c, nullptr)) return DFK_ERR_UNSUPPORTED_SHAPE;
        auto fits = [&](const dfk_config_t& k) { return partials_fit_static(k, M, d_model, d_ff, dtype, p_bytes, q_bytes); };
        if (!fits(c) && !enumerate_default(M, d_model, d_ff, dtype, DFK_VARIANT_AUTO, &c, fits)) return DFK_ERR_WORKSPACE;
    }
    void* ws = nullptr;
    bool first = false;
    if (hipError_t e = static_scratch(&ws, &first); e != hipSuccess) return hip_fail(e);
    const size_t nx = (size_t)M * d_model * elt_bytes(dtype), nw = (size_t)d_ff * d_model * elt_bytes(dtype);
    if (overlaps(ws, kStaticScratchBytes, Y, nx) || overlaps(ws, kStaticScratchBytes, X, nx) ||
        overlaps(ws, kStaticScratchBytes, Wg, nw) || overlaps(ws, kStaticScratchBytes, Wu, nw) ||
        overlaps(ws, kStaticScratchBytes, Wd, nw))
        return DFK_ERR_ALIAS;
    if (first) {   // counters and accumulator start from zero (a fill kernel on the caller's stream); calls keep them zero
        if (hipError_t e = launch_zero(ws, kWsHeaderBytes + kYaccBytes, (hipStream_t)stream); e != hipSuccess) return hip_fail(e);
    }
    return run_in(l, X, Wg, Wu, Wd, Y, M, d_model, d_ff, dtype, c, ws, (hipStream_t)stream);
}

namespace {
// Whether a configuration (valid for the problem) runs the block too.
bool block_carries(const dfk_config_t& k, int M, int d_model, int d_ff, dfk_dtype_t dtype) {
    if (k.path != DFK_PATH_MFMA) return false;
    if (k.kmajor == 5 || k.kmajor == 2) return mfma_config_valid(k, M, d_model, d_ff, dtype);
    if (k.variant == DFK_VARIANT_FUSED) return k.kmajor == 4 && mfma_km_block_config_valid(k, M, d_model, d_ff, dtype);
    return k.kmajor == 1 && d_model % 128 == 0 && mfma_km_config_valid(k, M, d_model, d_ff, dtype);
}
// The block's configuration without one from the caller: the choice of its layout (of the two-kernel variant), else the first
// candidate that carries it; the pair for up to 64 tokens, tuned or not, in the form of a single launch where that pays.
bool choose_block(int M, int d_model, int d_ff, dfk_dtype_t dtype, bool wd_t, dfk_config_t* out, int* tuned) {
    dfk_config_t c;
    if (wd_t ? !choose_wdt(M, d_model, d_ff, dtype, &c, tuned)
             : !choose(M, d_model, d_ff, dtype, DFK_VARIANT_TWO_KERNEL, &c, tuned)) return false;
    if (!block_carries(c, M, d_model, d_ff, dtype)) {
        if (tuned) *tuned = 0;
        bool found = false;
        for (const auto& k : wd_t ? candidates_wdt(M, d_model, d_ff, dtype) : candidates(M, d_model, d_ff, dtype))
            if (k.variant == DFK_VARIANT_TWO_KERNEL && block_carries(k, M, d_model, d_ff, dtype)) { c = k; found = true; break; }
        if (!found) return false;
    }
    if (!wd_t && single_launch_pays(M, d_model, d_ff)) single_launch_of(c, M, d_model, d_ff, dtype, true, &c);
    *out = c;
    return true;
}

dfk_status_t mlp_block(const void* H, const void* norm_weight, float eps, const void* Wg,
                       const void* Wu, const void* Wd, void* H_out, int M, int d_model, int d_ff,
                       dfk_dtype_t dtype, const dfk_config_t* cfg, void* workspace,
                       size_t workspace_bytes, void* stream, bool wd_t) {
    if (!H || !norm_weight || !H_out) return DFK_ERR_INVALID_ARG;
    if (!(eps >= 0.f) || !(eps < 1e30f)) return DFK_ERR_INVALID_ARG;
    if (dtype != DFK_BF16 && dtype != DFK_FP16)
        return dtype == DFK_FP32 ? DFK_ERR_UNSUPPORTED_SHAPE : DFK_ERR_INVALID_ARG;
    if ((uintptr_t)norm_weight % 16) return DFK_ERR_ALIGNMENT;
    // The output may be the input itself (the residual stream updated in place); any other
    // overlap is refused.
    dfk_status_t s = check(H, Wg, Wu, Wd, H_out, M, d_model, d_ff, dtype, cfg, workspace, workspace_bytes, true, true, wd_t);
    if (s != DFK_OK) return s;
    {
        const size_t nx = (size_t)M * d_model * 2, nv = (size_t)d_model * 2;
        if (overlaps(H_out, nx, norm_weight, nv) || overlaps(workspace, workspace_bytes, norm_weight, nv))
            return DFK_ERR_ALIAS;
    }
    dfk_config_t c;
    if (cfg) {
        if (!block_carries(*cfg, M, d_model, d_ff, dtype)) return DFK_ERR_UNSUPPORTED_SHAPE;
        c = *cfg;
    } else if (!choose_block(M, d_model, d_ff, dtype, wd_t, &c, nullptr)) {
        return DFK_ERR_UNSUPPORTED_SHAPE;
    }
    return run(H, Wg, Wu, Wd, H_out, M, d_model, d_ff, dtype, c, workspace, (hipStream_t)stream, norm_weight, eps, H);
}
}  // namespace

dfk_status_t dfk_mlp_block(const void* H, const void* norm_weight, float eps, const void* Wg,
                           const void* Wu, const void* Wd, void* H_out, int M, int d_model, int d_ff,
                           dfk_dtype_t dtype, const dfk_config_t* cfg, void* workspace,
                           size_t workspace_bytes, void* stream) {
    return mlp_block(H, norm_weight, eps, Wg, Wu, Wd, H_out, M, d_model, d_ff, dtype, cfg, workspace, workspace_bytes, stream, false);
}

dfk_status_t dfk_mlp_block_wdt(const void* H, const void* norm_weight, float eps, const void* Wg,
                               const void* Wu, const void* Wd_t, void* H_out, int M, int d_model, int d_ff,
                               dfk_dtype_t dtype, const dfk_config_t* cfg, void* workspace,
                               size_t workspace_bytes, void* stream) {
    return mlp_block(H, norm_weight, eps, Wg, Wu, Wd_t, H_out, M, d_model, d_ff, dtype, cfg, workspace, workspace_bytes, stream, true);
}

dfk_status_t dfk_check_args(const void* X, const void* Wg, const void* Wu, const void* Wd,
                            const void* Y, int M, int d_model, int d_ff, dfk_dtype_t dtype,
                            const dfk_config_t* cfg, const void* workspace, size_t workspace_bytes) {
    return check(X, Wg, Wu, Wd, Y, M, d_model, d_ff, dtype, cfg, workspace, workspace_bytes, false);
}

size_t dfk_workspace_bytes(int M_max, int d_model, int d_ff) {
    if (!shape_supported(M_max, d_model, d_ff)) return 0;
    return ws_layout(M_max, d_model, d_ff).total;
}

dfk_status_t dfk_workspace_init(void* workspace, size_t workspace_bytes, void* stream) {
    if (!workspace || workspace_bytes == 0) return DFK_ERR_INVALID_ARG;
    if ((uintptr_t)workspace % 256) return DFK_ERR_ALIGNMENT;
    hipError_t e = launch_zero(workspace, workspace_bytes, (hipStream_t)stream);
    return e == hipSuccess ? DFK_OK : hip_fail(e);
}

dfk_status_t dfk_set_workspace(void* workspace, size_t workspace_bytes) {
    if (workspace && (uintptr_t)workspace % 256) return DFK_ERR_ALIGNMENT;
    if (workspace && workspace_bytes == 0) return DFK_ERR_INVALID_ARG;
    std::lock_guard<std::mutex> lk(g_mu);
    g_ws.ptr = workspace;
    g_ws.bytes = workspace ? workspace_bytes : 0;
    return DFK_OK;
}

dfk_status_t dfk_set_trace_buffer(void* buffer, size_t bytes) {
    if (buffer && (uintptr_t)buffer % 8) return DFK_ERR_ALIGNMENT;
    std::lock_guard<std::mutex> lk(g_mu);
    g_trace.ptr = buffer;
    g_trace.bytes = buffer ? bytes : 0;
    return DFK_OK;
}

int dfk_num_candidates_wdt(int M, int d_model, int d_ff, dfk_dtype_t dtype) {
    if (!shape_supported(M, d_model, d_ff)) return 0;
    return (int)candidates_wdt(M, d_model, d_ff, dtype).size();
}

dfk_status_t dfk_get_candidate_wdt(int M, int d_model, int d_ff, dfk_dtype_t dtype, int i, dfk_config_t* out) {
    if (!out) return DFK_ERR_INVALID_ARG;
    if (!shape_supported(M, d_model, d_ff)) return DFK_ERR_UNSUPPORTED_SHAPE;
    auto c = candidates_wdt(M, d_model, d_ff, dtype);
    if (i < 0 || i >= (int)c.size()) return DFK_ERR_NOT_FOUND;
    *out = c[i];
    return DFK_OK;
}

dfk_status_t dfk_get_choice_wdt(int M, int d_model, int d_ff, dfk_dtype_t dtype, dfk_config_t* out, int* tuned_out) {
    if (!out) return DFK_ERR_INVALID_ARG;
    if (M < 1 || d_model < 1 || d_ff < 1) return DFK_ERR_INVALID_ARG;
    if (!shape_supported(M, d_model, d_ff)) return DFK_ERR_UNSUPPORTED_SHAPE;
    return choose_wdt(M, d_model, d_ff, dtype, out, tuned_out) ? DFK_OK : DFK_ERR_UNSUPPORTED_SHAPE;
}

dfk_status_t dfk_get_choice_block(int M, int d_model, int d_ff, dfk_dtype_t dtype, int w_down_t, dfk_config_t* out,
                                  int* tuned_out) {
    if (!out) return DFK_ERR_INVALID_ARG;
    if (M < 1 || d_model < 1 || d_ff < 1) return DFK_ERR_INVALID_ARG;
    if (dtype != DFK_BF16 && dtype != DFK_FP16) return dtype == DFK_FP32 ? DFK_ERR_UNSUPPORTED_SHAPE : DFK_ERR_INVALID_ARG;
    if (!shape_supported(M, d_model, d_ff)) return DFK_ERR_UNSUPPORTED_SHAPE;
    return choose_block(M, d_model, d_ff, dtype, w_down_t != 0, out, tuned_out) ? DFK_OK : DFK_ERR_UNSUPPORTED_SHAPE;
}

int dfk_num_candidates(int M, int d_model, int d_ff, dfk_dtype_t dtype) {
    if (!shape_supported(M, d_model, d_ff)) return 0;
    return (int)candidates(M, d_model, d_ff, dtype).size();
}

dfk_status_t dfk_get_candidate(int M, int d_model, int d_ff, dfk_dtype_t dtype, int i,
                               dfk_config_t* out) {
    if (!out) return DFK_ERR_INVALID_ARG;
    if (!shape_supported(M, d_model, d_ff)) return DFK_ERR_UNSUPPORTED_SHAPE;
    auto c = candidates(M, d_model, d_ff, dtype);
    if (i < 0 || i >= (int)c.size()) return DFK_ERR_NOT_FOUND;
    *out = c[i];
    return DFK_OK;
}

int dfk_config_valid(const dfk_config_t* cfg, int M, int d_model, int d_ff, dfk_dtype_t dtype) {
    if (!cfg) return 0;
    return config_valid(*cfg, M, d_model, d_ff, dtype) ? 1 : 0;
}

size_t dfk_tune_scratch_bytes(int M_max, int d_model, int d_ff, dfk_dtype_t dtype, int sets) {
    if (!shape_supported(M_max, d_model, d_ff) || sets < 1) return 0;
    return scratch_layout(M_max, d_model, d_ff, dtype, sets).total;
}

dfk_status_t dfk_time_config(const dfk_config_t* cfg, int M, int d_model, int d_ff, dfk_dtype_t dtype,
                             void* scratch, size_t scratch_bytes, int sets, int iters, void* stream,
                             double* usec_out) {
    if (!cfg || !scratch || !usec_out || sets < 1 || iters < 1) return DFK_ERR_INVALID_ARG;
    if (M < 1 || d_model < 1 || d_ff < 1) return DFK_ERR_INVALID_ARG;
    if (!shape_supported(M, d_model, d_ff)) return DFK_ERR_UNSUPPORTED_SHAPE;
    if (!config_valid(*cfg, M, d_model, d_ff, dtype)) return DFK_ERR_UNSUPPORTED_SHAPE;
    if ((uintptr_t)scratch % 256) return DFK_ERR_ALIGNMENT;
    if (scratch_bytes < scratch_layout(M, d_model, d_ff, dtype, sets).total) return DFK_ERR_WORKSPACE;
    return time_config(*cfg, M, d_model, d_ff, dtype, scratch, sets, iters, (hipStream_t)stream, true,
                       usec_out);
}

dfk_status_t dfk_time_kernels(const dfk_config_t* cfg, int M, int d_model, int d_ff, dfk_dtype_t dtype,
                              void* scratch, size_t scratch_bytes, int sets, int iters, void* stream,
                              double* usec_out) {
    if (!cfg || !scratch || !usec_out || sets < 1 || iters < 1 || iters > 1024) return DFK_ERR_INVALID_ARG;
    if (M < 1 || d_model < 1 || d_ff < 1) return DFK_ERR_INVALID_ARG;
    if (!shape_supported(M, d_model, d_ff)) return DFK_ERR_UNSUPPORTED_SHAPE;
    if (!config_valid(*cfg, M, d_model, d_ff, dtype)) return DFK_ERR_UNSUPPORTED_SHAPE;
    const int per = cfg->path == DFK_PATH_MFMA ? mfma_max_tokens_per_launch(*cfg, d_model) : valu_max_tokens_per_launch(*cfg, M, d_model, d_ff, dtype);
    if (M > per) return DFK_ERR_UNSUPPORTED_SHAPE;   // one set of launches per call only
    if ((uintptr_t)scratch % 256) return DFK_ERR_ALIGNMENT;
    if (scratch_bytes < scratch_layout(M, d_model, d_ff, dtype, sets).total) return DFK_ERR_WORKSPACE;
    return time_kernels(*cfg, M, d_model, d_ff, dtype, scratch, sets, iters, (hipStream_t)stream, usec_out);
}

// Whether two candidates of the 256-token pair make the same launches of M tokens: its rules (dfk_big_plan.h) can make one count of
// slices or splits of several configured ones, and its kernels take neither waves nor depth.  Tuning times such a launch once, under the
// first of its names in the list, which is the untuned one where that is among them.
static bool same_big_launches(const dfk_config_t& a, const dfk_config_t& b, int M, int d_ff) {
    auto of_pair = [&](const dfk_config_t& c) { return c.kmajor == 2 || (wdt_split(c) && M > mfma_km_tokens_per_launch()); };
    if (!of_pair(a) || !of_pair(b) || a.kmajor != b.kmajor || a.reduce != b.reduce || a.k2_col_blocks != b.k2_col_blocks) return false;
    auto up = [&](const dfk_config_t& c) { return big_gateup_launch(M, d_ff, c.splits); };
    auto down = [&](const dfk_config_t& c) { return big_down_launch(M, d_ff, c.k2_splits, c.k2_col_blocks, wdt_split(c), c.reduce == DFK_REDUCE_TICKET); };
    return up(a).splits == up(b).splits && up(a).groups == up(b).groups && down(a).splits == down(b).splits;
}

dfk_status_t dfk_tune(const int* M_list, int nM, int d_model, int d_ff, dfk_dtype_t dtype,
                      void* scratch, size_t scratch_bytes, int sets, int iters, void* stream) {
    if (!M_list || nM < 1 || !scratch || sets < 1 || iters < 1) return DFK_ERR_INVALID_ARG;
    if (d_model < 1 || d_ff < 1) return DFK_ERR_INVALID_ARG;
    if (!shape_supported(1, d_model, d_ff)) return DFK_ERR_UNSUPPORTED_SHAPE;
    if ((uintptr_t)scratch % 256) return DFK_ERR_ALIGNMENT;
    for (int i = 0; i < nM; ++i) {
        if (M_list[i] < 1) return DFK_ERR_INVALID_ARG;
        if (M_list[i] > DFK_MAX_M) return DFK_ERR_UNSUPPORTED_SHAPE;
        if (scratch_bytes < scratch_layout(M_list[i], d_model, d_ff, dtype, sets).total)
            return DFK_ERR_WORKSPACE;
    }
    g_tune_skipped = 0;
    g_tune_skip_status = DFK_OK;
    for (int i = 0; i < nM; ++i) {
        const int M = M_list[i];
        auto cands = candidates(M, d_model, d_ff, dtype);
        if (cands.empty()) return DFK_ERR_UNSUPPORTED_SHAPE;
        const size_t listed = cands.size();
        for (size_t k = 0; d_model % 128 && k < listed; ++k) {   // the pair's other form, which is not listed there
            dfk_config_t one;
            if (!single_launch_of(cands[k], M, d_model, d_ff, dtype, false, &one)) continue;
            auto same = [&](const dfk_config_t& o) { return same_cfg(o, one); };
            if (std::none_of(cands.begin(), cands.end(), same)) cands.push_back(one);
        }
        Entry best, best_of[3];
        best.usec = best_of[1].usec = best_of[2].usec = -1.0;
        bool fill = true;  // scratch layout depends on M: refill once per M (until a candidate has run)
        for (size_t k = 0; k < cands.size(); ++k) {
            const dfk_config_t& c = cands[k];
            if (std::any_of(cands.begin(), cands.begin() + k, [&](const dfk_config_t& o) { return same_big_launches(o, c, M, d_ff); })) continue;
            double us = 0.0;
            dfk_status_t s = time_config(c, M, d_model, d_ff, dtype, scratch, sets, iters,
                                         (hipStream_t)stream, fill, &us);
            if (s != DFK_OK) {   // a candidate that cannot be timed is left out, not the whole tune
                ++g_tune_skipped;
                g_tune_skip_status = s;
                continue;
            }
            fill = false;
            if (best.usec < 0.0 || us < best.usec) { best.cfg = c; best.usec = us; }
            if (k >= listed) continue;                            // (no entry of a variant, see table_put)
            Entry& bv = best_of[c.variant == DFK_VARIANT_FUSED ? 1 : 2];
            if (bv.usec < 0.0 || us < bv.usec) { bv.cfg = c; bv.usec = us; }
        }
        if (best.usec < 0.0) return g_tune_skip_status;   // every candidate of this M failed
        // the candidates for W_down as [d_model, d_ff] (timing does not depend on what the synthetic weights mean)
        Entry best_t;
        best_t.usec = -1.0;
        const auto cands_t = candidates_wdt(M, d_model, d_ff, dtype);
        for (size_t k = 0; k < cands_t.size(); ++k) {
            const dfk_config_t& c = cands_t[k];
            if (std::any_of(cands_t.begin(), cands_t.begin() + k, [&](const dfk_config_t& o) { return same_big_launches(o, c, M, d_ff); })) continue;
            if (cands_t[0].a2_dtype == DFK_FP32 && c.a2_dtype != DFK_FP32) continue;   // being faster is no reason to round A_2
            double us = 0.0;
            dfk_status_t s = time_config(c, M, d_model, d_ff, dtype, scratch, sets, iters, (hipStream_t)stream, false, &us);
            if (s != DFK_OK) {
                ++g_tune_skipped;
                g_tune_skip_status = s;
                continue;
            }
            if (best_t.usec < 0.0 || us < best_t.usec) { best_t.cfg = c; best_t.usec = us; }
        }
        std::lock_guard<std::mutex> lk(g_mu);
        for (int v = 1; v <= 2; ++v)
            if (best_of[v].usec >= 0.0) table_put(M, d_model, d_ff, (int)dtype, best_of[v], false);
        if (best_t.usec >= 0.0) table_put(M, d_model, d_ff, (int)dtype, best_t, false);
        table_put(M, d_model, d_ff, (int)dtype, best, true);
    }
    return DFK_OK;
}

int dfk_tune_skipped(dfk_status_t* last_status_out) {
    if (last_status_out) *last_status_out = g_tune_skip_status;
    return g_tune_skipped;
}

dfk_status_t dfk_get_choice(int M, int d_model, int d_ff, dfk_dtype_t dtype, dfk_config_t* out,
                            int* tuned_out) {
    if (!out) return DFK_ERR_INVALID_ARG;
    if (M < 1 || d_model < 1 || d_ff < 1) return DFK_ERR_INVALID_ARG;
    if (!shape_supported(M, d_model, d_ff)) return DFK_ERR_UNSUPPORTED_SHAPE;
    return choose(M, d_model, d_ff, dtype, DFK_VARIANT_AUTO, out, tuned_out) ? DFK_OK
                                                                             : DFK_ERR_UNSUPPORTED_SHAPE;
}

dfk_status_t dfk_set_choice(int M, int d_model, int d_ff, dfk_dtype_t dtype, const dfk_config_t* cfg,
                            double usec) {
    if (!cfg || M < 1 || d_model < 1 || d_ff < 1) return DFK_ERR_INVALID_ARG;
    if (!shape_supported(M, d_model, d_ff)) return DFK_ERR_UNSUPPORTED_SHAPE;
    if (!config_valid(*cfg, M, d_model, d_ff, dtype)) return DFK_ERR_UNSUPPORTED_SHAPE;
    std::lock_guard<std::mutex> lk(g_mu);
    Entry e;
    e.cfg = *cfg;
    e.usec = usec;
    table_put(M, d_model, d_ff, (int)dtype, e, true);
    return DFK_OK;
}

void dfk_clear_tuning(void) {
    std::lock_guard<std::mutex> lk(g_mu);
    g_table.clear();
}

dfk_status_t dfk_save_tuning(const char* path) {
    if (!path) return DFK_ERR_INVALID_ARG;
    std::lock_guard<std::mutex> lk(g_mu);
    FILE* f = std::fopen(path, "w");
    if (!f) return DFK_ERR_IO;
    std::fprintf(f, "# dfk tuning table v3: M d_model d_ff dtype variant path splits waves depth reduce "
                    "k2_splits k2_col_blocks a2_dtype k2_rows_by_wave kmajor usec\n");
    // One line per entry; a problem's chosen configuration comes after its other variant's line, and the loader
    // takes the last line of a problem as the choice.
    for (int pass = 0; pass < 2; ++pass)
        for (const auto& kv : g_table) {
            const int slot = std::get<4>(kv.first);
            const dfk_config_t& c = kv.second.cfg;
            if (pass == 0) {
                if (slot == 0) continue;
                auto chosen = g_table.find(Key(std::get<0>(kv.first), std::get<1>(kv.first), std::get<2>(kv.first),
                                               std::get<3>(kv.first), 0));
                if (chosen != g_table.end() && same_cfg(chosen->second.cfg, c)) continue;   // written in the second pass
            } else if (slot != 0) {
                continue;
            }
            std::fprintf(f, "%d %d %d %d %d %d %d %d %d %d %d %d %d %d %d %.3f\n", std::get<0>(kv.first),
                         std::get<1>(kv.first), std::get<2>(kv.first), std::get<3>(kv.first), c.variant,
                         c.path, c.splits, c.waves, c.depth, c.reduce, c.k2_splits, c.k2_col_blocks,
                         c.a2_dtype, c.k2_rows_by_wave, c.kmajor, kv.second.usec);
        }
    const bool ok = std::fclose(f) == 0;
    return ok ? DFK_OK : DFK_ERR_IO;
}

// A line of a version 2 table: there path VALU with a column block per 128 columns was the name of what is path VALU with kmajor = 1 since.
static void rename_v2(dfk_config_t* c, int M, int d_model, int d_ff, dfk_dtype_t dtype) {
    dfk_config_t n = *c;
    n.kmajor = 1; n.depth = c->waves == 8 ? 3 : 6;
    if (c->kmajor == 0 && half_off_128(n, M, d_model, d_ff, dtype, nullptr) && c->k2_col_blocks == (d_model + 127) / 128) *c = n;
}

dfk_status_t dfk_load_tuning(const char* path) {
    if (!path) return DFK_ERR_INVALID_ARG;
    FILE* f = std::fopen(path, "r");
    if (!f) return DFK_ERR_IO;
    std::vector<std::pair<Key, Entry>> fresh;   // in file order
    char line[512];
    dfk_status_t rc = DFK_OK;
    int version = 0;
    while (std::fgets(line, sizeof line, f)) {
        const char* p = line;
        while (*p == ' ' || *p == '\t') ++p;
        (void)std::sscanf(p, "# dfk tuning table v%d", &version);
        if (*p == '#' || *p == '\n' || *p == '\r' || *p == 0) continue;
        int M, dm, df, dt;
        Entry e;
        std::memset(&e, 0, sizeof e);
        const int n = std::sscanf(p, "%d %d %d %d %d %d %d %d %d %d %d %d %d %d %d %lf", &M, &dm, &df, &dt,
                                  &e.cfg.variant, &e.cfg.path, &e.cfg.splits, &e.cfg.waves, &e.cfg.depth,
                                  &e.cfg.reduce, &e.cfg.k2_splits, &e.cfg.k2_col_blocks, &e.cfg.a2_dtype,
                                  &e.cfg.k2_rows_by_wave, &e.cfg.kmajor, &e.usec);
        if (n != 16 || M < 1 || M > DFK_MAX_M || (dt != DFK_BF16 && dt != DFK_FP32 && dt != DFK_FP16) || dm < 8 ||
            df < 8 || dm % 8 || df % 8) {
            rc = DFK_ERR_IO;
            break;
        }
        if (version == 2) rename_v2(&e.cfg, M, dm, df, (dfk_dtype_t)dt);
        if (!config_valid(e.cfg, M, dm, df, (dfk_dtype_t)dt)) {
            rc = DFK_ERR_IO;
            break;
        }
        fresh.emplace_back(Key(M, dm, df, dt, 0), e);
    }
    std::fclose(f);
    if (rc != DFK_OK) return rc;  // table left untouched on a malformed file
    std::lock_guard<std::mutex> lk(g_mu);
    for (const auto& kv : fresh)
        table_put(std::get<0>(kv.first), std::get<1>(kv.first), std::get<2>(kv.first), std::get<3>(kv.first), kv.second, true);
    return DFK_OK;
}

dfk_status_t dfk_transpose_w_down(const void* Wd, void* Wd_t, int d_model, int d_ff, dfk_dtype_t dtype, void* stream) {
    if (!Wd || !Wd_t || d_model < 1 || d_ff < 1) return DFK_ERR_INVALID_ARG;
    if (dtype != DFK_BF16 && dtype != DFK_FP32 && dtype != DFK_FP16) return DFK_ERR_INVALID_ARG;
    if ((uintptr_t)Wd % 16 || (uintptr_t)Wd_t % 16) return DFK_ERR_ALIGNMENT;
    if ((d_ff + 31) / 32 > 65535) return DFK_ERR_UNSUPPORTED_SHAPE;
    const size_t nw = (size_t)d_ff * d_model * elt_bytes(dtype);
    if (overlaps(Wd, nw, Wd_t, nw)) return DFK_ERR_ALIAS;
    hipError_t e = launch_transpose(Wd, Wd_t, d_ff, d_model, dtype, (hipStream_t)stream);
    return e == hipSuccess ? DFK_OK : hip_fail(e);
}

dfk_status_t dfk_rms_normalize(const void* in, void* out, int M, int d_model, void* stream) {
    if (!in || !out || M < 1 || d_model < 1) return DFK_ERR_INVALID_ARG;
    if (M > 65535) return DFK_ERR_UNSUPPORTED_SHAPE;
    hipError_t e = launch_rms_normalize(in, out, M, d_model, (hipStream_t)stream);
    return e == hipSuccess ? DFK_OK : hip_fail(e);
}

dfk_status_t dfk_stream_read(const void* src, size_t bytes, void* sink, void* stream) {
    if (!src || !sink || bytes == 0) return DFK_ERR_INVALID_ARG;
    if (bytes % 16) return DFK_ERR_UNSUPPORTED_SHAPE;
    if ((uintptr_t)src % 16 || (uintptr_t)sink % 8) return DFK_ERR_ALIGNMENT;
    hipError_t e = launch_stream_read(src, bytes, sink, (hipStream_t)stream);
    return e == hipSuccess ? DFK_OK : hip_fail(e);
}

dfk_status_t dfk_read_gateup_pattern(const void* Wg, const void* Wu, int d_model, int d_ff, int splits, int waves,
                                     void* sink, void* stream) {
    if (!Wg || !Wu || !sink || d_model < 1 || d_ff < 1 || splits < 1) return DFK_ERR_INVALID_ARG;
    if (waves != 4 && waves != 8) return DFK_ERR_INVALID_ARG;
    if (d_ff % 8 || d_model % (128 * waves) || d_model > kMaxDModel || splits > d_ff / 8 || splits > 65535)
        return DFK_ERR_UNSUPPORTED_SHAPE;
    if ((uintptr_t)Wg % 16 || (uintptr_t)Wu % 16 || (uintptr_t)sink % 8) return DFK_ERR_ALIGNMENT;
    hipError_t e = launch_read_gateup_pattern(Wg, Wu, d_model, d_ff, splits, waves, sink, (hipStream_t)stream);
    return e == hipSuccess ? DFK_OK : hip_fail(e);
}

dfk_status_t dfk_fill_synthetic(void* dst, size_t elems, dfk_dtype_t dtype, float scale, unsigned seed,
                                void* stream) {
    if (!dst || elems == 0) return DFK_ERR_INVALID_ARG;
    if (dtype != DFK_BF16 && dtype != DFK_FP32 && dtype != DFK_FP16) return DFK_ERR_INVALID_ARG;
    if ((uintptr_t)dst % 4) return DFK_ERR_ALIGNMENT;
    hipError_t e = launch_fill(dst, elems, dtype, scale, seed, (hipStream_t)stream);
    return e == hipSuccess ? DFK_OK : hip_fail(e);
}

const char* dfk_status_string(dfk_status_t s) {
    switch (s) {
        case DFK_OK: return "ok";
        case DFK_ERR_INVALID_ARG: return "invalid argument";
        case DFK_ERR_UNSUPPORTED_SHAPE: return "unsupported shape or configuration";
        case DFK_ERR_ALIGNMENT: return "pointer not sufficiently aligned";
        case DFK_ERR_ALIAS: return "output or workspace overlaps an input";
        case DFK_ERR_WORKSPACE: return "workspace missing or too small";
        case DFK_ERR_HIP: return "HIP call failed";
        case DFK_ERR_IO: return "tuning file could not be read, written or parsed";
        case DFK_ERR_NOT_FOUND: return "not found";
    }
    return "unknown status";
}

int dfk_last_hip_error(void) { return g_last_hip_error; }

const char* dfk_version(void) { return "dfk 0.2 (gfx950)"; }

}  // extern "C"
