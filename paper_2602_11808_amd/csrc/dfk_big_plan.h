// Which launches the 256-token pair makes of a configuration: slices, splits and token groups, by rules on sizes.  Free of device code, so
// that a host program can check it.
#pragma once

#include <algorithm>

namespace dfk {

constexpr int kBigMaxRowTiles = 8;    // row tiles (8 d_ff rows each) of a slice in the gate/up kernel
// The same in its wide form, by token tiles per group (0: it is not built for them): with three and four, as many (an even number) as LDS
// holds three buffers of beside three of X; with two it would hold 18, and is built for 16, which are one round of 256 workgroups up to a
// d_ff of 32768.
constexpr int big_wide_tiles(int token_tiles) { return token_tiles == 2 ? 16 : token_tiles == 3 ? 14 : token_tiles == 4 ? 10 : 0; }
constexpr int big_token_tiles(int tokens) { return (tokens + 63) / 64; }   // of 16 tokens, per wavefront group of a workgroup

// One launch: workgroups along grid x (slices of d_ff; d_ff splits of the down projection, per column block) and token groups along grid
// y, of `tokens` each (a multiple of 64, or all there are).  `row`: grid x, with the workgroups that have no work.
struct BigLaunch { int splits, groups, tokens, row; };

inline BigLaunch big_divide(int m_count, int groups, int splits, int row) {
    const int tokens = groups > 1 ? ((m_count + groups - 1) / groups + 63) / 64 * 64 : m_count;
    return BigLaunch{splits, (m_count + tokens - 1) / tokens, tokens, row};
}

// Token groups (grid y): workgroups that each take a part of the launch's tokens, over fewer slices or splits of the weights.  What a
// gate/up workgroup reads per step is its tokens of X and its rows of the weights; one of 256 on a narrow layer has one to four row
// tiles beside up to 256 tokens, so most of the bytes that pass through its CU are X.  Half the tokens over twice the rows are fewer; the weights come out of
// L2 the second time.  It pays while the rows (at most eight tiles) stay few against the tokens saved.  Whole call, us, one group / two:
// beyond 192 tokens, at 230 or 256, 2048 x 2048 38.4 / 33.1, 3072 x 3072 53.0 / 42.8, 4096 x 4096 64.8 / 55.5, 2048 x 5504 49.4 / 47.2, 2304 x 8192
// 59.5 / 56.8, 8192 x 7168 142.7 / 128.9; up to 192 with four tiles, 160 tokens: 2048 x 2048 34.4 / 29.6, 1024 x 3840 29.5 / 27.8, 4096 x 4096 56.9 /
// 52.9, other side, 150: 2560 x 5120 47.6 / 49.8, 3072 x 8192 60.7 / 63.6, 4096 x 8192 73.2 / 73.1; up to 128 with three (two 64-k pieces share a step
// there), 114: 2048 x 2048 26.6 / 25.3, 3072 x 3072 37.8 / 35.8, other side: 1024 x 3840 23.9 / 24.9, 4096 x 4096 44.5 / 49.0.  Four groups are never the best.
inline int big_gateup_groups(int m_count, int d_ff) {
    const int tiles = (d_ff / 8 + 127) / 128;          // of the longest of 128 slices
    return m_count > 64 && tiles <= (m_count > 192 ? 8 : m_count > 128 ? 4 : 3) ? 2 : 1;
}
// Slices of the gate/up kernel: as many rounds of 256 workgroups as the wide form needs, where that is fewer than the given splits are.
// Each round reads all of X anew; that outweighs whatever else differs at both ends of the range.  Whole call, us, slices of up to eight
// tiles / wide: 4096 x 28672 at 70 tokens 144.1 / 129.0, 1024 x 20480 at 100 49.2 / 45.7 (W_down as [d_model, d_ff] 48.8 / 44.4), 5120 x 17408
// (nine tiles) at 100, 150 and 256 144.2 / 125.4, 172.0 / 144.6, 208.0 / 180.1, 2048 x 28672 at 160 105.8 / 97.0, block 8192 x 28672 at 150
// 336 / 311, 12288 x 22528 at 150 419 / 370, 4096 x 20480 at 230 164.8 / 145.4; two rounds where there were three or four: 8192 x 45056 at 120
// and 180 431 / 398, 503 / 480.
inline int big_wide_splits(int m_count, int d_ff, int splits) {
    const int max_tiles = big_wide_tiles(big_token_tiles(m_count)), groups = d_ff / 8;
    if (!max_tiles || splits <= 256) return splits;
    const int rounds = ((groups + max_tiles - 1) / max_tiles + 255) / 256, n = 256 * rounds;
    return n < splits && (groups + n - 1) / n > kBigMaxRowTiles ? n : splits;
}
// The gate/up launch of a configuration with `splits` slices.
inline BigLaunch big_gateup_launch(int m_count, int d_ff, int splits) {
    const int groups = splits <= 256 ? big_gateup_groups(m_count, d_ff) : 1;
    const int n = groups > 1 ? std::min(splits, 128) : big_wide_splits(m_count, d_ff, splits);
    return big_divide(m_count, groups, n, n);
}

// The down kernels', where the partial blocks are summed by a launch: up to 2048 wide there are few column blocks, and groups make
// workgroups of them without more partial sums; two as well up to 4096 wide with a d_ff of at most 4096, beyond 128 tokens or with W_down as
// [d_model, d_ff].  Whole call, us, one group / two / four, at 70, 114 and 230 tokens: 512 x 1536 14.1 / 13.5, 15.2 / 14.5, 20.9 / 19.1 / 18.5;
// 1024 x 3840 21.6 / 21.0, 23.9 / 23.1, 33.9 / 31.9 / 30.8; 1280 x 7168 31.5 / 29.8, 35.3 / 33.6, 45.9 / 41.8 / 44.2; 2048 x 5504 33.2 /
// 31.9, 38.4 / 35.8, 49.4 / 46.0 / 47.8; 4096 x 4096 47.0 / 47.1, 49.0 / 48.5, 55.5 / 51.2; W_down as [d_model, d_ff]: 512 x 1536 13.9 / 13.4,
// 15.1 / 14.0, 20.4 / 17.7 / 16.5; 1024 x 3840 21.5 / 20.7, 24.0 / 22.6, 32.6 / 29.7 / 27.3; 4096 x 4096 41.2 / 39.9, 44.4 / 44.0, 53.6 / 50.2.
// On the other side, at 80, 128 and 256: 2304 x 9216 44.0 / 48.1, 47.6 / 51.8, 64.6 / 66.1; 2560 x 5120 37.9 / 38.3, 42.2 / 41.5, 56.4 /
// 55.7; 4096 x 14336 82.0 / 88.1, 89.8 / 93.7, 115.0 / 116.2; W_down as [d_model, d_ff], 2304 x 8192 at 70 and 230 39.3 / 42.8, 56.5 / 56.5.
// The groups' workgroups read the same weights, on one XCD (big_down_launch): up to 32 MB of W_down, all that the XCDs' L2s hold; beyond 192
// tokens, where A_2 is the larger part, up to 64 MB; four groups up to 20 MB.  At 128 tokens: 768 x 18432 (27 MB) 39.2 / 39.2, 1152 x 14336
// (32 MB) 42.3 / 42.2, 2048 x 11264 (44 MB) 49.4 / 48.9, 1536 x 18432 (54 MB) 54.2 / 56.6, 2048 x 20480 (80 MB) 65.2 / 68.7; at 160: 1024 x
// 20480 (40 MB) 50.7 / 50.4 / 51.6, 2048 x 28672 (112 MB) 91.6 / 95.5, 512 x 20480 (20 MB) 40.4 / 38.8 / 37.4, 896 x 12288 (21 MB) 39.8 / 39.1 /
// 41.1; at 256: 1536 x 18432 72.0 / 70.1, 2048 x 16384 (64 MB) 76.3 / 72.1, 2048 x 20480 83.6 / 84.5, 1536 x 24576 (72 MB) 92.2 / 95.3, 512 x
// 28672 (28 MB) 58.6 / 55.4 / 56.9.
inline int big_down_groups(int m_count, int d_ff, int k2_col_blocks, bool wdt) {
    if (m_count <= 64 || k2_col_blocks > 32) return 1;
    if (k2_col_blocks > 16) return d_ff <= 4096 && (wdt || m_count > 128) ? 2 : 1;
    const long long bytes = (long long)k2_col_blocks * 256 * d_ff;                      // of W_down
    if (bytes > (m_count > 192 ? 64ll << 20 : 32ll << 20)) return 1;
    return m_count > 128 && k2_col_blocks <= 8 && bytes <= 20ll << 20 ? 4 : 2;
}
// The down launch of a configuration with `splits` splits.  `summed`: the partial blocks are added by a launch (else: atomics, and one counter
// per column block).  With groups a row of the grid has a multiple of 8 workgroups, the last ones without work, so that the same
// workgroup of every group is on the same XCD and finds the weights in its L2; and no XCD gets more of them than its 32 CUs, so fewer splits
// where those were many.  Then, if splits of whole 64-row steps are near, those (the transposed layout deals out whole steps in any case).
// Whole call, us, at 128, 160 and 256 tokens, row as long as it is and cut to 256 workgroups in all / so: 896 x 12288 38.5 / 35.7, 45.6 /
// 39.1, 52.1 / 43.6; 1152 x 5504 at 128 and 250 31.7 / 30.2, 37.2 / 35.7; 1664 x 9216 at 100 and 250 42.1 / 39.3, 53.8 / 51.2.
inline BigLaunch big_down_launch(int m_count, int d_ff, int splits, int k2_col_blocks, bool wdt, bool summed) {
    const int groups = summed ? big_down_groups(m_count, d_ff, k2_col_blocks, wdt) : 1;
    BigLaunch l = big_divide(m_count, groups, splits, splits * k2_col_blocks);
    if (l.groups == 1) return l;
    const int most = std::max(1, 32 / l.groups * 8 / k2_col_blocks);
    if (l.splits > most) {
        l.splits = most;
        for (int s = most; !wdt && 8 * s >= 5 * most; --s)
            if (d_ff % (64 * s) == 0) { l.splits = s; break; }
    }
    l.row = (l.splits * k2_col_blocks + 7) / 8 * 8;
    return l;
}

}  // namespace dfk
