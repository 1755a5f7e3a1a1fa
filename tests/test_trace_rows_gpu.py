"""Time stamps: a row per workgroup also where token groups make the grid two-dimensional, none from a buffer that is too small for that, and the
end of the down kernel stamped where a launch adds the splits' blocks up."""
import pytest

torch = pytest.importorskip("torch")

import dfk_inputs as di
import paper_2602_11808_amd as dfk

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
TWO = dfk.DFK_VARIANT_TWO_KERNEL


def _stamps(M, d, ff, cfg, rows, wdt=False):
    t = di.mlp_inputs(M, d, ff, seed=111)
    g = {k: di.to_torch(v, DEV) for k, v in t.items()}
    ws = dfk.new_workspace(M, d, ff, DEV)
    tr = torch.zeros(rows * 8 + 8, dtype=torch.int64, device=DEV)      # a guard row behind the buffer
    Y = torch.empty_like(g["X"])
    if wdt:
        wt = torch.empty((d, ff), dtype=g["Wd"].dtype, device=DEV)
        dfk.dfk_transpose_w_down(g["Wd"], wt)
    dfk.dfk_set_trace_buffer(tr[:rows * 8])
    try:
        if wdt:
            dfk.dfk_swiglu_mlp_wdt(g["X"], g["Wg"], g["Wu"], wt, Y, cfg, ws)
        else:
            dfk.dfk_swiglu_mlp_ex(g["X"], g["Wg"], g["Wu"], g["Wd"], Y, cfg, ws)
    finally:
        dfk.dfk_set_trace_buffer(None)
    torch.cuda.synchronize()
    s = tr.cpu().view(-1, 8)
    assert not bool(s[rows].any())
    return s[:rows]


# 128 slices x 2 groups; 5 splits x 4 column blocks x 4 or 2 groups
@pytest.mark.parametrize("wdt", [False, True])
@pytest.mark.parametrize("M,down", [(256, 80), (100, 40)])
def test_a_row_for_every_workgroup_of_a_token_group(M, down, wdt):
    d, ff = 512, 1536
    pick = dfk.dfk_get_choice_wdt(M, d, ff)[0] if wdt else dfk.dfk_get_choice(M, d, ff)[0]
    cfg = dfk.dfk_config_t(**dict(pick.as_dict(), splits=128, k2_splits=5, k2_col_blocks=4, kmajor=5 if wdt else 2))
    s = _stamps(M, d, ff, cfg, 256, wdt)
    assert bool((s[:, 0] > 0).all()) and bool((s[:, 2] >= s[:, 0]).all()) and bool((s[:, 1] >= s[:, 2]).all())
    assert int((s[:, 3] > 0).sum()) == down == int((s[:, 4] > 0).sum()) and bool((s[:down, 3] > 0).all())
    assert not bool(_stamps(M, d, ff, cfg, 255, wdt).any())            # one row short: untouched


def test_a_down_kernel_whose_blocks_a_launch_adds_up():
    M, d, ff = 40, 1024, 1536
    n = dfk.dfk_num_candidates(M, d, ff, dfk.DFK_BF16)
    pair = next(c for c in (dfk.dfk_get_candidate(M, d, ff, dfk.DFK_BF16, i) for i in range(n))
                if c.variant == TWO and c.kmajor == 1 and c.reduce == dfk.DFK_REDUCE_TICKET and c.waves == 8)
    one = dfk.dfk_config_t(**dict(pair.as_dict(), variant=dfk.DFK_VARIANT_FUSED, kmajor=4, depth=4))
    for cfg in (pair, one):
        s = _stamps(M, d, ff, cfg, cfg.splits + cfg.k2_splits * cfg.k2_col_blocks)
        s = s[s[:, 4] > 0]
        assert len(s) == cfg.k2_splits * cfg.k2_col_blocks
        assert bool((s[:, 5] >= s[:, 4]).all()) and bool((s[:, 6] >= s[:, 5]).all())
