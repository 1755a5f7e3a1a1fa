"""W_down as [d_model, d_ff] with the down projection split over d_ff (kmajor = 5 with column blocks): token groups of one to four tiles
and the counts beside their edges, both gate/up kernels in front, splits of one step and of unequal numbers of steps."""
import copy

import pytest

torch = pytest.importorskip("torch")

import dfk_inputs as di
import paper_2602_11808_amd as dfk
from oracle import oracle
from tests.helpers import assert_parity

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("dtype", ["bf16", "fp16"])
@pytest.mark.parametrize("shape", [(65, 256, 128), (128, 384, 640), (129, 640, 1152), (192, 512, 4224), (193, 1024, 2816), (256, 768, 8320),
                                   (17, 512, 1024), (33, 640, 1152), (64, 1024, 4096)], ids=lambda s: "M%d_d%d_ff%d" % s)
def test_split_down_projection_of_the_transposed_layout(shape, dtype):
    M, d, ff = shape
    t = di.mlp_inputs(M, d, ff, seed=79, dtype=dtype)
    w = di.tensor(1079, (d,), 1.0, dtype)
    ref = oracle.swiglu_mlp(t["X"], t["Wg"], t["Wu"], t["Wd"])
    ref_block = oracle.mlp_block(t["X"], w, 1e-5, t["Wg"], t["Wu"], t["Wd"])
    g = {k: di.to_torch(v, DEV) for k, v in t.items()}
    wn = di.to_torch(w, DEV)
    Wd_t = torch.empty((d, ff), dtype=g["Wd"].dtype, device=DEV)
    dfk.dfk_transpose_w_down(g["Wd"], Wd_t)
    ws = dfk.new_workspace(M, d, ff, DEV)
    dt = dfk.DFK_BF16 if dtype == "bf16" else dfk.DFK_FP16
    cfgs = [c for c in (dfk.dfk_get_candidate_wdt(M, d, ff, dt, i) for i in range(dfk.dfk_num_candidates_wdt(M, d, ff, dt)))
            if c.path == dfk.DFK_PATH_MFMA and c.k2_col_blocks > 1]
    assert cfgs and all(c.kmajor == 5 and c.k2_col_blocks == d // 128 for c in cfgs)
    for splits in (1, 2, ff // 64):                # the whole of d_ff, halves, single steps
        c = copy.copy(cfgs[0])
        c.k2_splits = splits
        cfgs.append(c)
    for cfg in cfgs:
        assert dfk.dfk_config_valid(cfg, M, d, ff, dt)
        print("case", shape, dtype, cfg, flush=True)
        first = None
        for _ in range(2):
            Y = torch.full_like(g["X"], float("nan"))
            dfk.dfk_swiglu_mlp_wdt(g["X"], g["Wg"], g["Wu"], Wd_t, Y, cfg, ws)
            torch.cuda.synchronize()
            assert_parity(di.as_f64(di.to_numpy(Y)), ref, dtype, cfg)
            first = Y.clone() if first is None else first
            assert torch.equal(first.view(torch.int16), Y.view(torch.int16)), cfg
        h = g["X"].clone()
        dfk.dfk_mlp_block_wdt(h, wn, 1e-5, g["Wg"], g["Wu"], Wd_t, h, cfg, ws)      # in place
        torch.cuda.synchronize()
        assert_parity(di.as_f64(di.to_numpy(h)), ref_block, dtype, cfg)
        assert int(torch.count_nonzero(ws[:4096 + 64 * 32768 * 4]).item()) == 0, cfg
    bad = copy.copy(cfgs[0])
    for field, value in (("k2_splits", ff // 64 + 1), ("k2_splits", 0), ("k2_col_blocks", d // 128 + 1), ("reduce", dfk.DFK_REDUCE_ATOMIC)):
        c = copy.copy(bad)
        setattr(c, field, value)
        assert not dfk.dfk_config_valid(c, M, d, ff, dt), (field, value)
