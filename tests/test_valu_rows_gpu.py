"""The plain-FMA down kernel with a split's rows divided among the threads of a column chunk: both sides of the row limit, one and
several column blocks, partial ones, every token-tile width."""
import copy

import pytest

torch = pytest.importorskip("torch")

import dfk_inputs as di
import paper_2602_11808_amd as dfk
from oracle import oracle
from tests.helpers import assert_parity

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
DT = {"bf16": dfk.DFK_BF16, "fp16": dfk.DFK_FP16, "fp32": dfk.DFK_FP32}


@pytest.mark.parametrize("dtype", ["bf16", "fp16", "fp32"])
@pytest.mark.parametrize("M", [1, 2, 3, 8, 11])
def test_rows_divided_among_threads(M, dtype):
    d, ff = 1352, 1000
    t = di.mlp_inputs(M, d, ff, seed=73, dtype=dtype)
    ref = oracle.swiglu_mlp(t["X"], t["Wg"], t["Wu"], t["Wd"])
    g = {k: di.to_torch(v, DEV) for k, v in t.items()}
    ws = dfk.new_workspace(M, d, ff, DEV)
    n = dfk.dfk_num_candidates(M, d, ff, DT[dtype])
    base = next(c for c in (dfk.dfk_get_candidate(M, d, ff, DT[dtype], i) for i in range(n))
                if c.path == dfk.DFK_PATH_VALU and c.variant == dfk.DFK_VARIANT_TWO_KERNEL)
    ran = 0
    for splits, blocks, waves in ((1, 2, 8), (5, 3, 8), (10, 2, 8), (10, 5, 4), (11, 5, 8), (4, 100, 8), (3, 1, 8), (7, 3, 3)):
        cfg = copy.copy(base)
        cfg.k2_splits, cfg.k2_col_blocks, cfg.waves = splits, blocks, waves
        if not dfk.dfk_config_valid(cfg, M, d, ff, DT[dtype]):
            continue
        print("case", M, dtype, cfg, flush=True)
        first = None
        for _ in range(2):
            Y = torch.full_like(g["X"], float("nan"))
            dfk.dfk_swiglu_mlp_ex(g["X"], g["Wg"], g["Wu"], g["Wd"], Y, cfg, ws)
            torch.cuda.synchronize()
            assert_parity(di.as_f64(di.to_numpy(Y)), ref, dtype, cfg)
            first = Y.clone() if first is None else first
            assert torch.equal(first.view(torch.uint8), Y.view(torch.uint8)), cfg
        ran += 1
    assert ran >= 6
