"""Gate/up kernel of the 256-token pair: where a workgroup's walk through the k range starts, on both sides of the rule's lines.  A window where
there are more than 64 steps and either more than 3 MB of X (256 x 6272) or rows a multiple of 16 KB apart (129 x 8192: 2.1 MB, one
64-k piece a step, 128 steps); else the whole range: rows 16 KB apart but 64 steps (65 x 8192: two pieces a step with one row tile per
slice), just short of 3 MB (255 x 6144), few steps."""
import pytest

torch = pytest.importorskip("torch")

import dfk_inputs as di
import paper_2602_11808_amd as dfk
from oracle import oracle
from tests.helpers import assert_parity

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("shape", [(65, 8192, 1024), (129, 8192, 1024), (256, 6272, 1024), (255, 6144, 1024), (200, 4096, 640)], ids=lambda s: "M%d_d%d_ff%d" % s)
def test_every_start_of_the_k_walk(shape):
    M, d, ff = shape
    t = di.mlp_inputs(M, d, ff, seed=73)
    ref = oracle.swiglu_mlp(t["X"], t["Wg"], t["Wu"], t["Wd"])
    g = {k: di.to_torch(v, DEV) for k, v in t.items()}
    ws = dfk.new_workspace(M, d, ff, DEV)
    cfg = next(c for c in (dfk.dfk_get_candidate(M, d, ff, dfk.DFK_BF16, i) for i in range(dfk.dfk_num_candidates(M, d, ff, dfk.DFK_BF16)))
               if c.kmajor == 2 and c.reduce == dfk.DFK_REDUCE_TICKET)
    first = None
    for _ in range(2):
        Y = torch.full_like(g["X"], float("nan"))
        dfk.dfk_swiglu_mlp_ex(g["X"], g["Wg"], g["Wu"], g["Wd"], Y, cfg, ws)
        torch.cuda.synchronize()
        assert_parity(di.as_f64(di.to_numpy(Y)), ref, "bf16", cfg)
        first = Y.clone() if first is None else first
        assert torch.equal(first.view(torch.uint8), Y.view(torch.uint8)), cfg
