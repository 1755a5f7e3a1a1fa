"""The 256-token pair at the edges of its forms: token groups of 1..4 tiles, the row-tile counts a slice can have, steps fewer
than buffers."""
import pytest

torch = pytest.importorskip("torch")

import dfk_inputs as di
import paper_2602_11808_amd as dfk
from oracle import oracle
from tests.helpers import assert_parity

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


# d_ff of 8-row groups just below 4, 6, 7 and 8 per slice at 256 slices: slices with one row tile less than the kernel's constant among them
@pytest.mark.parametrize("dtype", ["bf16", "fp16"])
@pytest.mark.parametrize("shape", [(65, 640, 8184), (128, 128, 12280), (129, 384, 14328), (150, 256, 16376), (192, 640, 8184), (193, 128, 16376),
                                   (5, 128, 1000)], ids=lambda s: "M%d_d%d_ff%d" % s)
def test_every_form_of_the_256_token_pair(shape, dtype):
    M, d, ff = shape
    t = di.mlp_inputs(M, d, ff, seed=67, dtype=dtype)
    ref = oracle.swiglu_mlp(t["X"], t["Wg"], t["Wu"], t["Wd"])
    g = {k: di.to_torch(v, DEV) for k, v in t.items()}
    ws = dfk.new_workspace(M, d, ff, DEV)
    dt = dfk.DFK_BF16 if dtype == "bf16" else dfk.DFK_FP16
    cfgs = [c for c in (dfk.dfk_get_candidate(M, d, ff, dt, i) for i in range(dfk.dfk_num_candidates(M, d, ff, dt))) if c.kmajor == 2]
    assert any(c.splits == min(256, ff // 8) for c in cfgs)
    for cfg in cfgs:
        for waves, depth in ((8, 3), (4, 4)):      # accepted, and the same kernels
            cfg.waves, cfg.depth = waves, depth
            print("case", shape, dtype, cfg, flush=True)
            Y = torch.full_like(g["X"], float("nan"))
            dfk.dfk_swiglu_mlp_ex(g["X"], g["Wg"], g["Wu"], g["Wd"], Y, cfg, ws)
            torch.cuda.synchronize()
            assert_parity(di.as_f64(di.to_numpy(Y)), ref, dtype, (shape, cfg))
            assert int(torch.count_nonzero(ws[:4096 + 64 * 32768 * 4]).item()) == 0, (shape, cfg)
