"""The single launch with A_2 in LDS, atomic reduction: both forms of taking Y out of the accumulator, on either side of the line
between them (two exchanges of two floats per thread cover tokens x d_model)."""
import pytest

torch = pytest.importorskip("torch")

import dfk_inputs as di
import paper_2602_11808_amd as dfk
from oracle import oracle
from tests.helpers import assert_parity

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("dtype", ["bf16", "fp16"])
@pytest.mark.parametrize("M,d", [(1, 1024), (1, 1152), (1, 2048), (1, 2176), (2, 1024), (3, 1024), (16, 1024), (17, 1152)])
def test_both_forms_of_the_drain(M, d, dtype):
    ff = 520
    t = di.mlp_inputs(M, d, ff, seed=101, dtype=dtype)
    ref = oracle.swiglu_mlp(t["X"], t["Wg"], t["Wu"], t["Wd"])
    g = {k: di.to_torch(v, DEV) for k, v in t.items()}
    ws = dfk.new_workspace(M, d, ff, DEV)
    dt = dfk.DFK_BF16 if dtype == "bf16" else dfk.DFK_FP16
    cfgs = [c for c in (dfk.dfk_get_candidate(M, d, ff, dt, i) for i in range(dfk.dfk_num_candidates(M, d, ff, dt)))
            if c.variant == dfk.DFK_VARIANT_FUSED and c.kmajor == 1 and c.reduce == dfk.DFK_REDUCE_ATOMIC]
    assert {c.waves for c in cfgs} == {4, 8}       # the line lies at 1024 and at 2048 columns times tokens
    for cfg in cfgs:
        print("case", M, d, dtype, cfg, flush=True)
        buf = torch.full((M + 1, d), 7.0, dtype=g["X"].dtype, device=DEV)
        for _ in range(2):
            dfk.dfk_swiglu_mlp_ex(g["X"], g["Wg"], g["Wu"], g["Wd"], buf[:M], cfg, ws)
            torch.cuda.synchronize()
            assert_parity(di.as_f64(di.to_numpy(buf[:M])), ref, dtype, cfg)
        assert bool((buf[M] == 7.0).all())
        assert int(torch.count_nonzero(ws[:4096 + 64 * 32768 * 4]).item()) == 0, cfg
