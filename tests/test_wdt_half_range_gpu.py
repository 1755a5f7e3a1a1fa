"""Half inputs, W_down as [d_model, d_ff], layers too small for the whole-rows kernels: values of A_2 beyond the range of half, which the plain-FMA
pair holds in fp32, come through whole, also after tuning."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import dfk_inputs as di
import paper_2602_11808_amd as dfk
from oracle import oracle
from tests.helpers import assert_parity

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("tune", [False, True])
@pytest.mark.parametrize("shape", [(65, 256, 128), (130, 384, 640), (17, 512, 256), (64, 1024, 384)], ids=lambda s: "M%d_d%d_ff%d" % s)
def test_a2_beyond_the_range_of_half(shape, tune):
    M, d, ff = shape
    t = di.mlp_inputs(M, d, ff, seed=101, dtype="fp16")
    for k, f in (("Wg", 128.0), ("Wu", 128.0), ("Wd", 2.0 ** -6)):
        t[k] = (t[k].astype("float32") * f).astype(t[k].dtype)
    H = di.as_f64(t["X"])
    gate, up = H @ di.as_f64(t["Wg"]).T, H @ di.as_f64(t["Wu"]).T
    assert abs(gate / (1.0 + np.exp(-gate)) * up).max() > 65504.0
    ref = oracle.swiglu_mlp(t["X"], t["Wg"], t["Wu"], t["Wd"])
    assert abs(ref).max() < 6e4
    g = {k: di.to_torch(v, DEV) for k, v in t.items()}
    Wd_t = g["Wd"].t().contiguous()
    ws = dfk.new_workspace(M, d, ff, DEV)
    try:
        if tune:
            sets = 2
            scratch = torch.empty(dfk.dfk_tune_scratch_bytes(M, d, ff, dfk.DFK_FP16, sets), dtype=torch.uint8, device=DEV)
            dfk.dfk_tune([M], d, ff, dfk.DFK_FP16, scratch, sets=sets, iters=3)
            pick, tuned = dfk.dfk_get_choice_wdt(M, d, ff, dfk.DFK_FP16)
            assert tuned and pick.a2_dtype == dfk.DFK_FP32, pick
        Y = torch.full_like(g["X"], float("nan"))
        dfk.dfk_swiglu_mlp_wdt(g["X"], g["Wg"], g["Wu"], Wd_t, Y, None, ws)
        torch.cuda.synchronize()
    finally:
        dfk.dfk_clear_tuning()
    assert_parity(di.as_f64(di.to_numpy(Y)), ref, "fp16", shape)
