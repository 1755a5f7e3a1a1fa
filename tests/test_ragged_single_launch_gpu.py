"""Widths that are no multiple of 128 in bf16, without a configuration: the pair's untuned choice as one launch of both kernels'
workgroups, on both sides of the rule (tokens, bytes of weights), one to four token tiles, against the oracle and bit for bit over calls."""
import pytest

torch = pytest.importorskip("torch")

import dfk_inputs as di
import paper_2602_11808_amd as dfk
from oracle import oracle
from tests.helpers import assert_parity

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("shape", [(1, 2008, 4008), (16, 2040, 4096), (16, 2008, 3960), (17, 1000, 1000), (33, 1032, 2056), (64, 1416, 1808), (40, 616, 1048),
                                   (70, 1000, 1000)], ids=lambda s: "M%d_d%d_ff%d" % s)
def test_untuned_call_off_128(shape):
    M, d, ff = shape
    t = di.mlp_inputs(M, d, ff, seed=89)
    ref = oracle.swiglu_mlp(t["X"], t["Wg"], t["Wu"], t["Wd"])
    g = {k: di.to_torch(v, DEV) for k, v in t.items()}
    ws = dfk.new_workspace(M, d, ff, DEV)
    pick, _ = dfk.dfk_get_choice(M, d, ff, dfk.DFK_BF16)
    first = None
    for rep in range(20):
        Y = torch.full_like(g["X"], float("nan"))
        dfk.dfk_swiglu_mlp_ex(g["X"], g["Wg"], g["Wu"], g["Wd"], Y, pick if rep == 19 else None, ws)    # (the pair itself last)
        torch.cuda.synchronize()
        if first is None:
            first = Y.clone()
            assert_parity(di.as_f64(di.to_numpy(Y)), ref, "bf16", shape)
        assert torch.equal(first.view(torch.int16), Y.view(torch.int16)), (shape, rep)
        assert int(torch.count_nonzero(ws[:4096 + 64 * 32768 * 4]).item()) == 0, shape
