"""The single launch of both kernels' workgroups with the down workgroups at the head of the grid, as if other launches held the CUs its gate/up
workgroups need: down workgroups park, the last one does their work, and the result is what it always is."""
import os

import pytest

torch = pytest.importorskip("torch")

import dfk_inputs as di
import paper_2602_11808_amd as dfk
from oracle import oracle
from tests.helpers import assert_parity

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


# 256 down workgroups, as many as CUs; fewer, so that only some of them wait; more; two column blocks each; one to four token tiles
@pytest.mark.parametrize("shape,dtype", [((2, 4096, 8192), "bf16"), ((17, 1024, 2816), "fp16"), ((33, 8192, 1024), "bf16"), ((64, 2304, 4096), "bf16"),
                                         ((16, 5120, 11264), "bf16")], ids=lambda s: "M%d_d%d_ff%d" % s if isinstance(s, tuple) else s)
def test_down_workgroups_that_come_first(shape, dtype, monkeypatch):
    M, d, ff = shape
    dt = dfk.DFK_BF16 if dtype == "bf16" else dfk.DFK_FP16
    t = di.mlp_inputs(M, d, ff, seed=103, dtype=dtype)
    t["w"] = di.tensor(1103, (d,), 1.0, dtype)
    ref = oracle.swiglu_mlp(t["X"], t["Wg"], t["Wu"], t["Wd"])
    ref_block = oracle.mlp_block(t["X"], t["w"], 1e-5, t["Wg"], t["Wu"], t["Wd"])
    g = {k: di.to_torch(v, DEV) for k, v in t.items()}
    ws = dfk.new_workspace(M, d, ff, DEV)
    cands = [dfk.dfk_get_candidate(M, d, ff, dt, i) for i in range(dfk.dfk_num_candidates(M, d, ff, dt))]
    for reduce in (dfk.DFK_REDUCE_TICKET, dfk.DFK_REDUCE_ATOMIC):
        cfg = next(c for c in cands if c.kmajor == 4 and c.reduce == reduce)
        wanted = None
        for first in (False, True, False, True):
            if first:
                monkeypatch.setenv("DFK_DEBUG_DOWN_FIRST", "1")
            else:
                monkeypatch.delenv("DFK_DEBUG_DOWN_FIRST", raising=False)
            print("case", shape, cfg, "down first" if first else "", flush=True)
            Y = torch.full_like(g["X"], float("nan"))
            dfk.dfk_swiglu_mlp_ex(g["X"], g["Wg"], g["Wu"], g["Wd"], Y, cfg, ws)
            torch.cuda.synchronize()
            assert_parity(di.as_f64(di.to_numpy(Y)), ref, dtype, (cfg, first))
            assert int(torch.count_nonzero(ws[:4096 + 64 * 32768 * 4]).item()) == 0, (cfg, first)
            if reduce == dfk.DFK_REDUCE_TICKET:
                wanted = Y.clone() if wanted is None else wanted
                assert torch.equal(wanted.view(torch.int16), Y.view(torch.int16)), (cfg, first)
    # the block in place: nothing is stored before every gate/up workgroup has read its input
    wanted = None
    for first in (False, True):
        if first:
            monkeypatch.setenv("DFK_DEBUG_DOWN_FIRST", "1")
        else:
            monkeypatch.delenv("DFK_DEBUG_DOWN_FIRST", raising=False)
        print("case block", shape, "down first" if first else "", flush=True)
        h = g["X"].clone()
        dfk.dfk_mlp_block(h, g["w"], 1e-5, g["Wg"], g["Wu"], g["Wd"], h, None, ws)
        torch.cuda.synchronize()
        assert_parity(di.as_f64(di.to_numpy(h)), ref_block, dtype, first)
        wanted = h.clone() if wanted is None else wanted
        assert torch.equal(wanted.view(torch.int16), h.view(torch.int16)), first
        assert int(torch.count_nonzero(ws[:4096 + 64 * 32768 * 4]).item()) == 0, first
