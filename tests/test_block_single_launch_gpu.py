"""dfk_mlp_block without a configuration: the pair's untuned choice as one launch of both kernels' workgroups, on both sides of the
rule (tokens, bytes of weights), one to four token tiles, out of place and in place."""
import pytest

torch = pytest.importorskip("torch")

import dfk_inputs as di
import paper_2602_11808_amd as dfk
from oracle import oracle
from tests.helpers import assert_parity, rel_err

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("shape,dtype", [((1, 1536, 5632), "bf16"), ((16, 1536, 5632), "fp16"), ((16, 1536, 5120), "bf16"), ((17, 1024, 1536), "bf16"),
                                         ((33, 1152, 2048), "fp16"), ((64, 1024, 2816), "bf16"), ((20, 896, 1024), "bf16")],
                         ids=lambda s: "M%d_d%d_ff%d" % s if isinstance(s, tuple) else s)
def test_untuned_block(shape, dtype):
    M, d, ff = shape
    eps = 1e-5
    t = di.mlp_inputs(M, d, ff, seed=83, dtype=dtype)
    t["w"] = di.tensor(1083, (d,), 1.0, dtype)
    ref = oracle.mlp_block(t["X"], t["w"], eps, t["Wg"], t["Wu"], t["Wd"])
    H64 = di.as_f64(t["X"])
    g = {k: di.to_torch(v, DEV) for k, v in t.items()}
    ws = dfk.new_workspace(M, d, ff, DEV)
    first = None
    for rep in range(20):
        out = g["X"].clone() if rep % 2 else torch.full_like(g["X"], float("nan"))
        src = out if rep % 2 else g["X"]
        dfk.dfk_mlp_block(src, g["w"], eps, g["Wg"], g["Wu"], g["Wd"], out, None, ws)
        torch.cuda.synchronize()
        if first is None:
            first = out.clone()
            got = di.as_f64(di.to_numpy(out))
            assert_parity(got, ref, dtype, shape)
            # the block's own share: the stated bars of the types
            assert rel_err(got - H64, ref - H64) <= {"bf16": 2e-2, "fp16": 2e-3}[dtype], shape
        assert torch.equal(first.view(torch.int16), out.view(torch.int16)), (shape, rep)
        assert int(torch.count_nonzero(ws[:4096 + 64 * 32768 * 4]).item()) == 0, shape
