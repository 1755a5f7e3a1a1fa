"""dfk_mlp_block without a configuration, on both sides of the rule that says when the pair runs as one launch of both kernels' workgroups (bytes of
weights), and both forms by name: one to four token tiles, out of place and in place, the same bits."""
import pytest

torch = pytest.importorskip("torch")

import dfk_inputs as di
import paper_2602_11808_amd as dfk
from oracle import oracle
from tests.helpers import assert_parity, rel_err

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


# the form the untuned block takes: one launch, the pair, or the pair because it is all there is
@pytest.mark.parametrize("shape,dtype,single", [((1, 1536, 5632), "bf16", True), ((16, 1536, 5632), "fp16", True), ((16, 1536, 5120), "bf16", False),
                                                ((17, 1024, 1536), "bf16", False), ((33, 1152, 2048), "fp16", False), ((64, 1024, 2816), "bf16", False),
                                                ((40, 1536, 5632), "bf16", True), ((20, 896, 1024), "bf16", None)],
                         ids=lambda s: "M%d_d%d_ff%d" % s if isinstance(s, tuple) else str(s))
def test_untuned_block(shape, dtype, single):
    M, d, ff = shape
    dt = dfk.DFK_BF16 if dtype == "bf16" else dfk.DFK_FP16
    pick, _ = dfk.dfk_get_choice_block(M, d, ff, dt)
    assert (pick.variant == dfk.DFK_VARIANT_FUSED) == bool(single), pick
    pair = dfk.dfk_config_t(**dict(pick.as_dict(), variant=dfk.DFK_VARIANT_TWO_KERNEL, kmajor=1))
    one = dfk.dfk_config_t(**dict(pick.as_dict(), variant=dfk.DFK_VARIANT_FUSED, kmajor=4, depth=4))
    cfgs = [None, pair] + ([one] if single is not None else [])
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
        dfk.dfk_mlp_block(src, g["w"], eps, g["Wg"], g["Wu"], g["Wd"], out, cfgs[rep // 2 % len(cfgs)], ws)
        torch.cuda.synchronize()
        if first is None:
            first = out.clone()
            got = di.as_f64(di.to_numpy(out))
            assert_parity(got, ref, dtype, shape)
            # the block's own share: the stated bars of the types
            assert rel_err(got - H64, ref - H64) <= {"bf16": 2e-2, "fp16": 2e-3}[dtype], shape
        assert torch.equal(first.view(torch.int16), out.view(torch.int16)), (shape, rep)
        assert int(torch.count_nonzero(ws[:4096 + 64 * 32768 * 4]).item()) == 0, shape
