"""Widths that are no multiple of 128 in bf16, without a configuration, on both sides of the rule that says when the pair runs as one launch of both
kernels' workgroups (tokens, bytes of weights, d_ff against d_model), and both forms by name: one to four token tiles, against the oracle and
bit for bit, and both through dfk_swiglu_mlp_static and after tuning."""
import pytest

torch = pytest.importorskip("torch")

import dfk_inputs as di
import paper_2602_11808_amd as dfk
from oracle import oracle
from tests.helpers import assert_parity

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("shape,single", [((1, 2008, 4008), True), ((16, 2040, 4096), True), ((16, 2008, 3960), False), ((17, 1000, 1000), False),
                                          ((33, 1032, 2056), True), ((64, 1416, 1808), True), ((40, 616, 1048), None), ((70, 1000, 1000), None)],
                         ids=lambda s: "M%d_d%d_ff%d" % s if isinstance(s, tuple) else str(s))
def test_untuned_call_off_128(shape, single):
    M, d, ff = shape
    t = di.mlp_inputs(M, d, ff, seed=89)
    ref = oracle.swiglu_mlp(t["X"], t["Wg"], t["Wu"], t["Wd"])
    g = {k: di.to_torch(v, DEV) for k, v in t.items()}
    ws = dfk.new_workspace(M, d, ff, DEV)
    pick, _ = dfk.dfk_get_choice(M, d, ff, dfk.DFK_BF16)
    assert (pick.variant == dfk.DFK_VARIANT_FUSED) == bool(single), pick
    pair = dfk.dfk_config_t(**dict(pick.as_dict(), variant=dfk.DFK_VARIANT_TWO_KERNEL, kmajor=1))
    one = dfk.dfk_config_t(**dict(pick.as_dict(), variant=dfk.DFK_VARIANT_FUSED, kmajor=4, depth=4))
    cfgs = [None, pair, "static"] + ([one] if single is not None else [])
    first = None
    for rep in range(20):
        cfg = cfgs[rep % len(cfgs)]
        Y = torch.full_like(g["X"], float("nan"))
        if cfg == "static":
            dfk.dfk_swiglu_mlp_static(g["X"], g["Wg"], g["Wu"], g["Wd"], Y)
        else:
            dfk.dfk_swiglu_mlp_ex(g["X"], g["Wg"], g["Wu"], g["Wd"], Y, cfg, ws)
        torch.cuda.synchronize()
        if first is None:
            first = Y.clone()
            assert_parity(di.as_f64(di.to_numpy(Y)), ref, "bf16", shape)
        assert torch.equal(first.view(torch.int16), Y.view(torch.int16)), (shape, rep)
        assert int(torch.count_nonzero(ws[:4096 + 64 * 32768 * 4]).item()) == 0, shape
    if single is not None:                        # the atomic reduction of that form
        one.reduce = dfk.DFK_REDUCE_ATOMIC
        Y = torch.full_like(g["X"], float("nan"))
        dfk.dfk_swiglu_mlp_ex(g["X"], g["Wg"], g["Wu"], g["Wd"], Y, one, ws)
        torch.cuda.synchronize()
        assert_parity(di.as_f64(di.to_numpy(Y)), ref, "bf16", one)
        assert int(torch.count_nonzero(ws[:4096 + 64 * 32768 * 4]).item()) == 0, shape


def test_tuning_times_the_single_launch_off_128():
    """After tuning a layer whose untuned choice is that form, the choice is no slower than it, and the fused variant's entry is another."""
    M, d, ff = 4, 2888, 7688
    untuned, _ = dfk.dfk_get_choice(M, d, ff, dfk.DFK_BF16)
    assert (untuned.variant, untuned.kmajor) == (dfk.DFK_VARIANT_FUSED, 4)
    try:
        scratch = torch.empty(dfk.dfk_tune_scratch_bytes(M, d, ff, dfk.DFK_BF16, 4), dtype=torch.uint8, device=DEV)
        dfk.dfk_tune([M], d, ff, dfk.DFK_BF16, scratch, sets=4, iters=20)
        assert dfk.dfk_tune_skipped()[0] == 0
        pick, tuned = dfk.dfk_get_choice(M, d, ff, dfk.DFK_BF16)
        us = [min(dfk.dfk_time_config(c, M, d, ff, dfk.DFK_BF16, scratch, 4, 40) for _ in range(5)) for c in (untuned, pick)]
        print("untuned", untuned, "tuned", pick, us, flush=True)
        assert tuned and us[1] < 1.03 * us[0]       # (the pair takes 1.05 times as long)
        t = di.mlp_inputs_torch(M, d, ff, seed=7, device=DEV)
        ws = dfk.new_workspace(M, d, ff, DEV)
        a, b = torch.empty_like(t["X"]), torch.empty_like(t["X"])
        dfk.dfk_swiglu_mlp_ex(t["X"], t["Wg"], t["Wu"], t["Wd"], a, None, ws)
        dfk.dfk_set_workspace(ws)
        dfk.dfk_swiglu_mlp_fused(t["X"], t["Wg"], t["Wu"], t["Wd"], b)
        torch.cuda.synchronize()
        assert float((a.float() - b.float()).norm() / b.float().norm()) < 1e-2
    finally:
        dfk.dfk_set_workspace(None)
        dfk.dfk_clear_tuning()
