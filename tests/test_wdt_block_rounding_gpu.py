"""Transposed block beyond 64 tokens: the product of input and normalisation weight is what is rounded, as up to 64 tokens.  With weights of one that
is no rounding at all, so a token's result depends on the token count by the order of fp32 sums only."""
import pytest

torch = pytest.importorskip("torch")

import dfk_inputs as di
import paper_2602_11808_amd as dfk

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("dtype", ["bf16", "fp16"])
@pytest.mark.parametrize("M,d,ff", [(65, 512, 1024), (130, 896, 4864), (200, 2048, 1536), (256, 1152, 2048)])
def test_a_token_beside_many_others(M, d, ff, dtype):
    """Another rounding of every input moves a sum by about a third of an output's spacing and so changes a good part of the outputs; the order of
    sums, and the values of A_2 that it moves across a rounding boundary, about one in a hundred."""
    t = di.mlp_inputs(M, d, ff, seed=107, dtype=dtype)
    g = {k: di.to_torch(v, DEV) for k, v in t.items()}
    H = g["X"] * torch.linspace(0.5, 3.0, M, device=DEV)[:, None].to(g["X"].dtype)       # scales that differ from token to token
    Wd_t = g["Wd"].t().contiguous()
    ones = torch.ones(d, dtype=H.dtype, device=DEV)
    ws = dfk.new_workspace(M, d, ff, DEV)
    dt = dfk.DFK_BF16 if dtype == "bf16" else dfk.DFK_FP16
    pick, _ = dfk.dfk_get_choice_wdt(M, d, ff, dt)
    assert pick.k2_col_blocks > 1, pick
    many = torch.empty_like(H)
    dfk.dfk_mlp_block_wdt(H, ones, 1e-5, g["Wg"], g["Wu"], Wd_t, many, None, ws)
    for lo in range(0, M, 64):
        part = H[lo:lo + 64].contiguous()
        few = torch.empty_like(part)
        dfk.dfk_mlp_block_wdt(part, ones, 1e-5, g["Wg"], g["Wu"], Wd_t, few, None, ws)
        torch.cuda.synchronize()
        differ = float((few != many[lo:lo + 64]).float().mean())
        print("case", (M, d, ff), dtype, lo, "differ", differ, flush=True)
        assert differ < 0.08, (lo, differ)
