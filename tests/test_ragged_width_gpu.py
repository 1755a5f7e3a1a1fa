"""d_model any multiple of 8 on the matrix cores (bf16): the last 128-k chunk and the last 128-column block are partial."""
import pytest

torch = pytest.importorskip("torch")

import dfk_inputs as di
import paper_2602_11808_amd as dfk
from oracle import oracle
from tests.helpers import assert_parity

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _pair(M, d, ff):
    n = dfk.dfk_num_candidates(M, d, ff, dfk.DFK_BF16)
    return [c for c in (dfk.dfk_get_candidate(M, d, ff, dfk.DFK_BF16, i) for i in range(n))
            if c.path == dfk.DFK_PATH_MFMA]


# one 8-wide piece in the last chunk, all but one, a few; one to four token tiles and two launches; ragged d_ff; chunk
# counts that do and do not divide among the wavefronts; column blocks paired (an even number of them) or not
@pytest.mark.parametrize("shape", [(2, 392, 520), (20, 504, 1000), (1, 520, 1000), (16, 632, 1536), (17, 1016, 2056), (33, 904, 520), (48, 1032, 1000), (64, 2296, 4104),
                                   (70, 888, 2816), (12, 2888, 7688)], ids=lambda s: "M%d_d%d_ff%d" % s)
def test_partial_last_chunk_and_column_block(shape):
    M, d, ff = shape
    t = di.mlp_inputs(M, d, ff, seed=53)
    ref = oracle.swiglu_mlp(t["X"], t["Wg"], t["Wu"], t["Wd"])
    g = {k: di.to_torch(v, DEV) for k, v in t.items()}
    ws = dfk.new_workspace(M, d, ff, DEV)
    cfgs = _pair(M, d, ff)
    assert {c.kmajor for c in cfgs} == {1}
    assert {c.reduce for c in cfgs} == {dfk.DFK_REDUCE_TICKET, dfk.DFK_REDUCE_ATOMIC}
    pick, _ = dfk.dfk_get_choice(M, d, ff, dfk.DFK_BF16)
    assert pick.path == dfk.DFK_PATH_MFMA
    for cfg in [None] + cfgs:
        print("case", shape, cfg, flush=True)
        # a guard row behind Y: columns past d_model must not be stored
        buf = torch.full((M + 1, d), 7.0, dtype=torch.bfloat16, device=DEV)
        Y = buf[:M]
        dfk.dfk_swiglu_mlp_ex(g["X"], g["Wg"], g["Wu"], g["Wd"], Y, cfg, ws)
        torch.cuda.synchronize()
        assert_parity(di.as_f64(di.to_numpy(Y)), ref, "bf16", (shape, cfg))
        assert bool((buf[M] == 7.0).all()), (shape, cfg)
        assert int(torch.count_nonzero(ws[:4096 + 64 * 32768 * 4]).item()) == 0, (shape, cfg)


def test_weights_that_are_not_finite_at_a_rows_end_stay_in_their_row():
    """An infinite last weight of one row (the element the pieces past the row's end are fetched from) reaches exactly
    the outputs the plain-FMA kernels let it reach."""
    M, d, ff = 3, 1000, 1536
    t = di.mlp_inputs(M, d, ff, seed=61)
    g = {k: di.to_torch(v, DEV) for k, v in t.items()}
    g["Wu"][5, -1] = float("inf")
    g["Wd"][7, -1] = float("inf")
    ws = dfk.new_workspace(M, d, ff, DEV)
    n = dfk.dfk_num_candidates(M, d, ff, dfk.DFK_BF16)
    cands = [dfk.dfk_get_candidate(M, d, ff, dfk.DFK_BF16, i) for i in range(n)]
    got = {}
    for path in (dfk.DFK_PATH_VALU, dfk.DFK_PATH_MFMA):
        cfg = next(c for c in cands if c.path == path and c.variant == dfk.DFK_VARIANT_TWO_KERNEL)
        Y = torch.empty_like(g["X"])
        dfk.dfk_swiglu_mlp_ex(g["X"], g["Wg"], g["Wu"], g["Wd"], Y, cfg, ws)
        torch.cuda.synchronize()
        got[path] = Y.float().cpu()
    a, b = got[dfk.DFK_PATH_VALU], got[dfk.DFK_PATH_MFMA]
    assert torch.equal(torch.isnan(a), torch.isnan(b)) and torch.equal(torch.isposinf(a), torch.isposinf(b))
    assert torch.equal(torch.isneginf(a), torch.isneginf(b)) and not bool(torch.isfinite(a).all())
