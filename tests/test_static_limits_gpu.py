"""dfk_swiglu_mlp_static where the untuned choice's partial sums exceed its array: it takes the best-ranked configuration that fits."""
import copy

import pytest

torch = pytest.importorskip("torch")

import dfk_inputs as di
import paper_2602_11808_amd as dfk

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def test_fewer_splits_of_the_same_pair_where_the_choice_does_not_fit():
    M, d, ff = 256, 2048, 11264                     # 16 splits: 33.5 MB of partial sums, of which about 27 fit beside A_2
    g = di.mlp_inputs_torch(M, d, ff, seed=5, device=DEV)
    pick, _ = dfk.dfk_get_choice(M, d, ff, dfk.DFK_BF16)
    assert (pick.kmajor, pick.k2_splits, pick.reduce) == (2, 16, dfk.DFK_REDUCE_TICKET)
    fewer = copy.copy(pick)
    fewer.k2_splits = 12
    ws = dfk.new_workspace(M, d, ff, DEV)
    want, got = torch.empty_like(g["X"]), torch.full_like(g["X"], float("nan"))
    print("case", (M, d, ff), fewer, flush=True)
    dfk.dfk_swiglu_mlp_ex(g["X"], g["Wg"], g["Wu"], g["Wd"], want, fewer, ws)
    dfk.dfk_swiglu_mlp_static(g["X"], g["Wg"], g["Wu"], g["Wd"], got)
    torch.cuda.synchronize()
    assert torch.equal(want.view(torch.uint8), got.view(torch.uint8))
