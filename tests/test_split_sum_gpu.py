"""The counter reduction of the 64-token pair's down kernel where the splits' blocks are divided among the threads: split counts
from one to more than there are threads per output, token counts on both sides of the form's limit."""
import copy

import pytest

torch = pytest.importorskip("torch")

import dfk_inputs as di
import paper_2602_11808_amd as dfk
from oracle import oracle
from tests.helpers import assert_parity

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("d,ff", [(1024, 1536), (1048, 1000)], ids=["whole_blocks", "partial_block"])
@pytest.mark.parametrize("M", [1, 3, 4, 5, 8, 9])
def test_sum_over_any_number_of_splits(M, d, ff):
    t = di.mlp_inputs(M, d, ff, seed=71)
    ref = oracle.swiglu_mlp(t["X"], t["Wg"], t["Wu"], t["Wd"])
    g = {k: di.to_torch(v, DEV) for k, v in t.items()}
    ws = dfk.new_workspace(M, d, ff, DEV)
    base = next(c for c in (dfk.dfk_get_candidate(M, d, ff, dfk.DFK_BF16, i) for i in range(dfk.dfk_num_candidates(M, d, ff, dfk.DFK_BF16)))
                if c.kmajor == 1 and c.variant == dfk.DFK_VARIANT_TWO_KERNEL and c.reduce == dfk.DFK_REDUCE_TICKET)
    nblk = (d + 127) // 128
    ran = 0
    for waves, depth in ((8, 3), (4, 6)):
        for width in (1, 2):                       # 128-column blocks per workgroup
            for splits in (1, 2, 7, 12, 16, 17, 40):
                cfg = copy.copy(base)
                cfg.waves, cfg.depth, cfg.k2_col_blocks, cfg.k2_splits = waves, depth, nblk // width, splits
                if nblk % width or not dfk.dfk_config_valid(cfg, M, d, ff, dfk.DFK_BF16):
                    continue
                print("case", M, d, ff, cfg, flush=True)
                first = None
                for _ in range(2):
                    Y = torch.full_like(g["X"], float("nan"))
                    dfk.dfk_swiglu_mlp_ex(g["X"], g["Wg"], g["Wu"], g["Wd"], Y, cfg, ws)
                    torch.cuda.synchronize()
                    assert_parity(di.as_f64(di.to_numpy(Y)), ref, "bf16", cfg)
                    first = Y.clone() if first is None else first
                    assert torch.equal(first.view(torch.uint8), Y.view(torch.uint8)), cfg
                assert int(torch.count_nonzero(ws[:4096 + 64 * 32768 * 4]).item()) == 0, cfg
                ran += 1
    assert ran >= 14
