"""256-token pair with the tokens divided among groups of workgroups: both sides of every line of the rules, last groups of few tokens and of all but
one, ragged d_ff, both layouts of W_down, with and without the normalisation.  The rules themselves are checked on the host (test_big_plan_host.py)."""
import pytest

torch = pytest.importorskip("torch")

import dfk_inputs as di
import paper_2602_11808_amd as dfk
from oracle import oracle
from tests.helpers import assert_parity

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

# tokens: two groups of 64 (the second of 1, 63 or 64), of 128 (65, 127, 128), four of 64; one group beyond the lines.  d_ff: three, four and
# eight row tiles of 128 slices and one more than each; fewer rows than slices; whole steps of the down kernel or not
CASES = [(65, 256, 3072), (127, 512, 3080), (128, 384, 1536), (129, 1024, 4096), (130, 512, 4104), (192, 640, 2048), (193, 2048, 1000), (200, 512, 8192),
         (256, 512, 8200), (255, 1152, 520), (129, 2176, 4096), (256, 2304, 4104), (70, 4096, 512), (256, 4224, 768), (68, 128, 64),
         # d_ff beyond the gate/up kernel's groups: two and four groups of the down kernel alone, up to 20, 32 and 64 MB of W_down and beyond; rows of the
         # grid that are filled up to a multiple of 8; splits cut to what fits, with whole 64-row steps and without
         (100, 256, 20480), (200, 384, 16392), (160, 896, 12288), (65, 640, 14336), (250, 1152, 9224), (130, 128, 28672), (256, 512, 28672)]


def _run(t, M, d, ff, dtype, cfg):
    g = {k: di.to_torch(v, DEV) for k, v in t.items()}
    ws = dfk.new_workspace(M, d, ff, DEV)
    buf = torch.full((M + 1, d), 7.0, dtype=g["X"].dtype, device=DEV)
    dfk.dfk_swiglu_mlp_ex(g["X"], g["Wg"], g["Wu"], g["Wd"], buf[:M], cfg, ws)
    torch.cuda.synchronize()
    assert bool((buf[M] == 7.0).all()), cfg
    assert int(torch.count_nonzero(ws[:4096 + 64 * 32768 * 4]).item()) == 0, cfg
    return buf[:M], g, ws


@pytest.mark.parametrize("M,d,ff", CASES)
def test_against_the_oracle(M, d, ff):
    dtype = "bf16" if M % 2 else "fp16"
    dt = dfk.DFK_BF16 if M % 2 else dfk.DFK_FP16
    t = di.mlp_inputs(M, d, ff, seed=97, dtype=dtype)
    ref = oracle.swiglu_mlp(t["X"], t["Wg"], t["Wu"], t["Wd"])
    pick, _ = dfk.dfk_get_choice(M, d, ff, dt)
    assert pick.kmajor == 2
    cfgs = [None] + [dfk.dfk_config_t(**dict(pick.as_dict(), **o)) for o in (dict(reduce=dfk.DFK_REDUCE_ATOMIC), dict(splits=min(512, ff // 8)), dict(k2_splits=1))]
    for cfg in cfgs:
        if cfg is not None and not dfk.dfk_config_valid(cfg, M, d, ff, dt):
            continue
        print("case", M, d, ff, cfg, flush=True)
        Y, g, ws = _run(t, M, d, ff, dtype, cfg)
        assert_parity(di.as_f64(di.to_numpy(Y)), ref, dtype, (M, d, ff, cfg))
    if ff % 128 == 0 and d >= 256:
        wt = torch.empty((d, ff), dtype=g["Wd"].dtype, device=DEV)
        dfk.dfk_transpose_w_down(g["Wd"], wt)
        Y = torch.full_like(g["X"], float("nan"))
        dfk.dfk_swiglu_mlp_wdt(g["X"], g["Wg"], g["Wu"], wt, Y, None, ws)
        torch.cuda.synchronize()
        assert_parity(di.as_f64(di.to_numpy(Y)), ref, dtype, (M, d, ff, "wdt"))


@pytest.mark.parametrize("M,d,ff", [(100, 512, 1536), (200, 1024, 4096)])
def test_the_block_in_both_layouts(M, d, ff):
    t = di.mlp_inputs(M, d, ff, seed=98)
    g = {k: di.to_torch(v, DEV) for k, v in t.items()}
    w = di.to_torch(di.mlp_inputs(1, d, 8, seed=99)["X"], DEV).reshape(d).contiguous()
    ref = oracle.mlp_block(t["X"], di.to_numpy(w), 1e-5, t["Wg"], t["Wu"], t["Wd"])
    ws = dfk.new_workspace(M, d, ff, DEV)
    wt = torch.empty((d, ff), dtype=g["Wd"].dtype, device=DEV)
    dfk.dfk_transpose_w_down(g["Wd"], wt)
    for fn, wd in ((dfk.dfk_mlp_block, g["Wd"]), (dfk.dfk_mlp_block_wdt, wt)):
        H = g["X"].clone()
        fn(H, w, 1e-5, g["Wg"], g["Wu"], wd, H, None, ws)       # in place
        torch.cuda.synchronize()
        assert_parity(di.as_f64(di.to_numpy(H)), ref, "bf16", fn.__name__)


@pytest.mark.parametrize("M", [193, 200, 230, 256])
def test_tuning_names_a_launch_once(M):
    """512 x 1536: 64 and 128 splits would be cut to the 12 that are listed too; the entry says what runs."""
    d, ff, bf = 512, 1536, dfk.DFK_BF16
    scratch = torch.empty(dfk.dfk_tune_scratch_bytes(M, d, ff, bf, 2), dtype=torch.uint8, device=DEV)
    n = dfk.dfk_num_candidates(M, d, ff, bf)
    offered = {c.k2_splits for c in (dfk.dfk_get_candidate(M, d, ff, bf, i) for i in range(n)) if c.kmajor == 2 and c.reduce == dfk.DFK_REDUCE_TICKET}
    assert {12, 64, 128} <= offered
    try:
        dfk.dfk_tune([M], d, ff, bf, scratch, sets=2, iters=5)
        c, tuned = dfk.dfk_get_choice(M, d, ff, bf)
        assert tuned and (c.kmajor != 2 or c.reduce != dfk.DFK_REDUCE_TICKET or c.k2_splits not in (64, 128)), c
    finally:
        dfk.dfk_clear_tuning()
