"""Counter reduction of the 64-token pair's down kernel: the launch that adds the splits' blocks up.  Split counts on both sides of its batches, both
workgroup sizes, both sides of the line in the single launch of both kernels' workgroups, a width off 128, the residual in place."""
import pytest

torch = pytest.importorskip("torch")

import dfk_inputs as di
import paper_2602_11808_amd as dfk
from oracle import oracle
from tests.helpers import assert_parity

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
TWO, FUSED = dfk.DFK_VARIANT_TWO_KERNEL, dfk.DFK_VARIANT_FUSED


def _cfg(M, d, ff, dt, **over):
    n = dfk.dfk_num_candidates(M, d, ff, dt)
    c = next(c for c in (dfk.dfk_get_candidate(M, d, ff, dt, i) for i in range(n))
             if c.variant == TWO and c.kmajor == 1 and c.reduce == dfk.DFK_REDUCE_TICKET and c.waves == (8 if d >= 1000 else 4))
    return dfk.dfk_config_t(**dict(c.as_dict(), **over))


@pytest.mark.parametrize("dtype", ["bf16", "fp16"])
@pytest.mark.parametrize("M,d,ff", [(1, 512, 1000), (3, 1024, 1536), (4, 1024, 1536), (17, 512, 1544), (64, 1024, 2048), (64, 4096, 520)])
def test_splits_are_summed_by_a_launch(M, d, ff, dtype):
    dt = dfk.DFK_BF16 if dtype == "bf16" else dfk.DFK_FP16
    t = di.mlp_inputs(M, d, ff, seed=91, dtype=dtype)
    ref = oracle.swiglu_mlp(t["X"], t["Wg"], t["Wu"], t["Wd"])
    g = {k: di.to_torch(v, DEV) for k, v in t.items()}
    ws = dfk.new_workspace(M, d, ff, DEV)
    single = [dict(variant=FUSED, kmajor=4, depth=4)] if d >= 1024 else []
    for form in [{}] + single:
        for splits in (1, 7, 8, 9, 16, 17, 33):
            cfg = _cfg(M, d, ff, dt, k2_splits=splits, **form)
            if not dfk.dfk_config_valid(cfg, M, d, ff, dt):
                continue
            print("case", M, d, ff, dtype, cfg, flush=True)
            first = None
            for _ in range(2):
                Y = torch.full_like(g["X"], float("nan"))
                dfk.dfk_swiglu_mlp_ex(g["X"], g["Wg"], g["Wu"], g["Wd"], Y, cfg, ws)
                torch.cuda.synchronize()
                assert_parity(di.as_f64(di.to_numpy(Y)), ref, dtype, cfg)
                first = Y.clone() if first is None else first
                assert torch.equal(first.view(torch.uint8), Y.view(torch.uint8)), cfg
            assert int(torch.count_nonzero(ws[:4096 + 64 * 32768 * 4]).item()) == 0, cfg


@pytest.mark.parametrize("M,d,ff", [(2, 1000, 1000), (33, 2008, 2400)])
def test_a_width_off_128(M, d, ff):
    t = di.mlp_inputs(M, d, ff, seed=92)
    ref = oracle.swiglu_mlp(t["X"], t["Wg"], t["Wu"], t["Wd"])
    g = {k: di.to_torch(v, DEV) for k, v in t.items()}
    ws = dfk.new_workspace(M, d, ff, DEV)
    for splits in (1, 9, 17):
        cfg = _cfg(M, d, ff, dfk.DFK_BF16, k2_splits=splits)
        buf = torch.full((M + 1, d), 7.0, dtype=torch.bfloat16, device=DEV)
        dfk.dfk_swiglu_mlp_ex(g["X"], g["Wg"], g["Wu"], g["Wd"], buf[:M], cfg, ws)
        torch.cuda.synchronize()
        assert_parity(di.as_f64(di.to_numpy(buf[:M])), ref, "bf16", cfg)
        assert bool((buf[M] == 7.0).all()), cfg


@pytest.mark.parametrize("M", [1, 20])
def test_a_block_in_place(M):
    """The sum adds the residual where it stores, so the output may be the input: the same bits."""
    d, ff = 896, 1536
    t = di.mlp_inputs(M, d, ff, seed=93)
    g = {k: di.to_torch(v, DEV) for k, v in t.items()}
    w = torch.linspace(0.5, 1.5, d, device=DEV).to(torch.bfloat16)
    ws = dfk.new_workspace(M, d, ff, DEV)
    out, H = torch.empty_like(g["X"]), g["X"].clone()
    dfk.dfk_mlp_block(g["X"], w, 1e-5, g["Wg"], g["Wu"], g["Wd"], out, None, ws)
    dfk.dfk_mlp_block(H, w, 1e-5, g["Wg"], g["Wu"], g["Wd"], H, None, ws)
    torch.cuda.synchronize()
    assert torch.equal(out, H)


@pytest.mark.parametrize("M", [1, 2, 3, 5, 8, 16])
def test_the_bits_do_not_depend_on_who_adds(M):
    """Small calls take the launch only under capture: replays give what the eager call gives, bit for bit, whatever the split count."""
    d, ff = 512, 1544
    t = di.mlp_inputs(M, d, ff, seed=94)
    g = {k: di.to_torch(v, DEV) for k, v in t.items()}
    ws = dfk.new_workspace(M, d, ff, DEV)
    for splits in (1, 2, 3, 7, 12, 16, 31):
        cfg = _cfg(M, d, ff, dfk.DFK_BF16, k2_splits=splits)
        eager = torch.empty_like(g["X"])
        dfk.dfk_swiglu_mlp_ex(g["X"], g["Wg"], g["Wu"], g["Wd"], eager, cfg, ws)
        torch.cuda.synchronize()
        Y = torch.empty_like(eager)
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            dfk.dfk_swiglu_mlp_ex(g["X"], g["Wg"], g["Wu"], g["Wd"], Y, cfg, ws)
        for _ in range(3):
            Y.fill_(float("nan"))
            graph.replay()
            torch.cuda.synchronize()
            assert torch.equal(Y, eager), (M, splits)


# fewest outputs per workgroup that a launch adds up, where its partial sums per output (4, 2, 1) differ with the tokens and the column blocks
@pytest.mark.parametrize("M", [1, 3, 4, 5, 8, 9])
@pytest.mark.parametrize("d,ff,dtype", [(1024, 1544, "bf16"), (1024, 1544, "fp16"), (1000, 1544, "bf16")])
def test_the_single_launch_gives_the_bits_of_the_pair(M, d, ff, dtype):
    dt = dfk.DFK_BF16 if dtype == "bf16" else dfk.DFK_FP16
    t = di.mlp_inputs(M, d, ff, seed=95, dtype=dtype)
    g = {k: di.to_torch(v, DEV) for k, v in t.items()}
    ws = dfk.new_workspace(M, d, ff, DEV)
    ran = 0
    for k2c in (8, 4):
        for splits in (1, 2, 3, 7, 12, 16):
            pair = _cfg(M, d, ff, dt, k2_splits=splits, k2_col_blocks=k2c)
            one = dfk.dfk_config_t(**dict(pair.as_dict(), variant=FUSED, kmajor=4, depth=4))
            if not (dfk.dfk_config_valid(pair, M, d, ff, dt) and dfk.dfk_config_valid(one, M, d, ff, dt)):
                continue
            out = []
            for cfg in (pair, one):
                Y = torch.full_like(g["X"], float("nan"))
                dfk.dfk_swiglu_mlp_ex(g["X"], g["Wg"], g["Wu"], g["Wd"], Y, cfg, ws)
                torch.cuda.synchronize()
                out.append(Y.view(torch.int16))
            assert torch.equal(*out), (pair, int((out[0] != out[1]).sum()))
            ran += 1
    assert ran >= 6
