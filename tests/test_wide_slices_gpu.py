"""256-token pair, gate/up kernel with slices of 9 to 16 row tiles: every token-tile count it is built for, shortest and longest slices and two rounds
of them, d_ff that leaves slices of two lengths, few and many steps of the k range, both layouts of W_down, with and without the normalisation.
Which d_ff and tokens get it is checked on the host (test_big_plan_host.py)."""
import pytest

torch = pytest.importorskip("torch")

import dfk_inputs as di
import paper_2602_11808_amd as dfk
from oracle import oracle
from tests.helpers import assert_parity

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

# up to 128, 192 and 256 tokens: slices of at most 16, 14 and 10 tiles; 2048 d_ff rows are one tile in each of 256 slices, so these have 9 (one
# slice of them, or all), 10, 11, 12, 13, 14, 16, and one more than the longest (two rounds, or the form for slices of up to 8)
CASES = [(65, 256, 16392), (128, 128, 18432), (127, 384, 22536), (100, 256, 28672), (97, 384, 32768), (128, 256, 32776), (66, 256, 61448),
         (129, 256, 16392), (192, 128, 20480), (150, 640, 24576), (191, 256, 26632), (160, 384, 28672), (130, 256, 28680), (192, 256, 53248),
         (193, 256, 16392), (256, 384, 20480), (255, 128, 20488)]


@pytest.mark.parametrize("M,d,ff", CASES)
def test_against_the_oracle(M, d, ff):
    dtype = "bf16" if M % 2 else "fp16"
    t = di.mlp_inputs(M, d, ff, seed=101, dtype=dtype)
    ref = oracle.swiglu_mlp(t["X"], t["Wg"], t["Wu"], t["Wd"])
    assert dfk.dfk_get_choice(M, d, ff, dfk.DFK_BF16 if M % 2 else dfk.DFK_FP16)[0].kmajor == 2
    g = {k: di.to_torch(v, DEV) for k, v in t.items()}
    ws = dfk.new_workspace(M, d, ff, DEV)
    buf = torch.full((M + 1, d), 7.0, dtype=g["X"].dtype, device=DEV)
    print("case", M, d, ff, flush=True)
    dfk.dfk_swiglu_mlp_ex(g["X"], g["Wg"], g["Wu"], g["Wd"], buf[:M], None, ws)
    torch.cuda.synchronize()
    assert bool((buf[M] == 7.0).all())
    assert_parity(di.as_f64(di.to_numpy(buf[:M])), ref, dtype, (M, d, ff))


# more than 64 steps, which wrap every ring many times: starts of the k walk over the whole range (X up to 3 MB), and in the window of 64 steps
# (X beyond), with steps that are no multiple of it
@pytest.mark.parametrize("M,d,ff", [(66, 8192, 16392), (150, 8192, 16512), (255, 4224, 16448), (256, 8320, 16392)])
def test_many_steps(M, d, ff):
    """Every sixteenth token against plain torch in 64 bits (the oracle takes minutes at these sizes), all of them against repeats."""
    g = torch.Generator(device=DEV)
    g.manual_seed(104)
    t = [(torch.randn(s, generator=g, device=DEV) * w).to(torch.bfloat16) for s, w in (((M, d), 1.0), ((ff, d), d ** -0.5), ((ff, d), d ** -0.5), ((ff, d), ff ** -0.5))]
    assert dfk.dfk_get_choice(M, d, ff)[0].kmajor == 2
    ws = dfk.new_workspace(M, d, ff, DEV)
    first = None
    for rep in range(3):
        buf = torch.full((M + 1, d), 7.0, dtype=torch.bfloat16, device=DEV)
        print("case", M, d, ff, rep, flush=True)
        dfk.dfk_swiglu_mlp_ex(*t, buf[:M], None, ws)
        torch.cuda.synchronize()
        assert bool((buf[M] == 7.0).all())
        first = buf.clone() if first is None else first
        assert torch.equal(first.view(torch.int16), buf.view(torch.int16)), rep       # fixed order: the same bits every time
    rows = sorted({0, 15, 16, 63, 64, M - 1} | set(range(3, M, 16)))
    x = t[0][rows].double()
    gate = torch.cat([x @ w.double().t() for w in t[1].split(2048)], 1)
    up = torch.cat([x @ w.double().t() for w in t[2].split(2048)], 1)
    a = gate / (1 + torch.exp(-gate)) * up
    ref = sum(p @ w.double() for p, w in zip(a.split(2048, 1), t[3].split(2048)))
    assert_parity(first[rows].double().cpu().numpy(), ref.cpu().numpy(), "bf16", (M, d, ff))


@pytest.mark.parametrize("M,ff", [(100, 30720), (150, 24576), (200, 18432)])
def test_the_block_in_both_layouts(M, ff):
    d = 256
    t = di.mlp_inputs(M, d, ff, seed=102)
    g = {k: di.to_torch(v, DEV) for k, v in t.items()}
    w = di.to_torch(di.mlp_inputs(1, d, 8, seed=103)["X"], DEV).reshape(d).contiguous()
    ref = oracle.mlp_block(t["X"], di.to_numpy(w), 1e-5, t["Wg"], t["Wu"], t["Wd"])
    ws = dfk.new_workspace(M, d, ff, DEV)
    wt = torch.empty((d, ff), dtype=g["Wd"].dtype, device=DEV)
    dfk.dfk_transpose_w_down(g["Wd"], wt)
    for fn, wd in ((dfk.dfk_mlp_block, g["Wd"]), (dfk.dfk_mlp_block_wdt, wt)):
        H = g["X"].clone()
        print("case", fn.__name__, M, d, ff, flush=True)
        fn(H, w, 1e-5, g["Wg"], g["Wu"], wd, H, None, ws)       # in place
        torch.cuda.synchronize()
        assert_parity(di.as_f64(di.to_numpy(H)), ref, "bf16", fn.__name__)
