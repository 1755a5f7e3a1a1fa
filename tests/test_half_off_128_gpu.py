"""Half inputs at widths off 128: the 64-token pair with A_2 in fp32 on the fp32 matrix instructions, against the oracle and the plain-FMA kernels."""
import pytest

torch = pytest.importorskip("torch")

import dfk_inputs as di
import paper_2602_11808_amd as dfk
from oracle import oracle
from tests.helpers import assert_parity

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
HALF, TWO = dfk.DFK_FP16, dfk.DFK_VARIANT_TWO_KERNEL


def _cands(M, d, ff):
    return [dfk.dfk_get_candidate(M, d, ff, HALF, i) for i in range(dfk.dfk_num_candidates(M, d, ff, HALF))]


def _matrix(c, d):
    return c.variant == TWO and c.k2_col_blocks == (d + 127) // 128


# one 8-wide piece in the last chunk, all but one, a few; four and eight wavefronts; one to four token tiles, two launches; ragged d_ff; splits
# with a partial last block, more splits than blocks
@pytest.mark.parametrize("shape", [(2, 392, 520), (20, 504, 1000), (1, 520, 1000), (16, 632, 1536), (17, 1016, 2056), (33, 904, 520), (48, 1032, 1000), (64, 2296, 4104),
                                   (70, 888, 2816), (4, 4104, 8)], ids=lambda s: "M%d_d%d_ff%d" % s)
def test_against_the_oracle(shape):
    M, d, ff = shape
    t = di.mlp_inputs(M, d, ff, seed=57, dtype="fp16")
    ref = oracle.swiglu_mlp(t["X"], t["Wg"], t["Wu"], t["Wd"])
    g = {k: di.to_torch(v, DEV) for k, v in t.items()}
    ws = dfk.new_workspace(M, d, ff, DEV)
    pick, _ = dfk.dfk_get_choice(M, d, ff, HALF)
    assert _matrix(pick, d) and pick.a2_dtype == dfk.DFK_FP32, pick
    cfgs = [pick]
    for over in (dict(k2_splits=1), dict(k2_splits=7), dict(splits=min(ff // 8, 512)), dict(waves=4)):
        c = dfk.dfk_config_t(**dict(pick.as_dict(), **over))
        if dfk.dfk_config_valid(c, M, d, ff, HALF):
            cfgs.append(c)
    for cfg in [None] + cfgs:
        print("case", shape, cfg, flush=True)
        buf = torch.full((M + 1, d), 7.0, dtype=torch.float16, device=DEV)      # a guard row behind Y
        dfk.dfk_swiglu_mlp_ex(g["X"], g["Wg"], g["Wu"], g["Wd"], buf[:M], cfg, ws)
        torch.cuda.synchronize()
        assert_parity(di.as_f64(di.to_numpy(buf[:M])), ref, "fp16", (shape, cfg))
        assert bool((buf[M] == 7.0).all()), (shape, cfg)
        assert int(torch.count_nonzero(ws[:4096 + 64 * 32768 * 4]).item()) == 0, (shape, cfg)
    Y = torch.empty_like(g["X"])
    dfk.dfk_swiglu_mlp_static(g["X"], g["Wg"], g["Wu"], g["Wd"], Y)
    torch.cuda.synchronize()
    assert_parity(di.as_f64(di.to_numpy(Y)), ref, "fp16", (shape, "static"))


def _both(M, d, ff, g):
    ws = dfk.new_workspace(M, d, ff, DEV)
    out = []
    for want in (True, False):
        cfg = next(c for c in _cands(M, d, ff) if c.variant == TWO and _matrix(c, d) == want)
        Y = torch.empty_like(g["X"])
        dfk.dfk_swiglu_mlp_ex(g["X"], g["Wg"], g["Wu"], g["Wd"], Y, cfg, ws)
        torch.cuda.synchronize()
        out.append(Y.double().cpu())
    return out


@pytest.mark.parametrize("M", [3, 40])
def test_a2_beyond_the_range_of_half(M):
    """Gate and up sums near 1000: A_2 is near 1e6, which half cannot hold; fp32 does, as in the plain-FMA kernels."""
    d, ff = 520, 1000
    t = di.mlp_inputs(M, d, ff, seed=58, dtype="fp16")
    g = {k: di.to_torch(v, DEV) for k, v in t.items()}
    g["X"] = (g["X"].float() * 300).half()
    g["Wg"], g["Wu"], g["Wd"] = (g["Wg"].float() * 4).half(), (g["Wu"].float() * 4).half(), (g["Wd"].float() * 2.0 ** -9).half()      # (Y within the range of half)
    a, b = _both(M, d, ff, g)
    x = g["X"].double().cpu()
    up = x @ g["Wu"].double().cpu().t()
    gate = x @ g["Wg"].double().cpu().t()
    assert float((gate * up).abs().max()) > 65504
    ref = (gate / (1 + torch.exp(-gate)) * up) @ g["Wd"].double().cpu()
    assert float(ref.abs().max()) < 65504
    # one rounding to half of the result: 2^-12 to 2^-11 of each value
    for y in (a, b):
        assert float((y - ref).norm() / ref.norm()) < 2.0 ** -11


def test_weights_that_are_not_finite_stay_where_the_plain_kernels_keep_them():
    M, d, ff = 3, 1000, 1536
    t = di.mlp_inputs(M, d, ff, seed=61, dtype="fp16")
    g = {k: di.to_torch(v, DEV) for k, v in t.items()}
    g["Wu"][5, -1] = float("inf")
    g["Wd"][7, -1] = float("inf")
    g["Wd"][ff - 1, 3] = float("nan")
    a, b = _both(M, d, ff, g)
    assert torch.equal(torch.isnan(a), torch.isnan(b)) and torch.equal(torch.isinf(a), torch.isinf(b)) and not bool(torch.isfinite(a).all())


def test_one_token_of_a_large_layer_stays_on_the_plain_kernels():
    assert not _matrix(dfk.dfk_get_choice(1, 2888, 7688, HALF)[0], 2888)
    assert _matrix(dfk.dfk_get_choice(2, 2888, 7688, HALF)[0], 2888)


def _plain(M, d, ff, **over):
    c = next(c for c in _cands(M, d, ff) if c.variant == TWO and c.path == dfk.DFK_PATH_VALU and c.kmajor == 0)
    return dfk.dfk_config_t(**dict(c.as_dict(), **over))


def test_plain_fma_by_name_within_the_static_scratch():
    """Eight tokens per launch: 160 splits of them fit the array, of 64 tokens they would not."""
    M, d, ff = 64, 1000, 1536
    t = di.mlp_inputs(M, d, ff, seed=63, dtype="fp16")
    ref = oracle.swiglu_mlp(t["X"], t["Wg"], t["Wu"], t["Wd"])
    g = {k: di.to_torch(v, DEV) for k, v in t.items()}
    Y = torch.full_like(g["X"], float("nan"))
    dfk.dfk_swiglu_mlp_static(g["X"], g["Wg"], g["Wu"], g["Wd"], Y, _plain(M, d, ff, k2_splits=160, k2_col_blocks=8))
    torch.cuda.synchronize()
    assert_parity(di.as_f64(di.to_numpy(Y)), ref, "fp16", "static")


@pytest.mark.parametrize("M", [3, 40])
def test_an_input_that_is_not_finite_stays_in_its_token(M):
    d, ff = 1000, 1536
    t = di.mlp_inputs(M, d, ff, seed=64, dtype="fp16")
    g = {k: di.to_torch(v, DEV) for k, v in t.items()}
    clean = [y.clone() for y in _both(M, d, ff, g)]
    g["X"][1, d - 1] = float("inf")
    g["X"][M - 1, 5] = float("nan")
    for y, was in zip(_both(M, d, ff, g), clean):
        assert bool(torch.isnan(y[M - 1]).all()) and not bool(torch.isfinite(y[1]).any())
        rest = [m for m in range(M) if m not in (1, M - 1)]
        assert torch.equal(y[rest], was[rest])
