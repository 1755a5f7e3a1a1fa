"""Gate values far below zero beside very large up values (bf16 only: half cannot hold them): SiLU(gate) is zero there, or small, and
so is its product with up, although gate times up is beyond fp32's range.  Every kernel family against the oracle."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import dfk_inputs as di
import paper_2602_11808_amd as dfk
from oracle import oracle
from tests.helpers import assert_parity

DEV = "cuda:0"
# d_ff row -> its gate and up value.  SiLU(-86) = -3.8e-36: the product with 5e36 is -19, gate * up is beyond fp32's range.
ROWS = {3: (-1.0e20, 1.0e35), 40: (-200.0, 3.0e38), 77: (-60.0, 1.0e25), 111: (-1.0e10, -1.0e38), 130: (-86.0, 5.0e36)}


def _inputs(M, d, ff):
    t = di.mlp_inputs(M, d, ff, seed=97)
    one = di.f32_to_bf16_bits(np.array([1.0], np.float32))[0]
    t["X"][:, 0] = one                      # k = 0 sets the gate and up values of these rows, and of no others
    t["Wg"][:, 0] = 0
    t["Wu"][:, 0] = 0
    for j, (g, u) in ROWS.items():
        t["Wg"][j, :] = 0
        t["Wu"][j, :] = 0
        t["Wg"][j, 0], t["Wu"][j, 0] = di.f32_to_bf16_bits(np.array([g, u], np.float32))
    return t


def test_the_product_of_gate_and_up_overflows_and_the_result_does_not():
    for j in (3, 40, 111, 130):
        g, u = ROWS[j]
        with np.errstate(over="ignore"):
            assert np.isinf(np.float32(u) * np.float32(g))
        assert abs(u * oracle.silu(g)) < 20.0


@pytest.mark.gpu
@pytest.mark.parametrize("shape", [(3, 1000, 520), (3, 1024, 520), (33, 1048, 520), (64, 1024, 520), (100, 256, 520)], ids=lambda s: "M%d_d%d" % s[:2])
def test_large_up_behind_a_closed_gate(shape):
    M, d, ff = shape
    t = _inputs(M, d, ff)
    ref = oracle.swiglu_mlp(t["X"], t["Wg"], t["Wu"], t["Wd"])
    assert np.all(np.isfinite(ref)) and float(np.max(np.abs(ref))) < 100.0
    g = {k: di.to_torch(v, DEV) for k, v in t.items()}
    ws = dfk.new_workspace(M, d, ff, DEV)
    Wd_t = g["Wd"].t().contiguous()
    n, nt = dfk.dfk_num_candidates(M, d, ff, dfk.DFK_BF16), dfk.dfk_num_candidates_wdt(M, d, ff, dfk.DFK_BF16)
    calls = [(dfk.dfk_swiglu_mlp_ex, g["Wd"], dfk.dfk_get_candidate(M, d, ff, dfk.DFK_BF16, i)) for i in range(n)]
    calls += [(dfk.dfk_swiglu_mlp_wdt, Wd_t, dfk.dfk_get_candidate_wdt(M, d, ff, dfk.DFK_BF16, i)) for i in range(nt)]
    for fn, wd, cfg in calls:
        print("case", shape, fn.__name__, cfg, flush=True)
        Y = torch.full_like(g["X"], float("nan"))
        fn(g["X"], g["Wg"], g["Wu"], wd, Y, cfg, ws)
        torch.cuda.synchronize()
        assert_parity(di.as_f64(di.to_numpy(Y)), ref, "bf16", (shape, cfg))
