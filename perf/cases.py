"""What the framework's speed is measured on: SwiGLU MLP calls as a serving program makes them.

Every case is one decoder-layer MLP, or a short chain of them, through the public entry points.  The scheduler's
own choice is used throughout (no tuning table is loaded): the token count of a serving step changes from step to
step, and this is what a program gets that has not profiled its shapes beforehand.  The fp32 test mode is left out,
it exists to check the other types.

Fields of a case:
    op       "mlp" Y = MLP(X); "block" H + MLP(RMSNorm(H)); the suffix "_wdt": W_down as [d_model, d_ff], the layout a
             linear layer keeps its weights in
    m        tokens of the call;  d, ff: layer widths;  dtype: "bf16" or "fp16"
    layers   1: one eager call.  More: that many layers with weights of their own, each reading what the one before it
             wrote, captured once in a graph that a pass replays (how a decode step is deployed)
"""
import math

import torch

import paper_2602_11808_amd as dfk

EPS = 1e-5
DTYPES = {"bf16": torch.bfloat16, "fp16": torch.float16}


def _case(name, op, m, d, ff, dtype="bf16", layers=1):
    return {"name": name, "op": op, "m": m, "d": d, "ff": ff, "dtype": dtype, "layers": layers}


def listed():
    return [
        # the smallest call: a toy or draft model's layer, one token; launches and host work are all there is
        _case("tiny M1", "mlp", 1, 512, 1536),
        # a half-billion-parameter model's decode step: 24 layers replayed from a graph, one token
        _case("small x24 M1", "block", 1, 896, 4864, layers=24),
        # a two-billion-parameter model's layer with its weights as linear layers keep them, a handful of users
        _case("2b wdt M8", "mlp_wdt", 8, 2304, 9216),
        # a width that is no multiple of 128, a few users
        _case("odd width M12", "mlp", 12, 2888, 7688),
        # the ordinary layer (Llama-3-8B-shaped): one user, then a replayed pass for sixteen
        _case("8b M1", "mlp", 1, 4096, 14336),
        _case("8b wdt x4 M16", "block_wdt", 16, 4096, 14336, layers=4),
        # the same layer under load: a full decode batch, then as many tokens as a call takes (chunked prefill)
        _case("8b M64", "mlp", 64, 4096, 14336),
        _case("8b M256", "mlp", 256, 4096, 14336),
        # the shard of a Llama-3-70B-shaped layer that one of four GPUs holds, in half, a ragged batch
        _case("70b shard fp16 M33", "mlp", 33, 8192, 7168, "fp16"),
        # a Qwen2.5-32B-shaped layer with its neighbours, a few users
        _case("32b block M4", "block", 4, 5120, 27648),
        # a whole Llama-3-70B-shaped layer with its neighbours, a ragged prefill chunk
        _case("70b block M150", "block", 150, 8192, 28672),
        # the largest layer (405B-sized), a few tokens
        _case("405b M2", "mlp", 2, 16384, 53248),
    ]


def _spread(rng, lo, hi):
    """Spread over the logarithm, both ends included."""
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def draw(rng):
    while True:
        op = rng.choice(["mlp", "mlp", "mlp", "block", "block", "mlp_wdt", "block_wdt"])
        m = min(256, int(_spread(rng, 1, 257)))
        ragged = op == "mlp" and rng.random() < 0.35
        if ragged:   # any multiple of 8; wide ones of this kind are not met
            d = int(_spread(rng, 512, 3000)) // 8 * 8
            ff = int(d * _spread(rng, 1.0, 5.5)) // 8 * 8
        else:
            d = int(round(_spread(rng, 4, 128))) * 128
            ff = max(1024, int(d * _spread(rng, 0.875, 5.5)) // 128 * 128)
        layers = rng.choice([4, 8]) if d * ff <= 4096 * 14336 and m <= 64 and not ragged and rng.random() < 0.25 else 1
        c = {"op": op, "m": m, "d": d, "ff": ff, "dtype": rng.choice(["bf16", "bf16", "bf16", "fp16"]), "layers": layers}
        if ff > 53248 or (op.endswith("_wdt") and m > 64 and d * ff > 8192 * 7168):
            continue
        w = work(c)
        if w["bytes"] <= 4.5e9 and w["flops"] <= 3e11:   # no more than the largest listed calls
            return c


def _inputs(case, seed):
    """X (or H) ~ N(0, 1), weights ~ N(0, 1 / fan_in), normalisation weights near 1, all rounded to the type."""
    m, d, ff, dt = case["m"], case["d"], case["ff"], DTYPES[case["dtype"]]
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)

    def normal(rows, cols, std):
        t = torch.empty((rows, cols), dtype=dt, device="cuda")
        step = max(1, (64 << 20) // cols)
        for lo in range(0, rows, step):
            hi = min(rows, lo + step)
            t[lo:hi] = torch.randn((hi - lo, cols), generator=g, device="cuda", dtype=torch.float32) * std
        return t

    x = normal(m, d, 1.0)
    layers = []
    for _ in range(case["layers"]):
        wd = (d, ff) if case["op"].endswith("_wdt") else (ff, d)
        layers.append({"gate": normal(ff, d, d ** -0.5), "up": normal(ff, d, d ** -0.5), "down": normal(*wd, ff ** -0.5),
                       "norm": (1.0 + 0.1 * torch.randn(d, generator=g, device="cuda")).to(dt)})
    return x, layers


def _call(op, x, w, y, ws):
    if op == "mlp":
        dfk.dfk_swiglu_mlp_ex(x, w["gate"], w["up"], w["down"], y, None, ws)
    elif op == "mlp_wdt":
        dfk.dfk_swiglu_mlp_wdt(x, w["gate"], w["up"], w["down"], y, None, ws)
    elif op == "block":
        dfk.dfk_mlp_block(x, w["norm"], EPS, w["gate"], w["up"], w["down"], y, None, ws)
    else:
        dfk.dfk_mlp_block_wdt(x, w["norm"], EPS, w["gate"], w["up"], w["down"], y, None, ws)


def prepare(case, seed):
    x, layers = _inputs(case, seed)
    ws = dfk.new_workspace(case["m"], case["d"], case["ff"], "cuda")
    ys = [torch.empty_like(x) for _ in layers]
    state = {"op": case["op"], "x": x, "layers": layers, "ys": ys, "ws": ws, "graph": None}
    if len(layers) > 1:
        _eager(state)                       # once before the capture, as torch asks for
        torch.cuda.synchronize()
        state["graph"] = torch.cuda.CUDAGraph()
        with torch.cuda.graph(state["graph"]):
            _eager(state)
    return state


def _eager(state):
    x = state["x"]
    for w, y in zip(state["layers"], state["ys"]):
        _call(state["op"], x, w, y, state["ws"])
        x = y


def run(state):
    if state["graph"] is not None:
        state["graph"].replay()
    else:
        _eager(state)
    return state["ys"][-1]


def work(case):
    m, d, ff, n = case["m"], case["d"], case["ff"], case["layers"]
    norm = 2 * d if case["op"].startswith("block") else 0
    return {"bytes": float(n * (6 * d * ff + 4 * m * d + norm)), "flops": float(n * 6 * m * d * ff)}


def tolerance(case):
    # Two roundings to the type per layer (A_2 and the output): an eager call is 2.3e-3 (bf16) / 2.9e-4 (fp16) off the
    # 64-bit result; a chain feeds its rounded values on (4 layers 4.8e-3, 24 layers 1.6e-2).  Four times that.
    grow = 1.0 + 0.3 * (case["layers"] - 1)
    return {"rel": (1e-2 if case["dtype"] == "bf16" else 1.2e-3) * grow, "max": (8e-2 if case["dtype"] == "bf16" else 1e-2) * grow}


def exact(case, seed):
    x, layers = _inputs(case, seed)
    x = x.double()
    wdt = case["op"].endswith("_wdt")
    for w in layers:
        h = x
        if case["op"].startswith("block"):
            h = x * w["norm"].double() / torch.sqrt((x * x).mean(1, keepdim=True) + EPS)
        y = torch.zeros_like(x)
        step = max(8, (64 << 20) // case["d"])
        for lo in range(0, case["ff"], step):
            hi = min(case["ff"], lo + step)
            gate, up = h @ w["gate"][lo:hi].double().t(), h @ w["up"][lo:hi].double().t()
            a = gate / (1.0 + torch.exp(-gate)) * up
            y += a @ (w["down"][:, lo:hi].double().t().contiguous() if wdt else w["down"][lo:hi].double())
        x = x + y if case["op"].startswith("block") else y
    return x
