"""Timed cases of the library's public entry points, over the range a user of it calls them in.

Kinds of a case:

  step     one decode step of an FFN stack: clada_signals_threshold on the previous step's logits, then the L layers of the
           stack in one call, captured once and replayed as a graph (graph = True) or called from Python (graph = False)
  layer    one layer's sparse decode call, as a model calls it whose next layer waits for this one
  prefill  dense prefill of one layer with the statistics and the pool, and the percentile base threshold
  cett     the error-bounded base-threshold search of one layer over its validation tokens
  static   a prefix-static mask (top-k of a prefix score) and the decode call over its list

Shapes, densities and distributions follow the configurations in synth.py and the sweeps of bench.py: weights N(0, std), hidden
states N(0, 1) (a batch's tokens share the fraction `shared` of their variance), Zipf logits with noise, thresholds at the quantile
`rho` of the layer's own activation magnitudes.  A threshold is put in the middle of a gap between two magnitudes, so that rounding
does not decide which neurons are kept.
"""
import math

import torch

import paper_2502_19078_amd as clada

_KIND = {"swiglu": 0, "relu": 1, "geglu": 2}
_DT = {"f32": torch.float32, "bf16": torch.bfloat16}
INF = float("inf")


def listed():
    bf = {"dtype": "bf16", "ffn": "swiglu", "std": 0.02}
    return [
        # a decode step of a small non-gated model: 24 layers of 8 MB, where launches weigh more than bytes
        dict(name="step_opt350m_b1", kind="step", L=24, d=1024, F=4096, B=1, V=50272, rho=0.70, shared=0.0, graph=True,
             dtype="bf16", ffn="relu", std=0.02),
        # the headline workload: 7B stack at batch 1, at its target sparsity
        dict(name="step_7b_b1", kind="step", L=32, d=4096, F=11008, B=1, V=32000, rho=0.45, shared=0.0, graph=True, **bf),
        # a 7B stack serving eight unrelated sequences: the union of the masks is nearly every neuron
        dict(name="step_mistral_b8", kind="step", L=32, d=4096, F=14336, B=8, V=32000, rho=0.45, shared=0.0, graph=True, **bf),
        # one fp32 layer of the toy configuration: the smallest call, launch latency only
        dict(name="layer_toy_f32_b1", kind="layer", d=512, F=1376, B=1, rho=0.40, shared=0.0, dtype="f32", ffn="swiglu",
             std=512 ** -0.5),
        # one layer of an 8B model at batch 1, called alone
        dict(name="layer_8b_b1", kind="layer", d=4096, F=14336, B=1, rho=0.45, shared=0.0, **bf),
        # one layer of a 13B model, sixteen sequences whose masks largely agree
        dict(name="layer_13b_b16", kind="layer", d=5120, F=13824, B=16, rho=0.50, shared=0.9, **bf),
        # a 7B layer kept in fp32 at a small batch
        dict(name="layer_7b_f32_b4", kind="layer", d=4096, F=11008, B=4, rho=0.45, shared=0.0, dtype="f32", ffn="swiglu", std=0.02),
        # prefill of a prompt of odd length, non-gated family
        dict(name="prefill_opt27_t333", kind="prefill", T=333, d=2560, F=10240, q=0.70, dtype="bf16", ffn="relu", std=0.02),
        # prefill and base threshold of the headline workload's prefix
        dict(name="prefill_7b_t512", kind="prefill", T=512, d=4096, F=11008, q=0.45, **bf),
        # the longest prefix of the configurations
        dict(name="prefill_8b_t4096", kind="prefill", T=4096, d=4096, F=14336, q=0.45, **bf),
        # offline calibration by the error bound
        dict(name="cett_7b_t512", kind="cett", T=512, d=4096, F=11008, bound=0.2, **bf),
        # prefix-static mask and decode over its list
        dict(name="static_7b_b1", kind="static", d=4096, F=11008, B=1, rho=0.45, shared=0.0, **bf),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _cost(case):
    w = work(case)
    return max(w["bytes"], w["flops"] / 50)


_LARGEST = None


def draw(rng):
    """One more case of the same ranges; widths and neuron counts away from the named models' among them."""
    global _LARGEST
    if _LARGEST is None:
        _LARGEST = max(_cost(c) for c in listed())
    while True:
        kind = rng.choice(["step", "step", "layer", "layer", "prefill", "prefill", "cett", "static"])
        ffn = rng.choice(["swiglu", "swiglu", "relu", "geglu"])
        dtype = "f32" if rng.random() < 0.2 else "bf16"
        d = rng.choice([512, 768, 1024, 1536, 2048, 2560, 3072, 3584, 4096, 4096, 5120, 5120, 6144, 8192])
        if dtype == "f32":
            d = min(d, 4096)
        F = _log_int(rng, 2 * d, 4 * d)
        F -= F % rng.choice([1, 2, 16, 128])
        c = dict(kind=kind, d=d, F=F, dtype=dtype, ffn=ffn, std=0.02)
        # a ReLU drops half of the neurons by itself: a threshold starts to matter above that
        rho = round(rng.uniform(0.60, 0.85) if ffn == "relu" else rng.uniform(0.30, 0.70), 2)
        shared = rng.choice([0.0, 0.5, 0.9, 1.0])
        if kind == "step":
            c.update(L=rng.randint(4, 40), B=rng.choice([1, 1, 1, 2, 4, 8, 13, 16, 24, 32]), V=_log_int(rng, 1000, 256000), rho=rho,
                     shared=shared, graph=rng.random() < 0.7)
            if dtype == "f32":
                c.update(B=min(c["B"], 4), L=min(c["L"], 8))
        elif kind == "layer":
            c.update(B=min(_log_int(rng, 1, 64), 16 if dtype == "f32" else 64), rho=rho, shared=shared)
        elif kind == "prefill":
            c.update(T=_log_int(rng, 16, 512 if dtype == "f32" else 4096), q=rho)
        elif kind == "cett":
            c.update(T=_log_int(rng, 64, 256 if dtype == "f32" else 1024), bound=round(rng.uniform(0.05, 0.3), 3))
            if ffn == "relu":
                c["ffn"] = "swiglu"
        else:
            c.update(B=rng.choice([1, 1, 4, 8, 16]), rho=rho, shared=shared)
        if _cost(c) <= (0.1 if kind == "cett" else 0.8) * _LARGEST:       # a search projects its tokens many times
            return c


# ------------------------------------------------------------------------------------------------ inputs
def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(seed)


def _normal(g, shape, std, dtype):
    return torch.randn(shape, generator=g, device="cuda", dtype=torch.float32).mul_(std).to(dtype)


def _layer(case, g):
    dt, F, d = _DT[case["dtype"]], case["F"], case["d"]
    relu = case["ffn"] == "relu"
    w = [_normal(g, (F, d), case["std"], dt) for _ in range(2 if relu else 3)]
    if relu:
        return clada.Layer(w[0], None, w[1], kind=1, b_in=_normal(g, F, case["std"], torch.float32),
                           b_out=_normal(g, d, case["std"], torch.float32))
    return clada.Layer(*w, kind=_KIND[case["ffn"]])


def _hidden(case, g, B):
    """[B][d], the tokens sharing the fraction `shared` of their variance."""
    own = _normal(g, (B, case["d"]), 1.0, torch.float32)
    c = case["shared"]
    if c > 0.0:
        own = math.sqrt(c) * _normal(g, (1, case["d"]), 1.0, torch.float32) + math.sqrt(1.0 - c) * own
    return own.to(_DT[case["dtype"]])


def _sigma(g, ffn):
    if ffn == "relu":
        return torch.clamp_min(g, 0.0)
    if ffn == "geglu":
        return 0.5 * g * (1.0 + torch.tanh(math.sqrt(2.0 / math.pi) * (g + 0.044715 * g ** 3)))
    return g * torch.sigmoid(g)


def _act(case, layer, x, dtype):
    g = x.to(dtype) @ layer.w_gate.to(dtype).t()
    if case["ffn"] == "relu":
        g = g + layer.b_in.to(dtype)
    return _sigma(g, case["ffn"])


def _thresholds(case, layer, x):
    """One threshold for the tokens x: the quantile rho of their magnitudes, moved into the widest gap near it."""
    m = _act(case, layer, x, torch.float64 if case["dtype"] == "f32" else torch.float32).abs().flatten().double().sort().values
    k = int(case["rho"] * m.numel())
    lo = max(0, k - 32)
    w = m[lo:k + 32]
    i = torch.argmax(w[1:] - w[:-1])
    return ((w[i] + w[i + 1]) * 0.5).float().reshape(1)


def _logits(g, B, V):
    """Zipf(1.1) over a permuted vocabulary plus unit noise, and token ids drawn from it."""
    prior = -1.1 * torch.log(torch.arange(1, V + 1, device="cuda", dtype=torch.float32))
    z = prior[torch.randperm(V, generator=g, device="cuda")] + torch.randn((B, V), generator=g, device="cuda")
    u = torch.rand((B, V), generator=g, device="cuda").clamp_(1e-20, 1.0 - 1e-7)
    return z.contiguous(), torch.argmax(z - torch.log(-torch.log(u)), dim=-1).to(torch.int32)


def prepare(case, seed):
    g = _gen(seed)
    k = case["kind"]
    d, F, B = case["d"], case["F"], case.get("B", 0)
    V, T = case.get("V", 0), case.get("T", 0)
    ctx = clada.Context(torch.cuda.current_device(), clada.workspace_bytes(d, F, B, T, V))
    s = {"case": case, "ctx": ctx}
    if k in ("prefill", "cett"):
        s["layer"] = _layer(case, g)
        s["x"] = _normal(g, (T, d), 1.0, _DT[case["dtype"]])
        return s
    if k == "step":
        L = case["L"]
        s["layers"] = [_layer(case, g) for _ in range(L)]
        s["arr"] = clada.layer_array(s["layers"])
        s["x"] = torch.stack([_hidden(case, g, B) for _ in range(L)])
        s["base"] = torch.cat([_thresholds(case, l, x) for l, x in zip(s["layers"], s["x"])])
        s["z"], s["tok"] = _logits(g, B, V)
        s["lam"], s["gam"] = (torch.full((L,), v, device="cuda") for v in (0.80, 0.12))
        s["tau"] = torch.empty(L, B, device="cuda")
        s["y"] = torch.empty_like(s["x"])
        if case["graph"]:
            side = torch.cuda.Stream()
            side.wait_stream(torch.cuda.current_stream())
            with torch.cuda.stream(side):
                _step(s)
                side.synchronize()
                clada.graph_begin(ctx)
                s["signals"] = _step(s)
                s["graph"] = clada.graph_end(ctx)
            torch.cuda.current_stream().wait_stream(side)
        return s
    s["layer"] = _layer(case, g)
    s["x"] = _hidden(case, g, B)
    if k == "layer":
        s["tau"] = _thresholds(case, s["layer"], s["x"]).expand(B).contiguous()
    else:
        s["score"] = torch.rand(F, generator=g, device="cuda") * _normal(g, F, 1.0, torch.float32).abs()
        s["k"] = max(1, int(round((1.0 - case["rho"]) * F)))
    return s


def _step(s):
    sur, ent, _ = clada.signals_threshold(s["ctx"], s["z"], s["tok"], s["base"], s["lam"], s["gam"], INF, INF, out=s["tau"])
    clada.sparse_ffn_stack_decode(s["ctx"], s["layers"], s["x"], s["tau"], y=s["y"], c_layers=s["arr"])
    return sur, ent


def run(state):
    case, ctx = state["case"], state["ctx"]
    k = case["kind"]
    if k == "step":
        if case["graph"]:
            state["graph"].launch()
            sur, ent = state["signals"]
        else:
            sur, ent = _step(state)
        return {"surprisal": sur, "entropy": ent, "tau": state["tau"], "y": state["y"]}
    if k == "layer":
        return {"y": clada.sparse_ffn_decode(ctx, state["layer"], state["x"], state["tau"])}
    if k == "prefill":
        st = clada.prefix_stats(ctx, state["layer"], state["x"])
        tau = clada.threshold_calibrate(ctx, st.abs_act_pool, case["q"])
        return {"sum_abs_act": st.sum_abs_act, "sum_sq_act": st.sum_sq_act, "max_abs_act": st.max_abs_act, "sum_sq_h": st.sum_sq_h,
                "A": st.A, "pool": st.abs_act_pool, "y": st.y, "tau": tau}
    if k == "cett":
        tau, mean = clada.threshold_search_cett(ctx, state["layer"], state["x"], case["bound"])
        return {"tau": tau, "mean": mean}
    idx, n = clada.static_mask_topk(ctx, state["score"], state["k"])
    y = clada.static_ffn_decode(ctx, state["layer"], state["x"], idx, n)
    return {"idx": idx[:state["k"]], "n": n, "y": y}        # entries past the count are not written


# ------------------------------------------------------------------------------------- what a pass cannot do without
def _union(case):
    """Share of a layer's neurons that at least one token keeps, from the distributions the inputs are drawn from."""
    n = 2048
    q = (torch.arange(n, dtype=torch.float64) + 0.5) / n
    z = math.sqrt(2.0) * torch.erfinv(2.0 * q - 1.0)
    s = case["std"] * math.sqrt(case["d"])
    if case["ffn"] == "relu":
        s = math.hypot(s, case["std"])
    tau = torch.quantile(_sigma(s * z, case["ffn"]).abs(), case["rho"])
    c, B = case["shared"], case["B"]
    if B == 1 or c >= 1.0:
        return 1.0 - case["rho"]
    common = z[4::8][:, None] * math.sqrt(c) + z[None, :] * math.sqrt(1.0 - c)
    keep = (_sigma(s * common, case["ffn"]).abs() >= tau).double().mean(dim=1)
    return float((1.0 - (1.0 - keep) ** B).mean())


def work(case):
    e = 4 if case["dtype"] == "f32" else 2
    d, F, k = case["d"], case["F"], case["kind"]
    relu = case["ffn"] == "relu"
    m = 2 if relu else 3
    if k in ("prefill", "cett"):
        T = case["T"]
        if k == "prefill":
            return {"bytes": m * F * d * e + 2 * T * d * e + 4 * T * F + 20 * F, "flops": 2 * m * T * d * F}
        # the projections once and the result: what the search itself costs is the implementation's
        return {"bytes": m * F * d * e + T * d * e, "flops": 2 * m * T * d * F}
    B = case["B"]
    if k == "static":
        n = max(1, int(round((1.0 - case["rho"]) * F)))
        return {"bytes": m * n * d * e + 2 * B * d * e + 4 * F, "flops": 2 * m * n * d * B}
    u, own = _union(case), 1.0 - case["rho"]
    w = {"bytes": (1 + (m - 1) * u) * F * d * e + 2 * B * d * e, "flops": 2 * B * (1 + (m - 1) * own) * F * d}
    if k == "step":
        w = {a: case["L"] * v for a, v in w.items()}
        w["bytes"] += 4 * B * case["V"]
        w["flops"] += 5 * B * case["V"]
    return w


# ------------------------------------------------------------------------------------------------ correctness
def tolerance(case):
    """Four times what the present outputs differ from the 64-bit ones, or more where the type's own rounding asks for it: bf16
    outputs are rounded once (2^-9 of a value) and a prefill's or search's h once more; fp32 sums over d and d_ff terms."""
    if case["dtype"] == "f32":
        return {"rel": 1e-5, "max": 2e-4}
    if case["kind"] == "cett":
        return {"rel": 1e-3, "max": 1e-3}
    return {"rel": 8e-3, "max": 4e-2}


def _ffn64(case, layer, x, keep=None):
    """(magnitudes, h, y) in 64 bits; keep(a) -> mask of the neurons that count."""
    a = _act(case, layer, x, torch.float64)
    h = a if case["ffn"] == "relu" else a * (x.double() @ layer.w_up.double().t())
    hk = h if keep is None else torch.where(keep(a), h, torch.zeros_like(h))
    y = hk @ layer.w_down.double()
    if layer.b_out is not None:
        y = y + layer.b_out.double()
    return a.abs(), h, y


def _exact_cett(case, layer, x):
    """Bisection over the bit patterns of the non-negative floats with the definition of the mean in 64 bits."""
    a, h, y = _ffn64(case, layer, x)
    a = a.float()
    w = layer.w_down.double()
    dense = y.norm(dim=1)

    def mean(eps):
        cut = (torch.where(a < eps, h, torch.zeros_like(h)) @ w).norm(dim=1)
        return float(torch.where(dense > 0, cut / dense, torch.zeros_like(dense)).mean())

    lo, hi, best = 0, 0x7F800000, 0.0
    while hi - lo > 1:
        mid = (lo + hi) // 2
        eps = torch.tensor([mid], dtype=torch.int32).view(torch.float32).item()
        got = mean(eps)
        if got <= case["bound"]:
            lo, best = mid, got
        else:
            hi = mid
    return {"tau": torch.tensor([lo], dtype=torch.int32).view(torch.float32), "mean": torch.tensor([best], dtype=torch.float64)}


def exact(case, seed):
    s = prepare(dict(case, graph=False) if case["kind"] == "step" else case, seed)
    k = case["kind"]
    if k == "step":
        lp = torch.log_softmax(s["z"].double(), dim=-1)
        sur = -lp.gather(1, s["tok"].long()[:, None])[:, 0]
        ent = -(lp.exp() * lp).sum(dim=-1)
        tau = s["base"][:, None].expand(case["L"], case["B"])
        y = torch.stack([_ffn64(case, l, x, lambda a: a.abs() >= t.double()[:, None])[2]
                         for l, x, t in zip(s["layers"], s["x"], tau)])
        return {"surprisal": sur, "entropy": ent, "tau": tau.double(), "y": y}
    if k == "layer":
        return {"y": _ffn64(case, s["layer"], s["x"], lambda a: a.abs() >= s["tau"].double()[:, None])[2]}
    if k == "prefill":
        a, h, y = _ffn64(case, s["layer"], s["x"])
        sq = (h * h).sum(dim=0)
        n = a.numel()
        rank = max(1, math.ceil(float(torch.tensor(case["q"], dtype=torch.float32)) * n))
        return {"sum_abs_act": a.sum(dim=0), "sum_sq_act": (a * a).sum(dim=0), "max_abs_act": a.amax(dim=0), "sum_sq_h": sq,
                "A": sq.sqrt() * s["layer"].w_down.double().norm(dim=1), "pool": a, "y": y,
                "tau": a.flatten().sort().values[rank - 1:rank]}
    if k == "cett":
        return _exact_cett(case, s["layer"], s["x"])
    best = torch.topk(s["score"].double(), s["k"]).indices.sort().values
    layer, x = s["layer"], s["x"]
    mask = torch.zeros(case["F"], dtype=torch.bool, device="cuda")
    mask[best] = True
    y = _ffn64(case, layer, x, lambda a: mask.expand_as(a))[2]
    return {"idx": best.to(torch.int32), "n": torch.tensor([s["k"]], dtype=torch.int32), "y": y}
