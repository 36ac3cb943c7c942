"""GPU parity: clada_prefix_stats (MFMA prefill + fused aggregates) and the calibration chain."""
import numpy as np
import pytest
import torch

import oracle
import synth
from gpu_util import DEV, TOL_Y, assert_close_y, least_workspace, nan_workspace, to_dev, to_np

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def clada():
    import paper_2502_19078_amd as m
    m.load_library()
    return m


def _rel(a, b):
    return np.linalg.norm(np.asarray(a, np.float64) - b) / max(np.linalg.norm(b), 1e-300)


@pytest.mark.parametrize("cfg_name,d,F,T", [
    ("c1", 512, 1376, 64),       # config 1 as written (fp32 MFMA)
    ("c1", 96, 200, 130),        # ragged in every dimension, K not a multiple of the 32-wide k-tile
    ("c1", 8, 5, 1),             # degenerate: one token, one k-chunk
    ("c2", 1024, 1000, 300),     # bf16 MFMA, ragged tiles
    ("c2", 4096, 384, 512),      # bf16, real K and prefix length of config 2, three neuron tiles
    ("c2", 72, 129, 257),
    ("c2", 64, 200, 300),        # two 32-deep k-tiles: shorter than the 256-token kernel's pipeline
    ("c2", 128, 100, 257),       # four k-tiles: exactly the four LDS stages, no steady-state iteration
    ("c2", 192, 129, 513),       # six k-tiles; the last 256-token tile holds one token
    ("c2", 320, 64, 129),        # ten k-tiles; second half of the only 256-token tile holds one token
    ("c2", 512, 700, 1024),      # 8 token tiles: the blocked tile order, 6 neuron tiles padded to 8
    ("c2", 256, 384, 2000),      # 16 token tiles (last one ragged), 3 neuron tiles
    ("c2", 64, 40, 1),           # bf16, one token: every row of a tile repeats it
    ("c2", 512, 32, 300),        # a single 32-deep k-tile in the 256 x 256 down projection
    ("c2", 768, 96, 520),        # three column tiles, three k-tiles
    ("c2", 512, 1024, 300),      # few tiles, long d_ff: the down projection splits d_ff four ways
    ("c2", 256, 800, 130),       # split three ways, 25 k-tiles (uneven parts)
])
@pytest.mark.parametrize("tile", [1, 2])
def test_prefix_stats_parity(clada, cfg_name, d, F, T, tile):
    """tile = workgroup tile of the bf16 gate/up GEMM (128 or 256 tokens); fp32 layers have one kernel."""
    cfg = synth.CONFIGS[cfg_name]
    if tile == 2 and cfg.dtype != "bf16":
        pytest.skip("the 256-token tile is a bf16 kernel")
    w = synth.layer_weights(cfg, 0, 1, d=d, d_ff=F)
    X = synth.prefix_hidden(cfg, 0, 1, T=T, d=d)
    ctx = clada.Context(0, clada.workspace_bytes(d, F, 0, T, 0))
    ctx.set_option("prefix.tile", tile)
    layer = clada.Layer(*[to_dev(a, cfg.dtype) for a in w])
    st = clada.prefix_stats(ctx, layer, to_dev(X, cfg.dtype))
    torch.cuda.synchronize()
    ref = oracle.prefix_stats(*w, X)
    tol = 1e-5
    # statistics come from fp32 accumulators of exact products in both dtypes
    assert _rel(to_np(st.abs_act_pool), ref["abs_act_pool"]) < tol
    np.testing.assert_allclose(to_np(st.abs_act_pool), ref["abs_act_pool"], rtol=1e-4, atol=1e-6)
    for name in ("sum_abs_act", "sum_sq_act", "max_abs_act", "sum_sq_h", "A"):
        got = to_np(getattr(st, name))
        np.testing.assert_allclose(got, ref[name], rtol=2e-5, atol=1e-7, err_msg=name)
    assert_close_y(to_np(st.y), ref["y"], TOL_Y[cfg.dtype], "prefill y")
    # A_j for T=1 reduces to |h_j| * ||W_down[j]||
    # calibration chain: the GPU quantile of the GPU pool is an exact order statistic of that pool
    tau = clada.threshold_calibrate(ctx, st.abs_act_pool, cfg.q)
    torch.cuda.synchronize()
    assert float(tau.item()) == oracle.calibrate(to_np(st.abs_act_pool), cfg.q)
    assert float(tau.item()) == pytest.approx(oracle.calibrate(ref["abs_act_pool"], cfg.q), rel=1e-4)


def test_prefix_stats_without_optional_outputs(clada):
    cfg = synth.CONFIGS["c2"]
    d, F, T = 256, 300, 100
    w = synth.layer_weights(cfg, 1, 0, d=d, d_ff=F)
    X = synth.prefix_hidden(cfg, 1, 0, T=T, d=d)
    ctx = clada.Context(0, clada.workspace_bytes(d, F, 0, T, 0))
    layer = clada.Layer(*[to_dev(a, cfg.dtype) for a in w])
    st = clada.prefix_stats(ctx, layer, to_dev(X, cfg.dtype), want_y=False, want_pool=False)
    torch.cuda.synchronize()
    ref = oracle.prefix_stats(*w, X, want_y=False)
    assert st.y is None and st.abs_act_pool is None
    np.testing.assert_allclose(to_np(st.A), ref["A"], rtol=2e-5, atol=1e-7)


def test_calibrated_threshold_gives_target_decode_sparsity(clada):
    """Prefill -> calibrate -> decode on fresh tokens: measured sparsity is near the target."""
    cfg = synth.CONFIGS["c2"]
    d, F, T = 1024, 2752, 512
    w = synth.layer_weights(cfg, 2, 0, d=d, d_ff=F)
    X = synth.prefix_hidden(cfg, 2, 0, T=T, d=d)
    ctx = clada.Context(0, clada.workspace_bytes(d, F, 8, T, 0))
    layer = clada.Layer(*[to_dev(a, cfg.dtype) for a in w])
    st = clada.prefix_stats(ctx, layer, to_dev(X, cfg.dtype), want_y=False)
    tau = clada.threshold_calibrate(ctx, st.abs_act_pool, cfg.q)
    x = synth.decode_hidden(cfg, 2, 0, 0, B=8, d=d)
    y, idx, cnt, bits = clada.sparse_ffn_decode(ctx, layer, to_dev(x, cfg.dtype), tau.expand(8).contiguous(),
                                                want_lists=True)
    torch.cuda.synchronize()
    rho = 1.0 - cnt[1:].float().mean().item() / F
    assert abs(rho - cfg.q) < 0.03


@pytest.mark.parametrize("cfg_name,layer_id", [("c4", 3), ("c2", 7)])
def test_prefix_stats_full_size_layers_sampled(clada, cfg_name, layer_id):
    """One full-size layer with the configuration's own prefix length (LLaMA-3-8B shape with 4096
    tokens, LLaMA2-7B shape with 512), in the launch the benchmark times.  The oracle is too slow
    for the whole prefill, so it checks what it can compute piece by piece: per-neuron aggregates
    and pool columns of sampled neurons (each neuron's statistics depend on its own three weight
    rows only), and the output rows of sampled tokens (the prefill output of a token is its dense
    decode)."""
    cfg = synth.CONFIGS[cfg_name]
    d, F, T = cfg.d, cfg.d_ff, cfg.T
    w = synth.layer_weights(cfg, 0, layer_id)
    X = synth.prefix_hidden(cfg, 0, layer_id)
    assert X.shape == (T, d)
    ctx = clada.Context(0, clada.workspace_bytes(d, F, 0, T, 0))
    layer = clada.Layer(*[to_dev(a, cfg.dtype) for a in w])
    st = clada.prefix_stats(ctx, layer, to_dev(X, cfg.dtype))
    torch.cuda.synchronize()
    rng = np.random.default_rng(11)
    # neurons at tile borders of both kernels' tilings plus random ones
    S = np.unique(np.concatenate([[0, 31, 32, 63, 64, 127, 128, F - 129, F - 128, F - 1],
                                  rng.integers(0, F, 54)])).astype(np.int64)
    ref = oracle.prefix_stats(w[0][S], w[1][S], w[2][S], X, want_y=False)
    pool = to_np(st.abs_act_pool[:, torch.from_numpy(S).to(DEV)])
    np.testing.assert_allclose(pool, ref["abs_act_pool"], rtol=1e-4, atol=1e-6)
    for name in ("sum_abs_act", "sum_sq_act", "max_abs_act", "sum_sq_h", "A"):
        np.testing.assert_allclose(to_np(getattr(st, name))[S], ref[name], rtol=2e-5, atol=1e-7, err_msg=name)
    toks = np.unique(np.concatenate([[0, 127, 128, 255, 256, T - 1], rng.integers(0, T, 4)]))
    y = to_np(st.y)
    for t in toks:
        assert_close_y(y[t:t + 1], oracle.dense_decode(*w, X[t:t + 1]), TOL_Y[cfg.dtype], f"prefill y, token {t}")


@pytest.mark.parametrize("n,kind", [
    (1, "normal"), (3, "normal"), (5, "normal"), (16384 * 4 + 7, "normal"), (3_000_001, "normal"),
    (13_000_003, "equal"),       # one value: the second pass has to add its 16-bit counts up on the way
    (700_000, "zeros"),          # half of the pool exactly zero, as a ReLU leaves it
    (1000, "inf"), (200_000, "tiny"), (70_000, "two"),
])
def test_calibrate_is_the_nearest_rank_quantile_bit_for_bit(clada, n, kind):
    """Against a sort of the same values, ranks at both ends and inside; two calls on one context in a row (the
    histograms have to be clear again), and replays of a captured call."""
    g = torch.Generator(device=DEV).manual_seed(n)
    v = torch.randn(n, generator=g, device=DEV).abs()
    if kind == "equal":
        v.fill_(0.25)
    elif kind == "zeros":
        v = torch.clamp_min(v - 0.67, 0.0)
    elif kind == "inf":
        v[::7] = float("inf")
    elif kind == "tiny":
        v *= 1e-42                                           # subnormal magnitudes: many ties
    elif kind == "two":
        v = torch.where(v > 0.5, torch.tensor(1.0, device=DEV), torch.nextafter(torch.tensor(1.0, device=DEV), torch.tensor(2.0, device=DEV)))
    ref = v.sort().values
    ctx = clada.Context(0, clada.workspace_bytes(64, 64, 0, 1, 0))
    for q in (0.0, 1.0 / 3.0, 0.45, 0.5, 0.9, 0.9999999):
        k = max(1, int(np.ceil(np.float64(np.float32(q)) * n)))
        for _ in range(2):
            got = clada.threshold_calibrate(ctx, v, q)
            assert torch.equal(got, ref[k - 1:k]), (n, kind, q, float(got), float(ref[k - 1]))
    out, side = torch.zeros(1, device=DEV), torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        clada.graph_begin(ctx)
        clada.threshold_calibrate(ctx, v, 0.45, out=out)
        gr = clada.graph_end(ctx)
        want = ref[max(1, int(np.ceil(np.float64(np.float32(0.45)) * n))) - 1]
        for _ in range(3):
            out.zero_()
            gr.launch()
            side.synchronize()
            assert out[0] == want
            clada.threshold_calibrate(ctx, v, 0.7)
            side.synchronize()


@pytest.mark.parametrize("d,F,T,relu,tile", [
    (64, 129, 129, True, 0),     # 128-token tiles of the non-gated family: one operand, a ragged second tile
    (128, 4000, 300, True, 1), (320, 700, 1030, True, 1),      # 8 and 9 token tiles: both tile orders
    (64, 128 * 86, 384, False, 0), (64, 128 * 85, 384, False, 0),      # 258 and 255 tiles: either side of one round
    (128, 300, 70, False, 0),    # spare workgroups many times the tiles
])
def test_prefill_tiles_of_short_prefixes_and_norms_on_spare_units(clada, d, F, T, relu, tile):
    """Every output against a float64 reference; A_j through the norms that idle compute units formed."""
    from paper_2502_19078_amd import binding
    g = torch.Generator(device=DEV).manual_seed(d + F + T)
    n = lambda *s, k: (torch.randn(s, generator=g, device=DEV) * k)
    w = [n(F, d, k=d ** -0.5).bfloat16() for _ in range(2 if relu else 3)]
    x = n(T, d, k=1.0).bfloat16()
    b_in, b_out = n(F, k=0.1), n(d, k=0.1)
    layer = clada.Layer(w[0], None, w[1], kind=binding.RELU, b_in=b_in, b_out=b_out) if relu else clada.Layer(*w)
    ctx = clada.Context(0, clada.workspace_bytes(d, F, 0, T, 0))
    ctx.set_option("prefix.tile", tile)
    got = clada.prefix_stats(ctx, layer, x)
    xd, w = x.double().cpu(), [a.double().cpu() for a in w]
    pre = xd @ w[0].t()
    a = torch.relu(pre + b_in.double().cpu()) if relu else pre * torch.sigmoid(pre)
    h = a if relu else a * (xd @ w[1].t())
    sq = (h * h).sum(0)
    want = {"sum_abs_act": a.abs().sum(0), "sum_sq_act": (a * a).sum(0), "max_abs_act": a.abs().amax(0), "sum_sq_h": sq,
            "A": sq.sqrt() * w[-1].norm(dim=1), "abs_act_pool": a.abs()}
    for k, v in want.items():                                # fp32 accumulation over d and T terms, a hardware exp2 of a few ulp
        assert _rel(to_np(getattr(got, k)), v.numpy()) < 2e-5, k
    y = h @ w[-1] + (b_out.double().cpu() if relu else 0.0)
    assert _rel(to_np(got.y), y.numpy()) < 5e-3              # h and y each rounded once to bf16: 2^-9 of a value


@pytest.mark.parametrize("d,F,T,kind,tile", [
    (64, 4100, 2050, "swiglu", 0),      # one k-tile a tile, more tiles than compute units: the transfers run tiles ahead
    (256, 4100, 2050, "geglu", 2), (192, 8300, 2500, "relu", 0),       # 297 and 330 tiles, ragged both ways
    (1024, 2905, 1300, "swiglu", 0),    # tiles of 96 neurons
    (256, 130, 64, "swiglu", 0), (512, 6401, 127, "geglu", 0),         # tiles of 64 neurons; d_ff off every multiple
    (256, 4097, 100, "relu", 0), (256, 16300, 129, "swiglu", 0), (256, 16500, 129, "swiglu", 0),
    (8192, 70, 2300, "swiglu", 0),      # 288 tiles of the down projection, not split
    (2048, 1000, 65, "relu", 0), (256, 63, 257, "swiglu", 2),
])
def test_pipelined_prefill_tiles(clada, d, F, T, kind, tile):
    """Every output against a float64 reference, and the same bits from a second call; d_ff is no multiple of the k-tile of the down
    projection, whose last rows of W_down do not exist."""
    from paper_2502_19078_amd import binding
    g = torch.Generator(device=DEV).manual_seed(d + F + T)
    n = lambda *s, k: (torch.randn(s, generator=g, device=DEV) * k)
    relu = kind == "relu"
    w = [n(F, d, k=d ** -0.5).bfloat16() for _ in range(2 if relu else 3)]
    x = n(T, d, k=1.0).bfloat16()
    b_in, b_out = n(F, k=0.1), n(d, k=0.1)
    layer = (clada.Layer(w[0], None, w[1], kind=binding.RELU, b_in=b_in, b_out=b_out) if relu
             else clada.Layer(*w, kind=binding.GEGLU if kind == "geglu" else binding.SWIGLU))
    ctx = clada.Context(0, clada.workspace_bytes(d, F, 0, T, 0))
    ctx.set_option("prefix.tile", tile)
    got, again = clada.prefix_stats(ctx, layer, x), clada.prefix_stats(ctx, layer, x)
    xd, wd = x.double(), [a.double() for a in w]
    pre = xd @ wd[0].t()
    if relu:
        h = a = torch.relu(pre + b_in.double())
    else:
        a = torch.nn.functional.gelu(pre, approximate="tanh") if kind == "geglu" else torch.nn.functional.silu(pre)
        h = a * (xd @ wd[1].t())
    sq = (h * h).sum(0)
    want = {"sum_abs_act": a.abs().sum(0), "sum_sq_act": (a * a).sum(0), "max_abs_act": a.abs().amax(0), "sum_sq_h": sq,
            "A": sq.sqrt() * wd[-1].norm(dim=1), "abs_act_pool": a.abs()}
    for k, v in want.items():                                # fp32 accumulation over d and T terms, a hardware exp2 of a few ulp
        assert _rel(to_np(getattr(got, k)), v.cpu().numpy()) < 2e-5, k
        assert torch.equal(getattr(got, k), getattr(again, k)), k
    y = h @ wd[-1] + (b_out.double() if relu else 0.0)
    assert _rel(to_np(got.y), y.cpu().numpy()) < 5e-3        # h and y each rounded once to bf16: 2^-9 of a value
    assert torch.equal(got.y, again.y)


def test_rows_past_d_ff_do_not_reach_the_output(clada):
    """An infinite last row of W_down: the k-tile's rows past d_ff are zeros, not that row again (0 * inf would be a NaN)."""
    d, F, T = 256, 70, 40
    g = torch.Generator(device=DEV).manual_seed(1)
    w = [(torch.randn(F, d, generator=g, device=DEV) * 0.06).bfloat16() for _ in range(3)]
    w[2][-1] = float("inf")
    x = torch.randn(T, d, generator=g, device=DEV).bfloat16()
    y = clada.prefix_stats(clada.Context(0, clada.workspace_bytes(d, F, 0, T, 0)), clada.Layer(*w), x).y
    g64, u64 = x.double() @ w[0].double().t(), x.double() @ w[1].double().t()
    h = (torch.nn.functional.silu(g64) * u64)[:, -1:]
    assert torch.equal(y.double(), h.sign().expand(T, d) * float("inf"))


@pytest.mark.parametrize("d,F,T,dtype,kind", [
    (512, 700, 33, "f32", "swiglu"), (260, 513, 64, "f32", "geglu"), (1024, 3001, 65, "f32", "relu"),      # 64- and 128-token tiles
    (132, 4099, 20, "f32", "swiglu"),   # 16 parts asked for, 12 taken; columns past d in the last tile
    (2048, 1111, 300, "f32", "relu"),   # four parts, output biases
    (72, 129, 60, "bf16", "swiglu"), (200, 65, 130, "bf16", "relu"),       # bf16 rows off the pipelined tiles
])
def test_plain_prefill_tiles_and_the_fp32_split(clada, d, F, T, dtype, kind):
    """Against a float64 reference, the same bits from a second call, and the same to rounding in a workspace without room for a split."""
    from paper_2502_19078_amd import binding
    g = torch.Generator(device=DEV).manual_seed(d + F + T)
    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    n = lambda *s, k: (torch.randn(s, generator=g, device=DEV) * k)
    relu = kind == "relu"
    w = [n(F, d, k=d ** -0.5).to(dt) for _ in range(2 if relu else 3)]
    x = n(T, d, k=1.0).to(dt)
    b_in, b_out = n(F, k=0.1), n(d, k=0.1)
    layer = (clada.Layer(w[0], None, w[1], kind=binding.RELU, b_in=b_in, b_out=b_out) if relu
             else clada.Layer(*w, kind=binding.GEGLU if kind == "geglu" else binding.SWIGLU))
    ctx = clada.Context(0, clada.workspace_bytes(d, F, 0, T, 0))
    got, again = clada.prefix_stats(ctx, layer, x), clada.prefix_stats(ctx, layer, x)
    xd, wd = x.double(), [a.double() for a in w]
    pre = xd @ wd[0].t()
    if relu:
        h = a = torch.relu(pre + b_in.double())
    else:
        a = torch.nn.functional.gelu(pre, approximate="tanh") if kind == "geglu" else torch.nn.functional.silu(pre)
        h = a * (xd @ wd[1].t())
    sq = (h * h).sum(0)
    want = {"sum_abs_act": a.abs().sum(0), "sum_sq_act": (a * a).sum(0), "max_abs_act": a.abs().amax(0), "sum_sq_h": sq,
            "A": sq.sqrt() * wd[-1].norm(dim=1), "abs_act_pool": a.abs()}
    for k, v in want.items():                                # fp32 accumulation over d and T terms, a hardware exp2 of a few ulp
        assert _rel(to_np(getattr(got, k)), v.cpu().numpy()) < 2e-5, k
        assert torch.equal(getattr(got, k), getattr(again, k)), k
    y = (h @ wd[-1] + (b_out.double() if relu else 0.0)).cpu().numpy()
    tol = 1e-5 if dtype == "f32" else 5e-3                   # bf16: h and y each rounded once, 2^-9 of a value
    assert _rel(to_np(got.y), y) < tol and torch.equal(got.y, again.y)
    tight = -(-T // 128) * 16 * F + T * (-(-F // 64) * 64) * 4 + 1024      # partial aggregates and h alone
    assert _rel(to_np(clada.prefix_stats(clada.Context(0, tight), layer, x).y), y) < tol


PADDED = [
    # tiles of 96 neurons that end at, before and behind d_ff rounded up to 64 (d_ff mod 192 = 64, 65, 80, 95, 96, 97), d a multiple of 256 or not
    (768, 64, 257, "swiglu", 2), (768, 257, 512, "geglu", 2), (1024, 272, 700, "swiglu", 2), (576, 95, 333, "swiglu", 2),
    (768, 287, 300, "geglu", 2), (768, 96, 257, "swiglu", 2), (576, 288, 512, "geglu", 2), (832, 289, 333, "swiglu", 2),
    (1024, 2976, 1300, "swiglu", 0), (1024, 2960, 1300, "geglu", 0),
    # 64, 128 and 256 neurons
    (256, 65, 100, "swiglu", 1), (256, 96, 60, "relu", 1), (512, 129, 200, "geglu", 1), (512, 97, 300, "relu", 1), (256, 300, 257, "relu", 2),
    (512, 65, 257, "swiglu", 2),
    # the plain tiles, bf16 and fp32
    (72, 97, 130, "swiglu", 0), (256, 96, 70, "f32", 0), (260, 65, 40, "f32", 0),
]


@pytest.mark.parametrize("d,F,T,kind,tile", PADDED)
def test_h_is_zero_past_d_ff(clada, d, F, T, kind, tile):
    """h is read in columns of 64, against rows of W_down that count as zero: what the workspace held there must not matter, and NaNs do."""
    from paper_2502_19078_amd import binding
    dt = torch.float32 if kind == "f32" else torch.bfloat16
    g = torch.Generator(device=DEV).manual_seed(d + F + T)
    w = [(torch.randn(F, d, generator=g, device=DEV) * d ** -0.5).to(dt) for _ in range(3)]
    x = torch.randn(T, d, generator=g, device=DEV).to(dt)
    layer = (clada.Layer(w[0], None, w[2], kind=binding.RELU) if kind == "relu"
             else clada.Layer(*w, kind=binding.GEGLU if kind == "geglu" else binding.SWIGLU))
    ctx = nan_workspace(clada, d, F, T, dt)
    ctx.set_option("prefix.tile", tile)
    y = clada.prefix_stats(ctx, layer, x).y
    pre = x.double() @ w[0].double().t()
    if kind == "relu":
        h = torch.relu(pre)
    else:
        a = torch.nn.functional.gelu(pre, approximate="tanh") if kind == "geglu" else torch.nn.functional.silu(pre)
        h = a * (x.double() @ w[1].double().t())
    want = (h @ w[2].double()).cpu().numpy()
    assert _rel(to_np(y), want) < (1e-5 if kind == "f32" else 5e-3)      # bf16: h and y each rounded once, 2^-9 of a value


# d, F, T, dtype, kind, tile: bf16 whose smallest workspace has room for 10 of 12 parts, for 3 of 12, for 4 of 8, for all, for one; d_ff below 2 d off
# multiples of 32 (not split); fp32 with room for none (y takes them) and for all
SPLITS = [(1024, 4096, 16, "bf16", "swiglu", 0), (512, 3333, 100, "bf16", "relu", 0), (256, 2085, 40, "bf16", "geglu", 0), (1024, 2720, 300, "bf16", "swiglu", 0),
          (768, 2111, 300, "bf16", "swiglu", 2), (1024, 1919, 64, "bf16", "swiglu", 0), (260, 3001, 40, "f32", "swiglu", 0), (512, 1111, 140, "f32", "relu", 0),
          (512, 4096, 300, "f32", "swiglu", 0)]


def _split_layer(clada, d, F, T, dtype, kind):
    from paper_2502_19078_amd import binding
    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    g = torch.Generator(device=DEV).manual_seed(d + F + T)
    w = [(torch.randn(F, d, generator=g, device=DEV) * d ** -0.5).to(dt) for _ in range(3)]
    layer = (clada.Layer(w[0], None, w[2], kind=binding.RELU, b_out=torch.randn(d, generator=g, device=DEV)) if kind == "relu"
             else clada.Layer(*w, kind=binding.GEGLU if kind == "geglu" else binding.SWIGLU))
    return layer, torch.randn(T, d, generator=g, device=DEV).to(dt)


@pytest.mark.parametrize("d,F,T,dtype,kind,tile", SPLITS)
def test_y_does_not_depend_on_the_room_for_a_split(clada, d, F, T, dtype, kind, tile):
    """The same bits from a context of the advised size, from the smallest one, and from some between and beyond."""
    layer, x = _split_layer(clada, d, F, T, dtype, kind)
    least = least_workspace(clada, lambda c: clada.prefix_stats(c, layer, x))
    advised = clada.workspace_bytes(d, F, 0, T, 0)
    want = None
    for n in (advised, least, least + 4 * T * d, least + 8 * T * d, least + 20 * T * d, advised + 64 * T * d):
        ctx = clada.Context(0, n)
        ctx.set_option("prefix.tile", tile)
        got = clada.prefix_stats(ctx, layer, x)
        if want is None:
            want = got
        for k in ("y", "A", "sum_sq_h"):
            assert torch.equal(getattr(got, k), getattr(want, k)), (k, n - least)
