"""GPU parity: clada_cett_eval and clada_threshold_search_cett (section 3.2.2) against the fp64 oracle."""
import numpy as np
import pytest
import torch

import oracle
import synth
from gpu_util import BAND, DEV, band_width, least_workspace, nan_workspace, to_dev, to_np

pytestmark = pytest.mark.gpu

# Per-token CETT: fp32 layers differ from fp64 by accumulation rounding only; bf16 layers round h
# to bf16 (at most 2^-9 relative per neuron) before both projections, so numerator and denominator
# norms each move by at most 2^-9 relative when the terms do not cancel: 2 * 2^-9 on the ratio
# (reached with a few dozen cut neurons; with thousands the independent roundings average out).
TOL_CETT = {"f32": 2e-5, "bf16": 2 * 2.0 ** -9}
# Search properties judged by the oracle just below / above tau: a few neurons inside that gap may
# fall on either side of the fp64 comparison, each moving one token's CETT by ~1e-3 relative.
TOL_SEARCH = {"f32": 1e-4, "bf16": 2 * 2.0 ** -9}
# tau_base: the device search stops at a boundary of its own feasible set; rounding moves the mean
# by <= TOL_CETT * bound, i.e. a handful of neighbouring pooled magnitudes.
TOL_TAU = {"f32": 1e-4, "bf16": 2e-3}


@pytest.fixture(scope="module")
def clada():
    import paper_2502_19078_amd as m
    m.load_library()
    return m


def _setup(clada, cfg_name, d, F, T, seed=0, layer_id=2, tile=0):
    cfg = synth.CONFIGS[cfg_name]
    w = synth.layer_weights(cfg, seed, layer_id, d=d, d_ff=F)
    X = synth.prefix_hidden(cfg, seed, layer_id, T=T, d=d)
    ctx = clada.Context(0, clada.workspace_bytes(d, F, 0, T, 0))
    ctx.set_option("prefix.tile", tile)
    layer = clada.Layer(*[to_dev(a, cfg.dtype) for a in w])
    return cfg, w, X, ctx, layer, to_dev(X, cfg.dtype)


def _cett_given_cut(w, X, cut):
    """Oracle CETT for a given cut set (bool [T][F]): ||sum of the cut contributions|| / ||dense output||,
    from the oracle's decode functions."""
    y_cut = oracle.decode_given_mask(*w, X, cut)
    dense = oracle.dense_decode(*w, X)
    nd = np.linalg.norm(dense, axis=1)
    return np.where(nd > 0, np.linalg.norm(y_cut, axis=1) / np.where(nd > 0, nd, 1.0), 0.0)


# last entry: option prefix.tile (0 = the library's choice, 2 = the 256-row tiles of both prefill GEMMs)
CASES = [
    ("c1", 512, 1376, 64, 0),    # config 1 as written (fp32)
    ("c1", 96, 200, 130, 0),     # ragged in every dimension
    ("c1", 8, 5, 1, 0),          # one token
    ("c2", 1024, 1000, 300, 0),  # bf16, ragged tiles
    ("c2", 72, 129, 257, 0),
    ("c2", 512, 416, 300, 2),    # 256 x 256 down-projection tiles: 13 k-tiles of 32, d_ff not a multiple of 64
    ("c2", 256, 64, 257, 2),     # two k-tiles; the second token tile holds one token
    ("c2", 256, 768, 257, 0),    # down projection split three ways along d_ff, row norms from the combining pass
]


@pytest.mark.parametrize("cfg_name,d,F,T,tile", CASES)
def test_cett_eval_parity(clada, cfg_name, d, F, T, tile):
    """The device's cut set is read off the device's own |a| pool (the same kernel feeds the masking
    pass), validated against the oracle's inside the band around eps, and the oracle is evaluated on
    that set: a neuron within rounding of eps may fall on either side, everything else is fixed."""
    cfg, w, X, ctx, layer, Xd = _setup(clada, cfg_name, d, F, T, tile=tile)
    a_ref = oracle.prefix_stats(*w, X, want_y=False)["abs_act_pool"]
    pool_ref = np.sort(a_ref.ravel())
    pool_gpu = clada.prefix_stats(ctx, layer, Xd, want_y=False).abs_act_pool.cpu().numpy()
    tol = TOL_CETT[cfg.dtype]
    for q in (0.0, 0.2, 0.45, 0.8):
        eps = float(np.float32(pool_ref[int(q * (len(pool_ref) - 1))] * 1.00037 + 1e-9))
        got, mean = clada.cett_eval(ctx, layer, Xd, eps)
        torch.cuda.synchronize()
        cut_gpu = pool_gpu < np.float32(eps)
        cut_ref = a_ref < eps
        flips = cut_gpu != cut_ref
        # the band of the decode masks (relative to eps, with the absolute floor for a tiny eps: q = 0 gives
        # eps ~ 1e-7, where the fp32 accumulation error of the pre-activation is what decides)
        assert not (flips & (np.abs(a_ref - eps) > band_width(eps))).any(), "cut sets differ outside the band"
        ref = _cett_given_cut(w, X, cut_gpu)
        np.testing.assert_allclose(to_np(got), ref, rtol=tol, atol=1e-6, err_msg=f"q={q}")
        assert float(mean.item()) == pytest.approx(ref.mean(), rel=tol, abs=1e-6)
        if not flips.any():
            np.testing.assert_allclose(to_np(got), oracle.cett(*w, X, eps)[0], rtol=tol, atol=1e-6)
    # limits: eps = 0 cuts nothing, eps = +inf cuts everything
    got, mean = clada.cett_eval(ctx, layer, Xd, 0.0)
    assert torch.all(got == 0) and float(mean.item()) == 0.0
    got, mean = clada.cett_eval(ctx, layer, Xd, float("inf"))
    np.testing.assert_allclose(to_np(got), 1.0, rtol=1e-6)


@pytest.mark.parametrize("cfg_name,d,F,T,tile", CASES)
@pytest.mark.parametrize("bound", [0.2, 0.05])
def test_cett_search_parity(clada, cfg_name, d, F, T, tile, bound):
    cfg, w, X, ctx, layer, Xd = _setup(clada, cfg_name, d, F, T, tile=tile)
    tau_d, mean_d = clada.threshold_search_cett(ctx, layer, Xd, bound)
    torch.cuda.synchronize()
    tau, mean = float(tau_d.item()), float(mean_d.item())
    tol = TOL_SEARCH[cfg.dtype]
    # What is unique: the result is feasible and sits at a boundary of the feasible set, both judged
    # by the oracle.  tau is one of the device's own magnitudes, so the oracle is asked just below it
    # (that neuron surely kept) and just above it (surely cut).
    m_below = oracle.cett(*w, X, tau * (1 - 1e-5))[1]
    m_above = oracle.cett(*w, X, tau * (1 + 1e-5))[1]
    assert m_below <= bound * (1 + tol) + 1e-6
    assert m_above >= bound * (1 - tol) - 1e-6
    assert mean == pytest.approx(m_below, rel=tol, abs=1e-6) and mean <= bound
    # and it agrees with the exact maximum where single-neuron wiggles are small against the bound
    tau_ref, mean_ref, rc = oracle.cett_search(*w, X, bound)
    assert rc == 0
    if T * F >= 20000:
        assert tau == pytest.approx(tau_ref, rel=TOL_TAU[cfg.dtype])


def test_cett_search_bound_zero_returns_smallest_magnitude(clada):
    """Nothing may be lost: the largest eps that cuts nothing is the smallest pooled magnitude."""
    cfg, w, X, ctx, layer, Xd = _setup(clada, "c1", 64, 96, 20)
    st = clada.prefix_stats(ctx, layer, Xd, want_y=False)
    pmin = float(st.abs_act_pool.min().item())
    tau, mean = clada.threshold_search_cett(ctx, layer, Xd, 0.0)
    assert float(tau.item()) == pmin and float(mean.item()) == 0.0


def test_cett_search_fewer_probes_stay_feasible_and_below(clada):
    cfg, w, X, ctx, layer, Xd = _setup(clada, "c2", 256, 384, 96)
    full = float(clada.threshold_search_cett(ctx, layer, Xd, 0.2, 31)[0].item())
    prev = 0.0
    for n in (4, 8, 12, 20):
        tau_d, mean_d = clada.threshold_search_cett(ctx, layer, Xd, 0.2, n)
        tau = float(tau_d.item())
        assert prev <= tau <= full and float(mean_d.item()) <= 0.2
        prev = tau
    # run to run the whole search is bit-reproducible
    again = float(clada.threshold_search_cett(ctx, layer, Xd, 0.2, 31)[0].item())
    assert again == full


def test_cett_argument_errors(clada):
    from paper_2502_19078_amd.binding import CladaError
    cfg, w, X, ctx, layer, Xd = _setup(clada, "c1", 64, 96, 20)
    for bad in (1.0, -0.1, float("nan")):
        with pytest.raises(CladaError):
            clada.threshold_search_cett(ctx, layer, Xd, bad)
    for n in (0, 32):
        with pytest.raises(CladaError):
            clada.threshold_search_cett(ctx, layer, Xd, 0.2, n)
    with pytest.raises(CladaError):
        clada.cett_eval(ctx, layer, Xd, float("nan"))
    small = clada.Context(0, 4096)
    with pytest.raises(CladaError):
        clada.threshold_search_cett(small, layer, Xd, 0.2)


def test_cett_search_full_size_7b_layer(clada):
    """Config 2's layer shape and prefix length as the validation set: the result is checked with two
    oracle evaluations (feasible at tau, over the bound just above it)."""
    cfg = synth.CONFIGS["c2"]
    d, F, T = cfg.d, cfg.d_ff, 128
    cfg, w, X, ctx, layer, Xd = _setup(clada, "c2", d, F, T, layer_id=5)
    tau_d, mean_d = clada.threshold_search_cett(ctx, layer, Xd, 0.2)
    torch.cuda.synchronize()
    tau, mean = float(tau_d.item()), float(mean_d.item())
    m_at = oracle.cett(*w, X, tau * (1 - 1e-5))[1]
    m_above = oracle.cett(*w, X, tau * 1.002)[1]
    assert m_at <= 0.2 * (1 + TOL_CETT["bf16"]) and m_above > 0.2 * (1 - TOL_CETT["bf16"])
    assert mean == pytest.approx(m_at, rel=TOL_CETT["bf16"])
    assert 0.19 < m_at <= 0.2002


def test_cett_search_graph_replay_matches_eager(clada):
    """The bracket lives on the device and every probe reads it there: the whole search can be
    captured once and replayed; each replay must give the eager bits."""
    cfg, w, X, ctx, layer, Xd = _setup(clada, "c2", 512, 640, 200)
    tau_e, mean_e = clada.threshold_search_cett(ctx, layer, Xd, 0.2)
    torch.cuda.synchronize()
    tau_e, mean_e = tau_e.clone(), mean_e.clone()
    out = torch.zeros(1, dtype=torch.float32, device=DEV)
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        clada.threshold_search_cett(ctx, layer, Xd, 0.2, out=out)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=side):
        clada.threshold_search_cett(ctx, layer, Xd, 0.2, out=out)
    for _ in range(3):
        out.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, tau_e)
        again = clada.threshold_search_cett(ctx, layer, Xd, 0.2)[0]      # eager call between replays
        torch.cuda.synchronize()
        assert torch.equal(again, tau_e)


# d, F, T, kind, dtype, weight std: searches large enough (2^20 magnitudes) to close a bracket by sampled thresholds first;
# rows of one, two and four 16-byte groups per thread, ragged neuron counts and tokens, every family
LARGE = [
    (1024, 11008, 96, "silu", "bf16", 0.02), (4096, 5003, 260, "silu", "bf16", 0.02), (2056, 16400, 67, "gelu", "bf16", 0.03),
    (8192, 8192, 128, "silu", "bf16", 0.005), (1024, 4096, 300, "relu", "bf16", 0.02), (512, 4100, 256, "silu", "f32", 0.04),
    (4096, 4096, 256, "relu", "f32", 0.02),
]


@pytest.mark.parametrize("d,F,T,kind,dtype,std", LARGE)
def test_large_search_ends_where_the_plain_bisection_does(clada, d, F, T, kind, dtype, std):
    """30 probes run the plain bisection and leave two neighbouring floats open, 31 the large search.  Its cut sums are
    formed in another order (rel. 1e-6 of a norm), which can move the result past the magnitudes that close to the bound."""
    from paper_2502_19078_amd import binding
    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    g = torch.Generator(device=DEV).manual_seed(d + F)
    n = lambda *s, k=std: torch.randn(s, generator=g, device=DEV) * k
    w = [n(F, d).to(dt) for _ in range(2 if kind == "relu" else 3)]
    layer = (clada.Layer(w[0], None, w[1], kind=binding.RELU, b_in=n(F), b_out=n(d)) if kind == "relu"
             else clada.Layer(*w, kind=binding.GEGLU if kind == "gelu" else binding.SWIGLU))
    x = n(T, d, k=1.0).to(dt)
    x[5] = x[6]                                              # two tokens with the same magnitudes
    ctx = clada.Context(0, clada.workspace_bytes(d, F, 0, T, 0))
    for bound in (0.02, 0.2, 0.6):
        t30, m30 = clada.threshold_search_cett(ctx, layer, x, bound, n_probes=30)
        for _ in range(2):
            t31, m31 = clada.threshold_search_cett(ctx, layer, x, bound)
            assert float(t31) == pytest.approx(float(t30), rel=2e-6), bound
            assert float(m31) == pytest.approx(float(m30), rel=1e-5) and float(m31) <= bound
            assert float(clada.cett_eval(ctx, layer, x, float(t31))[1]) == pytest.approx(float(m31), rel=2e-6)


def test_large_search_without_a_largest_threshold(clada):
    """A bias that dominates the output: every threshold satisfies the bound, and the largest finite float comes back, as
    from the plain bisection."""
    from paper_2502_19078_amd import binding
    d, F, T = 512, 4096, 257
    g = torch.Generator(device=DEV).manual_seed(1)
    w = [(torch.randn((F, d), generator=g, device=DEV) * 0.02).bfloat16() for _ in range(2)]
    layer = clada.Layer(w[0], None, w[1], kind=binding.RELU, b_in=None, b_out=torch.full((d,), 1e4, device=DEV))
    x = torch.randn((T, d), generator=g, device=DEV).bfloat16()
    ctx = clada.Context(0, clada.workspace_bytes(d, F, 0, T, 0))
    tau, mean = clada.threshold_search_cett(ctx, layer, x, 0.2)
    assert float(tau) == float(np.finfo(np.float32).max) and 0.0 < float(mean) < 0.2


# Above 1024 tokens the mean of a probe is formed by a launch of its own; the edge, ragged counts, rows in one and two parts.
@pytest.mark.parametrize("T,d,F,dtype", [(1024, 512, 1100, "bf16"), (1025, 512, 1100, "bf16"), (3001, 256, 1000, "bf16"),
                                          (2050, 2056, 2100, "bf16"), (1500, 512, 800, "f32")])
def test_large_search_over_many_tokens(clada, T, d, F, dtype):
    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    g = torch.Generator(device=DEV).manual_seed(T + d)
    n = lambda *s, k: torch.randn(s, generator=g, device=DEV) * k
    layer = clada.Layer(*[n(F, d, k=d ** -0.5).to(dt) for _ in range(3)])
    x = n(T, d, k=1.0).to(dt)
    ctx = clada.Context(0, clada.workspace_bytes(d, F, 0, T, 0))
    for bound in (0.05, 0.3):
        t30, m30 = clada.threshold_search_cett(ctx, layer, x, bound, n_probes=30)
        t31, m31 = clada.threshold_search_cett(ctx, layer, x, bound)
        assert float(t31) == pytest.approx(float(t30), rel=2e-6), bound
        assert float(m31) == pytest.approx(float(m30), rel=1e-5) and float(m31) <= bound
        assert float(clada.cett_eval(ctx, layer, x, float(t31))[1]) == pytest.approx(float(m31), rel=2e-6)


def test_search_cost_grows_with_the_tokens_not_with_their_square(clada):
    """65536 tokens of a narrow layer: 30 probes are the plain bisection, whose cost is linear in the tokens; the search with 31
    measures 0.8 of it (with a mean per workgroup and probe it was more than six times as slow)."""
    d, F, T = 512, 2048, 65536
    g = torch.Generator(device=DEV).manual_seed(3)
    layer = clada.Layer(*[(torch.randn((F, d), generator=g, device=DEV) * 0.03).bfloat16() for _ in range(3)])
    x = torch.randn((T, d), generator=g, device=DEV).bfloat16()
    ctx = clada.Context(0, clada.workspace_bytes(d, F, 0, T, 0))
    best = {}
    for n in (30, 31):
        clada.threshold_search_cett(ctx, layer, x, 0.2, n_probes=n)
        times = []
        for _ in range(3):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            clada.threshold_search_cett(ctx, layer, x, 0.2, n_probes=n)
            b.record()
            b.synchronize()
            times.append(a.elapsed_time(b))
        best[n] = min(times)
    assert best[31] < 2.0 * best[30], best


# d, F, T, dtype: one, three and seven thresholds a launch of the last stage (by the row norms' room: 1, 2, 4, 6 and more of them), just above
# the smallest search that is bracketed, d_ff below and above 2 d (the probes' sums kept or formed again), more magnitudes in
# the bracket than threads.
PER_LAUNCH = [(64, 4099, 64, "bf16"), (256, 3300, 80, "bf16"), (512, 2100, 130, "bf16"), (512, 1100, 263, "f32"), (1536, 2000, 140, "f32"),
              (1104, 4111, 64, "bf16"), (64, 140000, 64, "bf16")]


@pytest.mark.parametrize("d,F,T,dtype", PER_LAUNCH)
def test_search_thresholds_per_launch(clada, d, F, T, dtype):
    """Against the plain bisection of 30 probes.  The sums' order differs (rel. 1e-6 of a norm, so 1e-6 of a mean whose slope over the
    ranks is about one): the result may move by T F 1e-6 magnitudes and the one next to them, which lie up to 10 / (T F) apart."""
    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    g = torch.Generator(device=DEV).manual_seed(d + F)
    n = lambda *s, k: torch.randn(s, generator=g, device=DEV) * k
    layer = clada.Layer(*[n(F, d, k=d ** -0.5).to(dt) for _ in range(3)])
    x = n(T, d, k=1.0).to(dt)
    ctx = clada.Context(0, clada.workspace_bytes(d, F, 0, T, 0))
    for bound in (0.03, 0.25, 0.7):
        t30, m30 = clada.threshold_search_cett(ctx, layer, x, bound, n_probes=30)
        t31, m31 = clada.threshold_search_cett(ctx, layer, x, bound)
        again = clada.threshold_search_cett(ctx, layer, x, bound)
        assert torch.equal(t31, again[0]) and torch.equal(m31, again[1])
        assert float(t31) == pytest.approx(float(t30), rel=1e-5 + 20.0 / (T * F)), bound
        assert float(m31) <= bound and float(m31) == pytest.approx(float(m30), rel=1e-5 + 20.0 / (T * F))
        assert float(clada.cett_eval(ctx, layer, x, float(t31))[1]) == pytest.approx(float(m31), rel=2e-6)


# The search over a table: threads a token (1, 2, 4, 8), their edges, rows of one to four groups of 16 bytes a thread, windows just wide enough for
# one, sums in one buffer and two; inputs whose answer lies past the first table, whose first probes fail, whose tokens have more
# equal magnitudes than a table takes.
@pytest.mark.parametrize("d,F,T,dtype,how", [
    (512, 1200, 70, "f32", "plain"), (768, 1500, 64, "bf16", "plain"), (512, 4200, 64, "bf16", "plain"), (520, 2300, 128, "bf16", "plain"), (1024, 2100, 129, "bf16", "plain"), (2056, 2100, 256, "bf16", "plain"),
    (512, 1100, 257, "bf16", "plain"), (512, 1100, 512, "bf16", "plain"), (512, 1100, 513, "bf16", "plain"), (512, 2100, 1024, "bf16", "plain"),
    (6144, 6200, 64, "bf16", "plain"), (256, 11900, 900, "bf16", "plain"), (256, 12100, 900, "bf16", "plain"), (1028, 2100, 130, "f32", "plain"),
    (3072, 3100, 100, "f32", "plain"), (1024, 3000, 200, "bf16", "common"), (1024, 3000, 200, "f32", "common"), (1024, 4096, 300, "bf16", "rows"),
    (1024, 4096, 300, "bf16", "tokens"), (1024, 4096, 130, "bf16", "ties"), (512, 2048, 200, "f32", "ties"), (1024, 4096, 300, "bf16", "relu"),
])
def test_search_over_a_table(clada, d, F, T, dtype, how):
    """As above: against the plain bisection of 30 probes, with the same bounds."""
    from paper_2502_19078_amd import binding
    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    g = torch.Generator(device=DEV).manual_seed(d + F + T)
    n = lambda *s, k=1.0: torch.randn(s, generator=g, device=DEV) * k
    w = [n(F, d, k=d ** -0.5) for _ in range(3)]
    x = n(T, d)
    if how == "common":                                      # rows of W_down along one direction
        w[2] += n(1, d, k=d ** -0.5)
    if how == "rows":
        w[2] *= torch.exp(1.5 * n(F, 1))
    if how == "tokens":                                      # tokens of unequal norm
        x *= torch.exp(n(T, 1))
    if how == "ties":                                        # eight different gate rows
        w[0] = w[0][torch.arange(F, device=DEV) % 8]
    w = [a.to(dt) for a in w]
    layer = clada.Layer(w[0], None, w[2], kind=binding.RELU, b_in=n(F), b_out=n(d)) if how == "relu" else clada.Layer(*w)
    x = x.to(dt)
    x[3] = x[2]                                              # two tokens alike
    ctx = clada.Context(0, clada.workspace_bytes(d, F, 0, T, 0))
    for bound in (0.02, 0.2, 0.6):
        t30, m30 = clada.threshold_search_cett(ctx, layer, x, bound, n_probes=30)
        t31, m31 = clada.threshold_search_cett(ctx, layer, x, bound)
        again = clada.threshold_search_cett(ctx, layer, x, bound)
        assert torch.equal(t31, again[0]) and torch.equal(m31, again[1])
        assert float(t31) == pytest.approx(float(t30), rel=1e-5 + 20.0 / (T * F)), bound
        assert float(m31) <= bound and float(m31) == pytest.approx(float(m30), rel=1e-5 + 20.0 / (T * F))
        assert float(clada.cett_eval(ctx, layer, x, float(t31))[1]) == pytest.approx(float(m31), rel=2e-6)


@pytest.mark.parametrize("d,F,T,dtype,tile", [(768, 96, 257, "bf16", 2), (576, 288, 300, "bf16", 2), (1024, 2960, 1300, "bf16", 0), (576, 4128, 64, "bf16", 2),
                                              (768, 2015, 300, "bf16", 2), (512, 129, 200, "bf16", 1), (72, 97, 130, "bf16", 0), (256, 96, 70, "f32", 0)])
def test_what_the_workspace_held_does_not_reach_the_search(clada, d, F, T, dtype, tile):
    """The projections read h in columns of 64; a NaN behind d_ff would pass as a token that loses nothing.  Plain and bracketed searches."""
    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    g = torch.Generator(device=DEV).manual_seed(d + F + T)
    w = [(torch.randn(F, d, generator=g, device=DEV) * d ** -0.5).to(dt) for _ in range(3)]
    x = torch.randn(T, d, generator=g, device=DEV).to(dt)
    layer = clada.Layer(*w)
    ctx = nan_workspace(clada, d, F, T, dt)
    ctx.set_option("prefix.tile", tile)
    pool = clada.prefix_stats(ctx, layer, x, want_y=False).abs_act_pool.double()
    h = torch.nn.functional.silu(x.double() @ w[0].double().t()) * (x.double() @ w[1].double().t())
    dense = (h @ w[2].double()).norm(dim=1)
    exact = lambda eps: ((torch.where(pool < eps, h, 0.0) @ w[2].double()).norm(dim=1) / dense).cpu().numpy()      # (the device's own cut set)
    ctx = nan_workspace(clada, d, F, T, dt)
    ctx.set_option("prefix.tile", tile)
    eps = float(pool.flatten()[: 1 << 20].median())
    got, mean = clada.cett_eval(ctx, layer, x, eps)
    np.testing.assert_allclose(to_np(got), exact(eps), rtol=TOL_CETT[dtype], atol=1e-6)
    for bound in (0.05, 0.25):
        ctx = nan_workspace(clada, d, F, T, dt)
        ctx.set_option("prefix.tile", tile)
        tau, mean = clada.threshold_search_cett(ctx, layer, x, bound)
        assert float(mean) <= bound
        assert float(mean) == pytest.approx(exact(float(tau)).mean(), rel=TOL_CETT[dtype], abs=1e-6)


# Splits of the down projection whose parts the smallest workspace does not hold, in the calls of the error bound: plain and bracketed
# searches, kept sums in two buffers (d_ff >= 2 d) and formed again, biases
@pytest.mark.parametrize("d,F,T,dtype,kind", [
    (1024, 4096, 64, "bf16", "swiglu"), (512, 3333, 100, "bf16", "swiglu"), (512, 3333, 100, "bf16", "relu"), (512, 900, 300, "bf16", "geglu"),
    (1024, 1984, 140, "bf16", "swiglu"), (256, 2085, 40, "bf16", "relu"), (260, 3001, 90, "f32", "swiglu"), (512, 1111, 140, "f32", "relu"),
    (512, 2222, 256, "f32", "swiglu"), (256, 1031, 40, "f32", "relu")])
def test_cett_does_not_depend_on_the_room_for_a_split(clada, d, F, T, dtype, kind):
    from test_gpu_prefix import _split_layer
    layer, x = _split_layer(clada, d, F, T, dtype, kind)
    least = least_workspace(clada, lambda c: clada.cett_eval(c, layer, x, 0.1))
    advised = clada.workspace_bytes(d, F, 0, T, 0)
    want = None
    for n in (advised, least, least + 4 * T * d, least + 8 * T * d, least + 20 * T * d):
        ctx = clada.Context(0, n)
        got = [*clada.cett_eval(ctx, layer, x, 0.1), *clada.threshold_search_cett(ctx, layer, x, 0.2),
               *clada.threshold_search_cett(ctx, layer, x, 0.2, n_probes=30)]
        if want is None:
            want = got
            assert 0.0 < float(got[1]) < 1.0 and float(got[3]) <= 0.2
        for i, (a, b) in enumerate(zip(got, want)):
            assert torch.equal(a, b), (i, n - least)
