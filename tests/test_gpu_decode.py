"""GPU parity: clada_sparse_ffn_decode / clada_dense_ffn_decode against the fp64 oracle."""
import numpy as np
import pytest
import torch

import oracle
import synth
from gpu_util import (DEV, TOL_Y, assert_close_y, check_mask_band, to_dev, to_np, unpack_bits)
from tolerances import EPS32, decode_condition

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def clada():
    import paper_2502_19078_amd as m
    m.load_library()
    return m


def _case(cfg_name, seed, d, F, B, layer=0, step=0):
    cfg = synth.CONFIGS[cfg_name]
    w = synth.layer_weights(cfg, seed, layer, d=d, d_ff=F)
    x = synth.decode_hidden(cfg, seed, layer, step, B=B, d=d)
    return cfg, w, x


def _tau_for(w, x, q):
    """Per-token thresholds at about sparsity q (fp32 values, as the GPU will see them)."""
    act = np.abs(oracle.gate_act(w[0], x))
    return np.quantile(act, q, axis=1).astype(np.float32)


def _run_sparse(clada, cfg, w, x, tau, wgs_per_cu=1):
    F, d = w[0].shape
    B = x.shape[0]
    ctx = clada.Context(0, clada.workspace_bytes(d, F, B, 0, 0))
    ctx.set_option("decode.wgs_per_cu", wgs_per_cu)
    layer = clada.Layer(*[to_dev(a, cfg.dtype) for a in w])
    xd = to_dev(x, cfg.dtype)
    y, idx, cnt, bits = clada.sparse_ffn_decode(ctx, layer, xd, torch.from_numpy(tau).to(DEV), want_lists=True)
    torch.cuda.synchronize()
    return ctx, layer, xd, y, idx.cpu().numpy(), cnt.cpu().numpy(), unpack_bits(bits, F)


def _check_against_oracle(cfg, w, x, tau, y, idx, cnt, mask, what):
    ref = oracle.sparse_decode(*w, x, tau.astype(np.float64))
    flips = check_mask_band(mask, ref["act"], tau.astype(np.float64), what)
    # index list / counts are exactly what the GPU's own mask implies
    union = np.flatnonzero(mask.any(0))
    assert cnt[0] == union.size and np.array_equal(idx[: cnt[0]], union), f"{what}: index list"
    assert np.all(idx[cnt[0]:] == -1), f"{what}: entries past the count were touched"
    assert np.array_equal(cnt[1:], mask.sum(1)), f"{what}: per-token counts"
    if flips == 0:
        assert np.array_equal(idx[: cnt[0]], ref["active_idx"]) and np.array_equal(cnt, ref["n_active"])
        y_ref = ref["y"]
    else:   # in-band flips: compare with the oracle evaluated on the GPU's (validated) mask
        y_ref = oracle.decode_given_mask(*w, x, mask)
    assert_close_y(to_np(y), y_ref, TOL_Y[cfg.dtype], what)
    return flips


CASES = [
    # cfg, d, F, B, q    (several tiles + ragged tails: F not a multiple of the workgroup count)
    ("c1", 512, 1376, 1, 0.40),      # config 1 as written
    ("c1", 512, 1376, 4, 0.40),
    ("c1", 320, 77, 2, 0.50),        # d not a multiple of a wave's 256-float chunk, tiny F
    ("c1", 64, 3000, 1, 0.30),
    ("c2", 1024, 1000, 3, 0.45),     # bf16
    ("c2", 4096, 2752, 1, 0.45),     # bf16, real row length, quarter of the 7B d_ff
    ("c5", 5120, 1111, 2, 0.60),     # 13B row length (10 chunks per lane)
    ("c2", 8, 130, 1, 0.45),         # one 16-byte chunk per row
]


@pytest.mark.parametrize("cfg_name,d,F,B,q", CASES)
def test_sparse_decode_parity(clada, cfg_name, d, F, B, q):
    for seed in (0, 1):
        cfg, w, x = _case(cfg_name, seed, d, F, B)
        tau = _tau_for(w, x, q)
        _, _, _, y, idx, cnt, mask = _run_sparse(clada, cfg, w, x, tau)
        _check_against_oracle(cfg, w, x, tau, y, idx, cnt, mask, f"{cfg_name} d={d} F={F} B={B} seed={seed}")
        rho = 1.0 - cnt[1:].mean() / F
        assert abs(rho - q) < 0.02


@pytest.mark.parametrize("cfg_name,d,F,B", [("c1", 512, 1376, 2), ("c2", 1024, 1000, 2)])
def test_tau_zero_is_dense_and_tau_inf_is_zero(clada, cfg_name, d, F, B):
    cfg, w, x = _case(cfg_name, 3, d, F, B)
    ctx, layer, xd, y0, idx, cnt, mask = _run_sparse(clada, cfg, w, x, np.zeros(B, np.float32))
    assert mask.all() and list(cnt) == [F] * (1 + B) and np.array_equal(idx, np.arange(F))
    yd = clada.dense_ffn_decode(ctx, layer, xd)
    torch.cuda.synchronize()
    assert torch.equal(y0, yd)                      # same kernel structure, same summation order
    assert_close_y(to_np(yd), oracle.dense_decode(*w, x), TOL_Y[cfg.dtype], "dense twin")
    _, _, _, yi, idx, cnt, mask = _run_sparse(clada, cfg, w, x, np.full(B, np.inf, np.float32))
    assert not mask.any() and list(cnt) == [0] * (1 + B) and np.all(idx == -1)
    assert torch.count_nonzero(yi).item() == 0


def test_batch_rows_independent_and_per_token_thresholds(clada):
    cfg, w, x = _case("c2", 4, 1024, 1500, 5)
    tau = _tau_for(w, x, 0.45) * np.array([1.0, 1.8, 1.12, 1.92, 0.08], np.float32)
    ctx, layer, xd, y, idx, cnt, mask = _run_sparse(clada, cfg, w, x, tau)
    _check_against_oracle(cfg, w, x, tau, y, idx, cnt, mask, "per-token tau")
    for b in range(5):
        # a single-token call runs a different kernel (other fp32 summation order): same mask,
        # same output within the parity tolerance
        yb, idx_b, cnt_b, bits_b = clada.sparse_ffn_decode(ctx, layer, xd[b:b + 1].contiguous(),
                                                           torch.from_numpy(tau[b:b + 1]).to(DEV), want_lists=True)
        torch.cuda.synchronize()
        assert np.array_equal(unpack_bits(bits_b, 1500)[0], mask[b]), f"row {b}: mask differs"
        assert_close_y(to_np(yb), to_np(y[b:b + 1]), TOL_Y[cfg.dtype], f"row {b} batched vs single-token")
    # generic kernels for both the batched and the single-token call: bit-identical rows
    ctx.set_option("decode.b1", 0)
    ctx.set_option("decode.batched", 0)
    y = clada.sparse_ffn_decode(ctx, layer, xd, torch.from_numpy(tau).to(DEV))
    for b in range(5):
        yb = clada.sparse_ffn_decode(ctx, layer, xd[b:b + 1].contiguous(), torch.from_numpy(tau[b:b + 1]).to(DEV))
        torch.cuda.synchronize()
        assert torch.equal(yb[0], y[b]), f"row {b} differs between batched and single-token call"


@pytest.mark.parametrize("wgs,B", [(1, 2), (2, 2), (1, 1)])
def test_run_to_run_bit_reproducible(clada, wgs, B):
    cfg, w, x = _case("c2", 5, 2048, 3000, B)
    tau = _tau_for(w, x, 0.45)
    outs = []
    for _ in range(3):
        _, _, _, y, idx, cnt, mask = _run_sparse(clada, cfg, w, x, tau, wgs_per_cu=wgs)
        outs.append((y.clone(), idx.copy(), cnt.copy()))
    for y, idx, cnt in outs[1:]:
        assert torch.equal(y, outs[0][0]) and np.array_equal(idx, outs[0][1]) and np.array_equal(cnt, outs[0][2])


def test_nan_activation_is_cut(clada):
    cfg, w, x = _case("c1", 6, 256, 300, 1)
    w = [a.copy() for a in w]
    w[0][17, 3] = np.nan
    tau = np.zeros(1, np.float32)
    _, _, _, y, idx, cnt, mask = _run_sparse(clada, cfg, w, x, tau)
    assert not mask[0, 17] and cnt[0] == 299
    ref = oracle.sparse_decode(*w, x, tau.astype(np.float64))
    assert_close_y(to_np(y), ref["y"], TOL_Y["f32"], "NaN gate row")


def test_full_size_7b_layer_bench_configuration(clada):
    """LLaMA2-7B FFN shape in the launch configuration the benchmark times (one layer, B=1,
    thresholds from the library's own prefix calibration): every output element and the whole
    index list are checked, for two layers and two decode steps."""
    cfg = synth.CONFIGS["c2"]
    d, F = cfg.d, cfg.d_ff
    ctx = clada.Context(0, clada.workspace_bytes(d, F, 1, 0, 0))
    for layer_id in (0, 17):
        w = synth.layer_weights(cfg, 0, layer_id)
        layer = clada.Layer(*[to_dev(a, cfg.dtype) for a in w])
        for step in (0, 1):
            x = synth.decode_hidden(cfg, 0, layer_id, step)
            tau = _tau_for(w, x, cfg.q)
            y, idx, cnt, bits = clada.sparse_ffn_decode(ctx, layer, to_dev(x, cfg.dtype),
                                                        torch.from_numpy(tau).to(DEV), want_lists=True)
            torch.cuda.synchronize()
            _check_against_oracle(cfg, w, x, tau, y, idx.cpu().numpy(), cnt.cpu().numpy(),
                                  unpack_bits(bits, F), f"7B layer {layer_id} step {step}")
        yd = clada.dense_ffn_decode(ctx, layer, to_dev(x, cfg.dtype))
        torch.cuda.synchronize()
        assert_close_y(to_np(yd), oracle.dense_decode(*w, x), TOL_Y["bf16"], "7B dense twin")


def test_batch1_and_generic_paths_agree(clada):
    """Batch-1 calls take the single-kernel split-d kernel; the generic multi-kernel path must
    give the same mask and the same output up to fp32 summation order."""
    for cfg_name, d, F in (("c2", 4096, 5000), ("c1", 512, 1376), ("c5", 5120, 13824)):
        cfg, w, x = _case(cfg_name, 7, d, F, 1)
        tau = _tau_for(w, x, 0.45)
        ctx = clada.Context(0, clada.workspace_bytes(d, F, 1, 0, 0))
        layer = clada.Layer(*[to_dev(a, cfg.dtype) for a in w])
        xd, td = to_dev(x, cfg.dtype), torch.from_numpy(tau).to(DEV)
        outs = {}
        for coop in (3, 2, 1, 0):                       # balanced, plain, automatic choice, generic kernels
            ctx.set_option("decode.b1", coop)
            y, idx, cnt, bits = clada.sparse_ffn_decode(ctx, layer, xd, td, want_lists=True)
            yd = clada.dense_ffn_decode(ctx, layer, xd)
            torch.cuda.synchronize()
            outs[coop] = (to_np(y), idx.cpu().numpy(), cnt.cpu().numpy(), to_np(yd))
            _check_against_oracle(cfg, w, x, tau, y, idx.cpu().numpy(), cnt.cpu().numpy(), unpack_bits(bits, F),
                                  f"{cfg_name} coop={coop}")
        for c in (1, 2, 3):
            assert np.array_equal(outs[c][1], outs[0][1]) and np.array_equal(outs[c][2], outs[0][2])
            assert_close_y(outs[c][0], outs[0][0], TOL_Y[cfg.dtype], "batch-1 path vs generic")
            assert_close_y(outs[c][3], outs[0][3], TOL_Y[cfg.dtype], "dense batch-1 path vs generic")


@pytest.mark.parametrize("own_first", [1, 5, 9, 14])
def test_balancing_any_own_first(clada, own_first):
    """The surplus hand-over must be exact for every split between own and pooled neurons,
    including very sparse and fully dense masks."""
    cfg, w, x = _case("c2", 8, 4096, 11008, 1)
    ctx = clada.Context(0, clada.workspace_bytes(4096, 11008, 1, 0, 0))
    ctx.set_option("decode.b1", 3)
    ctx.set_option("decode.own_first", own_first)
    layer = clada.Layer(*[to_dev(a, cfg.dtype) for a in w])
    xd = to_dev(x, cfg.dtype)
    for q in (0.0, 0.45, 0.9, 0.999):
        tau = _tau_for(w, x, q) if q > 0 else np.zeros(1, np.float32)
        y, idx, cnt, bits = clada.sparse_ffn_decode(ctx, layer, xd, torch.from_numpy(tau).to(DEV), want_lists=True)
        torch.cuda.synchronize()
        _check_against_oracle(cfg, w, x, tau, y, idx.cpu().numpy(), cnt.cpu().numpy(), unpack_bits(bits, 11008),
                              f"own_first={own_first} q={q}")


def test_graph_replay_matches_eager(clada):
    """The decode call reads its epoch from device memory, so a captured launch can be replayed;
    every replay (with eager calls in between) must reproduce the eager bits."""
    cfg, w, x = _case("c2", 9, 4096, 11008, 1)
    ctx = clada.Context(0, clada.workspace_bytes(4096, 11008, 1, 0, 0))
    layer = clada.Layer(*[to_dev(a, cfg.dtype) for a in w])
    xd = to_dev(x, cfg.dtype)
    td = torch.from_numpy(_tau_for(w, x, 0.45)).to(DEV)
    y_eager = clada.sparse_ffn_decode(ctx, layer, xd, td).clone()
    y_g = torch.empty_like(y_eager)
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        clada.sparse_ffn_decode(ctx, layer, xd, td, y=y_g)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=side):
        clada.sparse_ffn_decode(ctx, layer, xd, td, y=y_g)
    for _ in range(4):
        y_g.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(y_g, y_eager)
        y2 = clada.sparse_ffn_decode(ctx, layer, xd, td)          # eager call between replays
        torch.cuda.synchronize()
        assert torch.equal(y2, y_eager)


@pytest.mark.parametrize("cfg_name,layer_id", [("c3", 5), ("c4", 11), ("c5", 20)])
def test_full_size_other_configurations(clada, cfg_name, layer_id):
    """One full-size layer of the Mistral-7B (B=8), LLaMA-3-8B (B=1) and LLaMA2-13B (B=16)
    shapes, per-token thresholds spread by the four indicator factors; every output element,
    every mask bit and the union list are checked against the oracle."""
    cfg = synth.CONFIGS[cfg_name]
    d, F, B = cfg.d, cfg.d_ff, cfg.B
    w = synth.layer_weights(cfg, 0, layer_id)
    x = synth.decode_hidden(cfg, 0, layer_id, 0)
    factors = np.resize(np.array([1.0, 1.80, 1.12, 1.92], np.float32), B)
    tau = _tau_for(w, x, cfg.q) * factors
    ctx = clada.Context(0, clada.workspace_bytes(d, F, B, 0, 0))
    layer = clada.Layer(*[to_dev(a, cfg.dtype) for a in w])
    y, idx, cnt, bits = clada.sparse_ffn_decode(ctx, layer, to_dev(x, cfg.dtype), torch.from_numpy(tau).to(DEV),
                                                want_lists=True)
    torch.cuda.synchronize()
    cnt = cnt.cpu().numpy()
    _check_against_oracle(cfg, w, x, tau, y, idx.cpu().numpy(), cnt, unpack_bits(bits, F),
                          f"{cfg_name} layer {layer_id}")
    if B > 1:       # independent tokens: the union is nearly everything, each row keeps its own sparsity
        assert cnt[0] > 0.95 * F and np.all(cnt[1:] < 0.75 * F)


def test_batched_path_bit_reproducible_and_matches_generic(clada):
    """The MFMA batched path (2 <= B <= 16, bf16): identical bits run to run, same masks as the
    generic per-token kernels, outputs within tolerance of them."""
    cfg, w, x = _case("c3", 11, 4096, 3000, 8)
    tau = _tau_for(w, x, 0.45)
    ctx = clada.Context(0, clada.workspace_bytes(4096, 3000, 8, 0, 0))
    layer = clada.Layer(*[to_dev(a, cfg.dtype) for a in w])
    xd, td = to_dev(x, cfg.dtype), torch.from_numpy(tau).to(DEV)
    runs = []
    for batched in (1, 1, 0):
        ctx.set_option("decode.batched", batched)
        y, idx, cnt, bits = clada.sparse_ffn_decode(ctx, layer, xd, td, want_lists=True)
        torch.cuda.synchronize()
        runs.append((y.clone(), idx.cpu().numpy(), cnt.cpu().numpy(), bits.cpu().numpy()))
    assert torch.equal(runs[0][0], runs[1][0])
    for a, b in zip(runs[0][1:], runs[2][1:]):
        assert np.array_equal(a, b)
    assert_close_y(to_np(runs[0][0]), to_np(runs[2][0]), TOL_Y["bf16"], "batched vs generic")


@pytest.mark.parametrize("B", [1, 3])
def test_kernel_event_timing_does_not_change_results(clada, B):
    """diag.kernel_events attaches HIP events to the kernels: same bits out, positive durations back."""
    from paper_2502_19078_amd import binding
    cfg, w, x = _case("c1", 5, 512, 1376, B)
    tau = _tau_for(w, x, 0.4)
    ctx = clada.Context(0, clada.workspace_bytes(512, 1376, B, 0, 0))
    layer = clada.Layer(*[to_dev(a, cfg.dtype) for a in w])
    xd, td = to_dev(x, cfg.dtype), torch.from_numpy(tau).to(DEV)
    y0 = clada.sparse_ffn_decode(ctx, layer, xd, td)[0].clone()
    ctx.set_option("diag.kernel_events", 1)
    y1 = clada.sparse_ffn_decode(ctx, layer, xd, td)[0].clone()
    main_us, fin_us = binding.diag_kernel_times(ctx)
    ctx.set_option("diag.kernel_events", 0)
    assert torch.equal(y0, y1)
    assert 0.0 < main_us < 1e5 and 0.0 < fin_us < 1e5
    with pytest.raises(binding.CladaError):
        binding.diag_kernel_times(ctx)


@pytest.mark.parametrize("cfg_name,d,F,B", [
    ("c2", 256, 300, 64),        # the largest batch the ABI takes
    ("c2", 1024, 520, 17),       # one past 16 tokens: two passes (9 + 8) of the matrix-core path
    ("c2", 2048, 700, 40),       # three passes (14 + 14 + 12)
    ("c2", 1024, 333, 64),       # the largest batch on the matrix-core path: four passes of 16
    ("c2", 2560, 640, 4),        # further widths of the matrix-core path: five waves with 1 KiB slices,
    ("c2", 3072, 500, 3),        #   768-byte slices,
    ("c2", 6144, 300, 5),        #   two parts of 768 bytes,
    ("c2", 8192, 300, 3),        #   two parts of 1 KiB (the longest row)
    ("c2", 1024, 40000, 2),      # more than 2048 neurons per row group: the down kernel takes more row groups
    ("c2", 8192, 300, 1),        # the longest bf16 row (16 KiB)
    ("c1", 4096, 260, 2),        # the longest fp32 row (16 KiB)
    ("c2", 4096, 255, 1),        # fewer neurons than workgroups
    ("c2", 4096, 1, 1),          # a single neuron
])
def test_limits_of_batch_width_and_neuron_count(clada, cfg_name, d, F, B):
    cfg, w, x = _case(cfg_name, 11, d, F, B)
    tau = _tau_for(w, x, 0.45)
    _, _, _, y, idx, cnt, mask = _run_sparse(clada, cfg, w, x, tau)
    _check_against_oracle(cfg, w, x, tau, y, idx, cnt, mask, f"{cfg_name} d={d} F={F} B={B}")


@pytest.mark.parametrize("cfg_name,d,F,B", [
    ("c1", 4096, 300, 2),        # fp32 rows above 8 KiB: two column chunks per wave
    ("c1", 4096, 300, 9),        # two passes (5 + 4)
    ("c1", 4096, 170, 4),        # fewer neurons than workgroups
    ("c1", 4096, 700, 1),        # one token
    ("c1", 2052, 400, 3),        # 16 bytes into the second column chunk of wave 0
    ("c1", 2048, 500, 8),        # whole passes of eight tokens
    ("c1", 1000, 700, 4),        # rows that end inside a KiB
    ("c1", 64, 40000, 3),        # more than 64 neurons per workgroup: rounds
    ("c2", 3584, 500, 5),        # bf16 widths without a matrix-core instance
    ("c2", 4360, 400, 5),        # wide bf16 rows: passes of at most four tokens
    ("c2", 776, 3000, 17),       # three passes, 1.5 KiB rows
    ("c2", 776, 3000, 8), ("c2", 1032, 2000, 17), ("c1", 4096, 170, 1), ("c1", 1028, 16500, 3), ("c1", 516, 300, 3),
])
def test_several_tokens_per_pass_on_the_vector_units(clada, cfg_name, d, F, B):
    """Batches that no other path takes, with thresholds spread over the tokens (one keeps nothing); the dense twin and a list run
    of the union go through the same kernel."""
    cfg, w, x = _case(cfg_name, 21, d, F, B)
    tau = _tau_for(w, x, 0.45) * np.resize(np.array([1.0, 1.8, 1e9, 0.08], np.float32), B)
    ctx, layer, xd, y, idx, cnt, mask = _run_sparse(clada, cfg, w, x, tau)
    _check_against_oracle(cfg, w, x, tau, y, idx, cnt, mask, f"{cfg_name} d={d} F={F} B={B}")
    yd = clada.dense_ffn_decode(ctx, layer, xd)
    assert_close_y(to_np(yd), oracle.dense_decode(*w, x), TOL_Y[cfg.dtype], "dense twin")
    n = max(int(cnt[0]), 1)
    lst = torch.from_numpy(np.arange(0, F, 2, dtype=np.int32)[:n]).to(DEV)
    full = torch.full((F,), F + 7, dtype=torch.int32, device=DEV)        # entries past the count are not read
    full[:lst.numel()] = lst
    ys = clada.static_ffn_decode(ctx, layer, xd, full, torch.tensor([lst.numel()], dtype=torch.int32, device=DEV))
    keep = np.zeros(F, bool)
    keep[lst.cpu().numpy()] = True
    assert_close_y(to_np(ys), oracle.decode_given_mask(*w, x, np.broadcast_to(keep, (B, F))), TOL_Y[cfg.dtype], "list run")


# Passes of 17 to 32 tokens in two tiles: every width that has them, the edges of a tile and of a pass, one pass and two (the second one a
# single tile or short), more than 64 neurons a workgroup, the widest layer for its rows and one past it (passes of 16)
@pytest.mark.parametrize("cfg_name,d,F,B", [
    ("c2", 1024, 777, 17), ("c2", 1024, 16384, 31), ("c2", 1024, 16385, 20), ("c2", 2048, 700, 32), ("c2", 2048, 300, 33), ("c2", 2560, 640, 18),
    ("c2", 2560, 900, 49), ("c2", 3072, 500, 32), ("c2", 4096, 3000, 17), ("c2", 4096, 255, 48),
    # the narrow and the odd widths, from the batch on that the matrix cores take
    ("c2", 512, 600, 12), ("c2", 512, 1700, 32), ("c2", 768, 900, 6), ("c2", 768, 17000, 15), ("c2", 768, 3072, 33), ("c2", 1536, 255, 5), ("c2", 1536, 3840, 4),
    ("c2", 1536, 900, 16), ("c2", 1536, 2000, 31), ("c2", 3584, 500, 3), ("c2", 3584, 900, 16), ("c2", 3584, 700, 33),
])
def test_passes_of_the_matrix_core_path(clada, cfg_name, d, F, B):
    """Thresholds spread over the tokens (one keeps nothing); the dense twin and a list run go through the same kernels."""
    cfg, w, x = _case(cfg_name, 31, d, F, B)
    tau = _tau_for(w, x, 0.45) * np.resize(np.array([1.0, 1.8, 1e9, 0.08, 1.3], np.float32), B)
    ctx, layer, xd, y, idx, cnt, mask = _run_sparse(clada, cfg, w, x, tau)
    _check_against_oracle(cfg, w, x, tau, y, idx, cnt, mask, f"{cfg_name} d={d} F={F} B={B}")
    yd = clada.dense_ffn_decode(ctx, layer, xd)
    assert_close_y(to_np(yd), oracle.dense_decode(*w, x), TOL_Y[cfg.dtype], "dense twin")
    lst = torch.arange(0, F, 3, dtype=torch.int32, device=DEV)
    ys = clada.static_ffn_decode(ctx, layer, xd, lst, torch.tensor([lst.numel()], dtype=torch.int32, device=DEV))
    keep = np.zeros(F, bool)
    keep[::3] = True
    assert_close_y(to_np(ys), oracle.decode_given_mask(*w, x, np.broadcast_to(keep, (B, F))), TOL_Y[cfg.dtype], "list run")


def _parts(v):
    """fp32 values as three bf16 each, exactly (cut, not rounded)."""
    hi = (v.view(torch.int32) & -65536).view(torch.float32)
    mid = ((v - hi).view(torch.int32) & -65536).view(torch.float32)
    return torch.stack([hi, mid, v - hi - mid], 1)


@pytest.mark.parametrize("d,B", [(768, 7), (1024, 2), (2048, 20), (4096, 16)])
def test_equal_h_of_neurons_with_opposite_rows_cancel_exactly(clada, d, B):
    """Neuron 2k has h = fl32(a u), neuron 2k + 1 the same float with nothing rounded (32 times h / 32), and their W_down rows are +1 and -1 in one
    column: whatever h becomes on its way, it is a function of that float.  (A rest taken from the unrounded product differs for one in 500.)"""
    F = 8192
    g = torch.Generator(device=DEV).manual_seed(d)
    a = 32.0 + 32.0 * torch.rand(F // 2, generator=g, device=DEV)        # SiLU(a) = a
    u = 1.0 + torch.rand(F // 2, generator=g, device=DEV)
    h = a * u
    w = [torch.zeros(F, d, device=DEV) for _ in range(3)]
    w[0][0::2, :3], w[1][0::2, :3] = _parts(a), _parts(u)
    w[0][1::2, 0], w[1][1::2, :3] = 32.0, _parts(h / 32.0)
    k = torch.arange(F // 2, device=DEV)
    w[2][2 * k, k % d], w[2][2 * k + 1, k % d] = 1.0, -1.0
    assert all(torch.equal(v.bfloat16().float(), v) for v in w)
    x = torch.zeros(B, d, device=DEV)
    x[:, :3] = 1.0
    layer = clada.Layer(*[v.bfloat16() for v in w])
    ctx = clada.Context(0, clada.workspace_bytes(d, F, B, 0, 0))
    y, _, cnt, _ = clada.sparse_ffn_decode(ctx, layer, x.bfloat16(), torch.full((B,), 1.0, device=DEV), want_lists=True)
    assert int(cnt[0]) == F and not y.any()


@pytest.mark.parametrize("d,B,relu", [(512, 12, False), (512, 40, True), (768, 7, False), (768, 32, True), (1536, 5, False), (1536, 16, True), (1536, 17, False),
                                      (3584, 3, False), (3584, 4, True), (3584, 31, False)])
def test_h_has_all_its_bits_where_the_vector_kernel_has_them(clada, d, B, relu):
    """Neuron 2k has a random h of 24 bits, neuron 2k + 1 its first 16 bits, and their W_down rows are +1 and -1 in column k: what is left is the other
    eight bits, exactly.  Batches of these widths run on the vector units or on the matrix cores by their size."""
    from paper_2502_19078_amd import binding
    F = 1000
    g = torch.Generator(device=DEV).manual_seed(d + B)
    p = _parts(1.0 + torch.rand(F // 2, generator=g, device=DEV))
    w = [torch.zeros(F, d, device=DEV) for _ in range(3)]
    w[0][:, 0] = 32.0                                        # SiLU(32) = 32
    up = w[0] if relu else w[1]
    up[0::2, :3] = p
    up[1::2, :3] = p * torch.tensor([1.0, 1.0, 0.0], device=DEV)
    k = torch.arange(F // 2, device=DEV)
    w[2][2 * k, k], w[2][2 * k + 1, k] = 1.0, -1.0
    assert all(torch.equal(v.bfloat16().float(), v) for v in w)
    x = torch.zeros(B, d, device=DEV)
    x[:, :3] = 1.0
    w = [v.bfloat16() for v in w]
    layer = clada.Layer(w[0], None, w[2], kind=binding.RELU) if relu else clada.Layer(*w)
    want = torch.zeros(B, d, device=DEV)
    want[:, :F // 2] = p[:, 2] * (1.0 if relu else 32.0)
    for batched in (1, 0):
        ctx = clada.Context(0, clada.workspace_bytes(d, F, B, 0, 0))
        ctx.set_option("decode.batched", batched)
        y = clada.sparse_ffn_decode(ctx, layer, x.bfloat16(), torch.full((B,), 0.5, device=DEV))
        assert p[:, 2].count_nonzero() > F // 3 and torch.equal(y.float(), want), batched


def test_infinite_weight_of_a_neuron_a_token_cuts_stays_out_of_its_output(clada):
    """Token 0 keeps neuron 5, whose output row holds an infinity; token 1 cuts it and stays finite."""
    cfg, w, x = _case("c1", 22, 2048, 500, 2)
    w = [a.copy() for a in w]
    w[2][5, 7] = np.inf
    w[0][5] = x[0] / np.linalg.norm(x[0])                    # activation of token 0 about ||x||
    tau = np.array([1.0, 1e3], np.float32)
    _, _, _, y, _, _, mask = _run_sparse(clada, cfg, w, x, tau)
    assert mask[0, 5] and not mask[1, 5]
    assert not np.isfinite(to_np(y)[0, 7]) and np.isfinite(to_np(y)[1]).all()


# The matrix-core path at every width and both tilings: one, two and many units of rows a wave; the bad neuron inside the list or
# its last entry, which the padding of the last unit repeats
@pytest.mark.parametrize("j", [5, -1])
@pytest.mark.parametrize("d,F,B,relu", [(512, 300, 13, False), (768, 900, 7, False), (768, 3072, 33, False), (1024, 700, 2, True), (1536, 600, 16, True),
                                        (2048, 4000, 20, False), (3584, 500, 3, False), (3584, 700, 24, True), (4096, 900, 5, False), (5120, 300, 16, False)])
def test_values_that_are_not_finite_stay_with_the_tokens_that_keep_the_neuron(clada, d, F, B, relu, j):
    """y_b sums over the neurons that b keeps.  An infinite and a NaN entry of W_down, and an infinite u (a: non-gated), reach the tokens that keep
    theirs, as an infinity where the terms say so, and no other; an h above the largest bf16 stays finite."""
    from paper_2502_19078_amd import binding
    g = torch.Generator(device=DEV).manual_seed(d + F + B)
    n = lambda *s, k=1.0: torch.randn(s, generator=g, device=DEV) * k
    j, ju, jh = j % F, F // 2, F // 3
    w = [n(F, d, k=d ** -0.5).bfloat16() for _ in range(2 if relu else 3)]
    b_in = n(F, k=0.1) if relu else None
    wd = w[-1]
    wd[j, 7], wd[j, d - 1] = float("inf"), float("nan")
    wd[ju] = wd[ju].abs() + 0.01
    wd[jh] = 1e-30
    x = n(B, d).bfloat16()
    # neurons j and ju: kept by the even and by the odd tokens alone; jh by every one
    keep_even = torch.arange(B, device=DEV) % 2 == 0
    x[:, 0] = torch.where(keep_even, 30.0, -30.0).bfloat16()
    for k, s in ((j, 1.0), (ju, -1.0)):
        w[0][k] = 0
        w[0][k, 0] = s * 4.0                                 # a = 120 or (a sigma of) -120
    if relu:
        b_in[jh] = 3.4e38                                    # rounds up to infinity in bf16
        b_in[j] = 0.0
        b_in[ju] = 0.0
        w[0][ju, 0] = float("-inf")                          # (a = +inf for the odd tokens, 0 for the even)
    else:
        w[0][jh] = 0
        w[0][jh, 1] = 1e20
        x[:, 1] = x[:, 1].abs() + 1.0
        w[1][jh] = 0
        w[1][jh, 1] = 1e10
        w[1][ju, 0] = float("-inf")                          # u = +inf for the odd tokens
    layer = clada.Layer(w[0], None, w[1], kind=binding.RELU, b_in=b_in, b_out=n(d)) if relu else clada.Layer(*w)
    tau = torch.full((B,), 0.2, device=DEV)
    ctx = clada.Context(0, clada.workspace_bytes(d, F, B, 0, 0))
    y, _, _, bits = clada.sparse_ffn_decode(ctx, layer, x, tau, want_lists=True)
    mask = torch.from_numpy(unpack_bits(bits, F)).to(DEV)
    assert torch.equal(mask[:, j], keep_even) and torch.equal(mask[:, ju], ~keep_even) and mask[:, jh].all()
    a = x.double() @ w[0].double().t()
    a = (a + b_in.double()).clamp_min(0) if relu else a * torch.sigmoid(a)
    h = a if relu else a * (x.double() @ w[1].double().t())
    want = torch.where(mask, h, 0.0)
    special = torch.zeros(F, dtype=torch.bool, device=DEV)
    special[[j, ju]] = True
    y64 = (want * ~special).nan_to_num(0.0) @ wd.double().nan_to_num(0.0, 0.0, 0.0)
    if relu:
        y64 += layer.b_out.double()
    for b in range(B):
        cols = torch.ones(d, dtype=torch.bool, device=DEV)
        if keep_even[b]:                                     # (the neuron j's own terms)
            assert y[b, 7] == torch.sign(h[b, j]) * float("inf") and torch.isnan(y[b, d - 1]), b
            cols[7] = cols[d - 1] = False
            r = y64[b] + h[b, j] * wd[j].double()
            assert (y[b].double() - r)[cols].norm() <= 2 ** -8 * r[cols].norm(), b
        else:
            assert (y[b] == float("inf")).all(), b
    ref = clada.sparse_ffn_stack_decode(ctx, [layer, layer, layer], torch.stack([x] * 3), tau.repeat(3, 1))
    assert all(torch.equal(r.nan_to_num(7.0), y.nan_to_num(7.0)) for r in ref)


def test_sizes_beyond_the_limits_are_rejected(clada):
    from paper_2502_19078_amd.binding import CladaError
    cfg, w, x = _case("c2", 12, 256, 64, 1)
    ctx = clada.Context(0, clada.workspace_bytes(256, 64, 64, 0, 0))
    layer = clada.Layer(*[to_dev(a, cfg.dtype) for a in w])
    xb = torch.zeros(65, 256, dtype=torch.bfloat16, device=DEV)
    with pytest.raises(CladaError):
        clada.sparse_ffn_decode(ctx, layer, xb, torch.zeros(65, device=DEV))
    small = clada.Context(0, 1024)                       # workspace too small for the call
    with pytest.raises(CladaError):
        clada.sparse_ffn_decode(small, layer, to_dev(x, cfg.dtype), torch.zeros(1, device=DEV))


def test_bounded_wait_of_the_balanced_kernel_gives_up_cleanly(clada):
    """The balanced kernel polls for the other workgroups' masks a bounded number of times.  With the
    limit forced to zero from the host nearly every workgroup gives up at once: every kernel still runs
    to its end, the output is NaN rather than a silent partial sum, and the context reports the fault."""
    cfg, w, x = _case("c2", 13, 4096, 11008, 1)
    layer = clada.Layer(*[to_dev(a, cfg.dtype) for a in w])
    xd = to_dev(x, cfg.dtype)
    td = torch.from_numpy(_tau_for(w, x, 0.45)).to(DEV)
    ctx = clada.Context(0, clada.workspace_bytes(4096, 11008, 1, 0, 0))
    ctx.set_option("decode.b1", 3)
    good = clada.sparse_ffn_decode(ctx, layer, xd, td).clone()
    assert not ctx.device_fault() and torch.isfinite(good.float()).all()
    ctx.set_option("decode.spin_limit", 0)
    bad = clada.sparse_ffn_decode(ctx, layer, xd, td)
    torch.cuda.synchronize()
    assert ctx.device_fault() and torch.isnan(bad.float()).all()
    fresh = clada.Context(0, clada.workspace_bytes(4096, 11008, 1, 0, 0))      # a new context is clean
    fresh.set_option("decode.b1", 3)
    again = clada.sparse_ffn_decode(fresh, layer, xd, td)
    torch.cuda.synchronize()
    assert not fresh.device_fault() and torch.equal(again, good)


def test_many_balanced_calls_on_one_context_stay_identical(clada):
    """The balanced kernel tags its records with an 8-bit call counter that lives on the device: more than
    256 calls on one context (the tag wraps) must keep giving the first call's bits, and the oracle's result."""
    cfg, w, x = _case("c2", 14, 4096, 11008, 1)
    tau = _tau_for(w, x, 0.45)
    layer = clada.Layer(*[to_dev(a, cfg.dtype) for a in w])
    xd, td = to_dev(x, cfg.dtype), torch.from_numpy(tau).to(DEV)
    ctx = clada.Context(0, clada.workspace_bytes(4096, 11008, 1, 0, 0))
    ctx.set_option("decode.b1", 3)
    y0, idx0, cnt0, bits0 = clada.sparse_ffn_decode(ctx, layer, xd, td, want_lists=True)
    torch.cuda.synchronize()
    _check_against_oracle(cfg, w, x, tau, y0, idx0.cpu().numpy(), cnt0.cpu().numpy(), unpack_bits(bits0, 11008),
                          "first balanced call")
    y0, idx0 = y0.clone(), idx0.clone()
    for i in range(1, 321):
        if i % 40 == 0:
            y, idx, cnt, _ = clada.sparse_ffn_decode(ctx, layer, xd, td, want_lists=True)
            assert torch.equal(idx, idx0) and torch.equal(cnt, cnt0), f"call {i}: index list changed"
        else:
            y = clada.sparse_ffn_decode(ctx, layer, xd, td)
        assert torch.equal(y, y0), f"call {i}: output bits changed"
    assert not ctx.device_fault()


# fp32 layers with d = 4096 and one or seven neurons: the shapes (and, for the first four, the very inputs)
# on which a seeded shape hunt measured 2e-5 .. 1e-4 against the oracle
FEW_NEURONS = [(2, 1, 1, 16, "silu", 0.0), (302, 20, 1, 64, "silu", 0.2), (315, 14, 7, 33, "silu", 0.95),
               (402, 3, 1, 17, "gelu_tanh", 0.95), (7, 0, 1, 16, "silu", 0.45), (7, 1, 7, 33, "silu", 0.45)]


@pytest.mark.parametrize("seed,layer,F,B,sigma,q", FEW_NEURONS)
def test_fp32_few_neurons_meet_the_bar_their_conditioning_allows(clada, seed, layer, F, B, sigma, q):
    """With a handful of neurons y inherits the relative error of single dot products, eps32 * kappa, and a
    near-cancelling up-projection dot (kappa ~ 1e4) puts it above 1e-5 in ANY fp32 evaluation (pinned on the
    CPU in test_tolerances.py).  The bar per row is 1e-5 + eps32 * kappa_row, kappa from fp64 numpy; rows
    with kappa < 150 thereby stay at (1 +- 1) e-5."""
    from paper_2502_19078_amd import binding
    cfg = synth.CONFIGS["c1"]
    d = 4096
    x = synth.decode_hidden(cfg, seed, layer, 0, B=B, d=d)
    w = synth.layer_weights(cfg, seed, layer, d=d, d_ff=F)
    act = np.abs(oracle.gate_act(w[0], x, sigma=sigma))
    tau = np.quantile(act, q, axis=1).astype(np.float32) * np.resize(np.array([1.0, 1.8, 1.12], np.float32), B)
    ctx = clada.Context(0, clada.workspace_bytes(d, F, B, 0, 0))
    layer_d = clada.Layer(*[to_dev(a, "f32") for a in w], kind=binding.GEGLU if sigma == "gelu_tanh" else binding.SWIGLU)
    xd = to_dev(x, "f32")
    worst = 0.0
    for b1 in (1, 0):                                   # split-d kernel where the shape has one, generic kernel
        ctx.set_option("decode.b1", b1)
        y, idx, cnt, bits = clada.sparse_ffn_decode(ctx, layer_d, xd, torch.from_numpy(tau).to(DEV), want_lists=True)
        yd = clada.dense_ffn_decode(ctx, layer_d, xd)
        torch.cuda.synchronize()
        mask = unpack_bits(bits, F)
        check_mask_band(mask, oracle.gate_act(w[0], x, sigma=sigma), tau.astype(np.float64), "few neurons")
        for got, m, what in ((y, mask, "sparse"), (yd, np.ones((B, F), bool), "dense twin")):
            kappa, _ = decode_condition(*w, x, m, sigma)
            ref = oracle.decode_given_mask(*w, x, m, sigma=sigma)
            assert_close_y(to_np(got), ref, TOL_Y["f32"], f"{what} b1={b1}", extra=EPS32 * kappa)
            nr = np.linalg.norm(ref, axis=1)
            rel = np.linalg.norm(to_np(got) - ref, axis=1)[nr > 0] / nr[nr > 0]
            worst = max(worst, float(rel.max()))
    print(f"[few neurons] seed={seed} F={F} B={B}: worst row {worst:.2e}")


@pytest.mark.parametrize("d,F,q", [(6144, 700, 0.45), (8192, 1030, 0.5), (8192, 14336, 0.45),
                                   (8192, 28672, 0.5),      # 70B-class layer: 112 neurons per workgroup, two rounds of the split-d kernel
                                   (1024, 40000, 0.45)])    # 157 per workgroup: three rounds
def test_rows_of_12_and_16_kib_on_the_split_d_kernel(clada, d, F, q):
    """Batch 1 at d = 6144 and 8192 (bf16): the split-d kernel with x in LDS, balanced and not, and the generic
    kernel give the same mask and, each, the oracle's output."""
    cfg, w, x = _case("c2", 15, d, F, 1)
    tau = _tau_for(w, x, q)
    layer = clada.Layer(*[to_dev(a, cfg.dtype) for a in w])
    xd, td = to_dev(x, cfg.dtype), torch.from_numpy(tau).to(DEV)
    ctx = clada.Context(0, clada.workspace_bytes(d, F, 1, 0, 0))
    masks = []
    for b1 in (1, 2, 3, 0):
        ctx.set_option("decode.b1", b1)
        y, idx, cnt, bits = clada.sparse_ffn_decode(ctx, layer, xd, td, want_lists=True)
        torch.cuda.synchronize()
        mask = unpack_bits(bits, F)
        _check_against_oracle(cfg, w, x, tau, y, idx.cpu().numpy(), cnt.cpu().numpy(), mask, f"d={d} F={F} decode.b1={b1}")
        masks.append(mask)
        yd = clada.dense_ffn_decode(ctx, layer, xd)
        assert_close_y(to_np(yd), oracle.dense_decode(*w, x), TOL_Y[cfg.dtype], f"dense twin decode.b1={b1}")
    assert all(np.array_equal(m, masks[0]) for m in masks)
    assert not ctx.device_fault()


@pytest.mark.parametrize("d,B", [(1032, 2), (3584, 5), (776, 8)])
def test_bf16_dots_of_the_vector_kernel_keep_subnormals_and_full_precision(clada, d, B):
    """Weights of 2^-129 and below (subnormal in bf16) against inputs of 2^60: every product counts.  W_down scaled so that the
    outputs are ordinary numbers; 64-bit reference, bf16 outputs (2^-9 of a value, and kept sums that cancel a little)."""
    from paper_2502_19078_amd import binding
    F = 512
    g = torch.Generator(device=DEV).manual_seed(d)
    n = lambda *s: torch.randn(s, generator=g, device=DEV, dtype=torch.float64)
    wg = (n(F, d) * 2.0 ** -129).bfloat16()
    assert (wg != 0).float().mean() > 0.9 and wg.double().abs().max() < 2.0 ** -126
    wd = (n(F, d) * 2.0 ** 60).bfloat16()
    x = (n(B, d) * 2.0 ** 60).bfloat16()
    b_in = torch.zeros(F, device=DEV)
    if d > 1280:                                             # the non-gated family: y is linear in the activation
        layer = clada.Layer(wg, None, wd, kind=binding.RELU, b_in=b_in, b_out=None)
        up = None
    else:                                                    # gated: SiLU(g) = g / 2 for such a g
        up = (n(F, d) * 0.02).bfloat16()
        wd = (n(F, d)).bfloat16()
        layer = clada.Layer(wg, up, wd)
    ctx = clada.Context(0, clada.workspace_bytes(d, F, B, 0, 0))
    y = clada.sparse_ffn_decode(ctx, layer, x, torch.zeros(B, device=DEV))
    gd = x.double() @ wg.double().t()
    h = torch.clamp_min(gd, 0.0) if up is None else 0.5 * gd * (x.double() @ up.double().t())
    want = h @ wd.double()
    assert want.abs().min() > 0 and torch.isfinite(y.float()).all()
    err = (y.double() - want).norm(dim=1) / want.norm(dim=1)
    assert float(err.max()) < 4e-3, err


@pytest.mark.parametrize("dtype,d,F", [("f32", 1028, 257), ("f32", 2048, 300), ("f32", 2052, 259), ("f32", 4096, 513),
                                       ("bf16", 1032, 300), ("bf16", 4088, 259), ("bf16", 4104, 300), ("bf16", 6152, 513)])
@pytest.mark.parametrize("kind", ["swiglu", "relu"])
def test_vector_kernel_row_requests(clada, dtype, d, F, kind):
    """Rows a little longer and shorter than whole requests, one to three rows per workgroup, through every number of tokens that has an
    instance: dense, sparse and by lists of no, one and all neurons, against float64."""
    from paper_2502_19078_amd import binding
    dt, tol = (torch.float32, TOL_Y["f32"]) if dtype == "f32" else (torch.bfloat16, 5e-3)      # bf16: y rounded once, 2^-9 of a value
    g = torch.Generator(device=DEV).manual_seed(d + F)
    w = [(torch.randn(F, d, generator=g, device=DEV) * d ** -0.5).to(dt) for _ in range(3)]
    layer = clada.Layer(w[0], None, w[2], kind=binding.RELU) if kind == "relu" else clada.Layer(*w)
    for B in (1, 2, 3, 4, 5, 8):
        x = torch.randn(B, d, generator=g, device=DEV).to(dt)
        ctx = clada.Context(0, clada.workspace_bytes(d, F, B, 0, 0))
        ctx.set_option("decode.batched", 0)
        pre = x.double() @ w[0].double().t()
        a = torch.relu(pre) if kind == "relu" else torch.nn.functional.silu(pre)
        up = x.double() @ w[1].double().t()
        h = a if kind == "relu" else a * up
        # one neuron alone: its dots' cancellation goes straight through, eps32 sum|x_i w_i| / |dot| each (sigma passes on at most 1 + |g| of it)
        kappa = lambda m, dot: (x.abs().double() @ m[0].abs().double()) / dot[:, 0].abs()
        one = EPS32 * (kappa(w[0], pre) * (1 + pre[:, 0].abs()) + (0 if kind == "relu" else kappa(w[1], up)))
        ref = lambda keep: (torch.where(keep, h, 0.0) @ w[2].double()).cpu().numpy()
        every = torch.ones_like(a, dtype=torch.bool)
        assert_close_y(to_np(clada.dense_ffn_decode(ctx, layer, x)), ref(every), tol, f"dense B={B}")
        s = a.abs().flatten().sort().values
        k = int(0.7 * len(s))
        k += int((s[k + 1:k + 33] - s[k:k + 32]).argmax())   # a gap, so that rounding decides nothing
        tau = ((s[k] + s[k + 1]) / 2).float().expand(B).contiguous()
        y = clada.sparse_ffn_decode(ctx, layer, x, tau)
        assert_close_y(to_np(y), ref(a.abs() >= tau.double()[:, None]), tol, f"sparse B={B}")
        for n in (0, 1, F):
            idx = torch.arange(F, dtype=torch.int32, device=DEV)
            y = clada.static_ffn_decode(ctx, layer, x, idx, torch.tensor([n], dtype=torch.int32, device=DEV))
            assert_close_y(to_np(y), ref(every & (torch.arange(F, device=DEV) < n)), tol, f"list of {n} B={B}",
                           one if n == 1 else None)
