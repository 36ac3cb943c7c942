"""Which kernels a call launches, and what a refused launch leaves behind: the library's host side on the CPU, over a runtime
that only writes the launches down (fake_hip.py)."""
import re
import shutil

import pytest

import test_gpu_cett
import test_gpu_prefix
import test_gpu_stack
from fake_hip import build_runtime, run_steps

pytestmark = pytest.mark.skipif(shutil.which("g++") is None, reason="no g++")


@pytest.fixture(scope="module")
def fake(tmp_path_factory):
    return build_runtime(tmp_path_factory.mktemp("fake_hip"))


def _names(result):
    assert result["status"] == 0, result
    return [r[0] for r in result["launches"]]


def test_a_calibration_that_was_cut_short_does_not_reach_the_next_one(fake):
    """The histograms are zero between calls only if the last kernel of a call ran: after a refused launch the next call clears
    them before it counts, and no call after that."""
    calib = {"do": "calibrate", "n": 1 << 20}
    clear = lambda r: [i for i, n in enumerate(_names(r)) if "k_calib_clear" in n]
    for refused in (0, 1, 2):                                # the first, second, third launch of the call
        r = run_steps(fake, [{"do": "ctx", "sizes": [0, 0, 0, 64, 0]}, calib, {"do": "fail", "in": refused}, calib, calib, calib])
        assert clear(r[1]) == [] and r[3]["status"] == 7     # CLADA_ERR_HIP
        assert len(r[3]["launches"]) == refused              # nothing is launched behind the refused one
        assert clear(r[4]) == [0] and clear(r[5]) == []
    # a clearing that was only recorded has not run: the next call clears again
    r = run_steps(fake, [{"do": "ctx", "sizes": [0, 0, 0, 64, 0]}, {"do": "fail", "in": 2}, calib, {"do": "capturing", "on": 1}, calib,
                   {"do": "capturing", "on": 0}, calib, calib])
    assert clear(r[4]) == [0] and clear(r[6]) == [0] and clear(r[7]) == []


def test_search_forms_the_mean_once_per_probe_above_1024_tokens(fake):
    """In place (every workgroup reads all tokens' norms) only up to 1024 tokens, where a table answers the search first and what it leaves open is
    measured three steps of the bisection a launch: 31 steps and the one that takes in the last are eleven launches, an even number twelve."""
    d, F = 1024, 4096
    r = run_steps(fake, [{"do": "ctx", "sizes": [d, F, 0, 1025, 0]}] + [{"do": "search", "d": d, "F": F, "T": T} for T in (1024, 1025)])
    count = lambda res, name: sum(name in n for n in _names(res))
    assert (count(r[1], "k_cett_between"), count(r[1], "k_cett_take")) == (12, 0)
    assert (count(r[2], "k_cett_between"), count(r[2], "k_cett_take")) == (32, 31)


@pytest.mark.parametrize("T,d,F,dtype,large", [
    (4096, 256, 512, "bf16", True), (4097, 256, 512, "bf16", False), (16384, 64, 512, "bf16", False), (65536, 256, 1024, "bf16", False),
    (65536, 64, 2048, "bf16", True), (16384, 64, 512, "f32", True), (2048, 520, 512, "bf16", False), (2047, 512, 512, "bf16", False),
])
def test_search_over_many_tokens_of_a_narrow_layer_is_the_plain_bisection(fake, T, d, F, dtype, large):
    """A probe inside the bracket costs a workgroup per token, which a bf16 projection of a few hundred neurons does not."""
    r = run_steps(fake, [{"do": "ctx", "sizes": [d, F, 0, T, 0]}, {"do": "search", "d": d, "F": F, "T": T, "dtype": dtype}])
    assert any("k_cett_between" in n for n in _names(r[1])) == large


@pytest.mark.parametrize("d,F,T,dtype,room,want", [
    # parts per launch (1: or all of them by the same workgroups) in a workspace with `room` times [T][d] behind h (0: the smallest that the call accepts), and the launches that add up
    (1024, 4096, 16, "bf16", 12, ([12], 1)), (1024, 4096, 16, "bf16", 11, ([11, 1], 2)), (1024, 4096, 16, "bf16", 0, ([10, 2], 2)),
    (512, 3333, 100, "bf16", 0, ([3] * 4, 4)), (512, 3333, 100, "bf16", 5, ([5, 5, 2], 3)), (512, 3333, 100, "bf16", 100, ([12], 1)),
    (1024, 2111, 100, "bf16", 0, ([1], 1)), (1024, 2111, 100, "bf16", 2, ([2] * 4, 4)),
    (1024, 1919, 64, "bf16", 100, ([1], 0)), (260, 3001, 40, "f32", 0, ([1], 1)), (260, 3001, 40, "f32", 3, ([3, 3, 3, 2], 4)),
    (260, 3001, 40, "f32", 11, ([11], 1)),
])
def test_parts_of_the_down_projection_by_the_room_there_is(fake, d, F, T, dtype, room, want):
    up = lambda n: (n + 255) // 256 * 256
    es, Fp, tiles = 4 if dtype == "f32" else 2, -(-F // 64) * 64, -(-T // 128) * -(-d // (256 if dtype == "bf16" else 128))
    part = up(-(-T // 128) * 16 * F)
    least = part + up(T * Fp * 4) + (8 * 4 * T * d if (F % 32, d % 256) == (0, 0) else 0)
    step = {"do": "prefix", "d": d, "F": F, "T": T, "dtype": dtype}
    assert run_steps(fake, [{"do": "ctx", "bytes": least - 256}, step])[1]["status"] == 5      # CLADA_ERR_WORKSPACE
    r = run_steps(fake, [{"do": "ctx", "bytes": part + up(T * Fp * es) + room * 4 * T * d if room else least}, step])[1]
    down = [x[1] for x in r["launches"] if "k_prefix_down" in x[0] and "combine" not in x[0]]
    assert r["status"] == 0 and down == [-(-tiles * n // 8) * 8 for n in want[0]]      # (padded to a multiple of eight workgroups)
    assert sum("combine" in n for n in _names(r)) == want[1]


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("d,F,T", [(260, 3001, 90), (512, 3333, 100), (1024, 4096, 16), (2048, 8191, 200), (4096, 9001, 64), (1024, 1919, 64), (8192, 20011, 300)])
def test_the_advised_workspace_holds_all_parts_of_either_type(fake, d, F, T, dtype):
    if d == 8192 and dtype == "f32":
        d = 4096                                             # (the widest fp32 row)
    if d % 8 and dtype == "bf16":
        d = 264
    for tile in (0, 1, 2):
        r = run_steps(fake, [{"do": "ctx", "sizes": [d, F, 0, T, 0]}, {"do": "option", "name": "prefix.tile", "value": tile}]
                      + [{"do": do, "d": d, "F": F, "T": T, "dtype": dtype, "kind": kind} for do in ("prefix", "search") for kind in ("swiglu", "relu")])
        for x in r[2:]:
            down = [n for n in _names(x) if "k_prefix_down" in n and "combine" not in n]
            assert down and not any("Lb1ELb1E" in n for n in down), down      # (the instances that form some parts at a time)


def _stack_grid(r):
    """[(partial outputs per layer, layers)] of the launches over several layers; None if the call ran another way."""
    names = _names(r)
    if not all("k_ffn_stack" in n and "persistent" not in n for n in names):
        return None
    return [tuple(x[1:3]) for x in r["launches"] if "k_ffn_stack_reduce" not in x[0]]


@pytest.mark.parametrize("d,F,L,kw,want", [
    # rounds of eight layers as whole slices (32 workgroups a layer), the thin rest as single classes
    (4096, 11008, 8, {}, [(32, 8)]), (4096, 11008, 9, {}, [(32, 8), (256, 1)]), (4096, 11008, 11, {}, [(32, 8), (256, 3)]),
    (4096, 11008, 12, {}, [(32, 12)]), (4096, 11008, 17, {}, [(32, 16), (256, 1)]), (4096, 11008, 32, {}, [(32, 32)]),
    (4096, 11008, 50, {}, [(32, 48), (256, 2)]), (4096, 11008, 54, {}, [(32, 48), (32, 6)]), (4096, 11008, 5, {}, [(32, 5)]),
    (4096, 11008, 4, {}, [(256, 4)]), (2560, 10240, 10, {"kind": "relu"}, [(32, 8), (256, 2)]), (2560, 10240, 5, {}, [(256, 5)]),
    (2560, 10240, 12, {}, [(32, 8), (256, 4)]), (2560, 10240, 13, {}, [(32, 13)]),
    (2048, 16384, 10, {}, [(32, 10)]), (2048, 16384, 17, {}, [(32, 16), (256, 1)]), (2048, 16384, 18, {}, [(32, 16), (256, 2)]),
    (2048, 8192, 7, {}, [(256, 4), (256, 3)]), (1024, 4096, 17, {}, [(32, 17)]), (1024, 4096, 7, {}, [(256, 4), (256, 3)]),
    (2048, 5504, 9, {"dtype": "f32"}, [(32, 8), (256, 1)]), (5120, 13824, 33, {}, [(32, 32), (256, 1)]),
    # the lanes' side of the rule
    (5120, 13824, 5, {}, None), (5120, 13824, 6, {}, [(32, 6)]), (5120, 5120, 4, {}, [(256, 4)]), (5120, 5120, 5, {"dense": True}, None),
    (4096, 11008, 9, {"dense": True}, None), (4096, 11008, 8, {"dense": True}, [(32, 8)]), (4096, 8192, 9, {"dense": True}, [(32, 8), (256, 1)]),
    (4096, 16384, 9, {"dense": True, "kind": "relu"}, [(32, 8), (256, 1)]), (2048, 16384, 9, {"dense": True}, None),
    (2048, 12288, 9, {"dense": True}, [(32, 9)]), (6144, 12288, 9, {}, None), (512, 1376, 3, {"dtype": "f32"}, [(256, 3)]),
])
def test_batch_1_stacks_fill_their_rounds(fake, d, F, L, kw, want):
    r = run_steps(fake, [{"do": "ctx", "sizes": [d, F, 1, 0, 0]}, dict({"do": "stack", "d": d, "F": F, "L": L, "B": 1}, **kw)])
    assert _stack_grid(r[1]) == want


@pytest.mark.parametrize("dtype,widths", [("bf16", (64, 512, 768, 1024, 1536, 2048, 2560, 3072, 3584, 4096, 5120, 6144, 7168, 8192)),
                                          ("f32", (32, 256, 512, 768, 1024, 1536, 2048, 2560, 3072, 4096))])
@pytest.mark.parametrize("kind", ["swiglu", "relu", "geglu"])
def test_no_stack_or_call_is_refused(fake, dtype, widths, kind):
    """Every row length there is a kernel for, in every mode: a rule that admits a shape has an instance for it in both families."""
    steps = []
    for d in widths:
        for F in (200, 300, 20000):
            steps += [{"do": "ctx", "sizes": [d, F, 16, 0, 0]}]
            for mode in (3, 2, 1, 0):
                steps += [{"do": "option", "name": "decode.stack", "value": mode}]
                steps += [{"do": "stack", "d": d, "F": F, "L": L, "B": B, "kind": kind, "dtype": dtype, "dense": dense}
                          for L in (1, 2, 9) for B in (1, 2, 16) for dense in (False, True)]
            steps += [{"do": "decode", "d": d, "F": F, "B": B, "kind": kind, "dtype": dtype} for B in (1, 5, 12)]
    assert [(s, r["status"]) for s, r in zip(steps, run_steps(fake, steps)) if r["status"] != 0] == []


@pytest.mark.parametrize("first", [{"d": 4096, "F": 11008, "L": 8, "B": 1}, {"d": 4096, "F": 11008, "L": 8, "B": 4}, {"d": 1024, "F": 300, "L": 1, "B": 1}])
def test_first_stack_call_makes_the_lanes_whichever_way_it_takes(fake, first):
    """A capture must not have to create streams: not one that needs the lanes after a first call that did not."""
    lanes = [{"d": 6144, "F": 12288, "L": 5, "B": 1}, {"d": 5120, "F": 13824, "L": 40, "B": 16}]
    r = run_steps(fake, [{"do": "ctx", "sizes": [6144, 13824, 16, 0, 0]}, dict({"do": "stack"}, **first), {"do": "capturing", "on": 1}]
                  + [dict({"do": "stack"}, **kw) for kw in lanes])
    assert r[1]["created"] == 6 and r[3]["created"] == r[4]["created"] == 0
    assert len(r[3]["launches"]) == 2 * 5 and _batched_layers(r[4]) is None        # (they do go round the lanes)
    # a first call that is captured creates nothing it does not need
    r = run_steps(fake, [{"do": "ctx", "sizes": [4096, 11008, 4, 0, 0]}, {"do": "capturing", "on": 1}, dict({"do": "stack"}, **first)])
    assert r[2]["created"] == 0


def _row(mod, name):
    return [pytest.param(*r, id="-".join(map(str, r))) for r in getattr(mod, name)]


@pytest.mark.parametrize("d,F,L,relu,dtype", _row(test_gpu_stack, "ONE_LAUNCH"))
def test_the_device_tests_of_one_launch_take_it(fake, d, F, L, relu, dtype):
    r = run_steps(fake, [{"do": "ctx", "sizes": [d, F, 1, 0, 0]}, {"do": "option", "name": "decode.b1", "value": 2}]
                  + [{"do": "stack", "d": d, "F": F, "L": L, "B": 1, "kind": "relu" if relu else "swiglu", "dtype": dtype, "dense": x} for x in (False, True)])
    assert _stack_grid(r[2]) is not None
    # (the dense twin of the same row may go round the lanes: few layers of 10 KiB rows, large ones of 4 KiB)
    assert _stack_grid(r[3]) is not None or (d, L < 6) == (5120, True) or (d, F > 12288) == (2048, True)


@pytest.mark.parametrize("d,F,L,relu,B,dense,occ2", _row(test_gpu_stack, "LANES"))
def test_the_device_tests_of_the_lanes_take_them(fake, d, F, L, relu, B, dense, occ2):
    """A gate/up launch per layer and pass, of the two-per-unit instance where it is asked for and the layer is short enough."""
    r = run_steps(fake, [{"do": "ctx", "sizes": [d, F, B, 0, 0]}, {"do": "option", "name": "decode.lane_occ2", "value": occ2}]
                  + [{"do": "stack", "d": d, "F": F, "L": L, "B": B, "kind": "relu" if relu else "swiglu", "dense": dense}])
    main = [n for n in _names(r[2]) if ("k_bat_gateup" if B > 1 else "k_ffn_decode_b1") in n]
    assert len(main) == L * -(-B // 16) and all(x[3] == 1 for x in r[2]["launches"])
    if B == 1:
        two = dense and not relu and d in (2048, 4096) and occ2 == 1 and F <= 64 * 256
        assert r[2]["created"] == 6 and len(set(main)) == 1
        # (the instance's last template flag)
        assert ("Lb0ELb0ELb0ELb0ELb1EEEv" in main[0]) == two, main[0]


@pytest.mark.parametrize("d,F,L", test_gpu_stack.GRAPH_SHAPES)
def test_the_device_tests_of_captures_take_both_ways(fake, d, F, L):
    r = run_steps(fake, [{"do": "ctx", "sizes": [d, F, 1, 0, 0]}, {"do": "stack", "d": d, "F": F, "L": L, "B": 1}])
    assert (_stack_grid(r[1]) is None) == (d == 6144)


def test_the_device_tests_of_bracketed_searches_bracket(fake):
    """All of them, with one, three and seven thresholds a launch (the kernel's last template number is the steps: 1, 2, 3)."""
    steps = set()
    for d, F, T, dtype in test_gpu_cett.PER_LAUNCH:
        r = run_steps(fake, [{"do": "ctx", "sizes": [d, F, 0, T, 0]}, {"do": "search", "d": d, "F": F, "T": T, "dtype": dtype}])
        between = {n for n in _names(r[1]) if "k_cett_between" in n}
        assert len(between) == 1, (d, F, T, dtype)
        steps.add(between.pop().split("k_cett_betweenI")[1].split("Li")[3][0])
    assert steps == {"1", "2", "3"}


def test_the_device_tests_of_padded_columns_take_every_tile(fake):
    """Which gate/up kernel each of them runs; the first ten are there for tiles of 96 neurons (three pairs of 16 for each of two waves)."""
    seen = []
    for d, F, T, kind, tile in test_gpu_prefix.PADDED:
        step = {"do": "prefix", "d": d, "F": F, "T": T, "kind": "swiglu" if kind == "f32" else kind, "dtype": "f32" if kind == "f32" else "bf16"}
        r = run_steps(fake, [{"do": "ctx", "sizes": [d, F, 0, T, 0]}, {"do": "option", "name": "prefix.tile", "value": tile}, step])
        seen.append([n for n in _names(r[2]) if "k_prefix_gateup" in n][0])
    is_ = lambda n, wm, nb, single: f"TileShapeILi{wm}ELi{nb}E" in n and f"ELb{single}EEEvNS_" in n
    assert all(is_(n, 4, 3, 0) for n in seen[:10])
    # 64, 128 and 256 neurons, gated and not; the plain kernel in both types
    for want in ((2, 1, 0), (2, 2, 0), (2, 1, 1), (4, 4, 0), (4, 4, 1)):
        assert any(is_(n, *want) for n in seen[10:]), (want, seen)
    assert {n.split("k_prefix_gateupI")[1][:4] for n in seen if "k_prefix_gateupI" in n} == {"Li2E", "Li4E"}


def _batched_layers(r):
    """Layers of the batched launches over several layers; None if the units went round the lanes (a layer per launch)."""
    z = [x[3] for x in r["launches"] if "k_bat_down" in x[0]]
    _names(r)
    return z if z and max(z) > 1 else None


@pytest.mark.parametrize("d,F,L,B,kw,want", [
    (4096, 14336, 32, 8, {}, [32]), (4096, 11008, 40, 16, {}, [20, 20]), (5120, 13824, 20, 16, {}, [20]), (5120, 13824, 40, 2, {}, [40]),
    (5120, 5120, 40, 32, {}, [20, 20]), (2048, 2048, 50, 2, {}, [25, 25]), (4096, 900, 7, 33, {}, [7]), (1024, 2048, 20, 64, {}, [7, 7, 6]),
    # long stacks of large layers stay with the lanes
    (5120, 13824, 40, 16, {}, None), (4096, 16384, 40, 16, {}, None), (4096, 16384, 20, 32, {}, None), (5120, 20480, 40, 16, {"kind": "relu"}, None),
    (4096, 16384, 40, 4, {}, [20, 20]), (4096, 16384, 40, 5, {}, None), (4096, 16384, 20, 16, {"dense": True}, [20]),
])
def test_batched_stacks_are_launched_over_many_layers(fake, d, F, L, B, kw, want):
    r = run_steps(fake, [{"do": "ctx", "sizes": [d, F, B, 0, 0]}, dict({"do": "stack", "d": d, "F": F, "L": L, "B": B}, **kw)])
    assert _batched_layers(r[1]) == want


@pytest.mark.parametrize("d,F,L,B,lanes", [
    # row groups of a lone pass (CG: column groups of 256): 42 doubled, 18 doubled, 24, 20, 12 and 10 doubled twice or three times, at 16 tokens a pass and fewer
    (1536, 76000, 20, 13, False), (1536, 76000, 20, 12, True), (1536, 84000, 18, 16, False), (3584, 66000, 12, 15, False), (3584, 66000, 12, 14, True), (3584, 73000, 20, 32, False),
    (2560, 100000, 9, 16, False), (3072, 82000, 9, 16, False), (5120, 99000, 5, 16, False), (5120, 80000, 6, 16, True), (5120, 99000, 8, 10, True),
    (6144, 90000, 5, 16, False), (8192, 70000, 5, 16, True), (4096, 130000, 5, 16, True),
])
def test_a_lane_holds_the_partial_outputs_of_its_units(fake, d, F, L, B, lanes):
    """64 x 16 rows of partial outputs lie in front of a lane's h; a unit that has more of them does not go round the lanes."""
    r = run_steps(fake, [{"do": "ctx", "sizes": [d, F, B, 0, 0]}, {"do": "stack", "d": d, "F": F, "L": L, "B": B}])
    per_pass = -(-B // -(-B // 16))
    for x in r[1]["launches"]:
        if x[5] and "k_bat_down" in x[0]:
            assert x[1] // -(-d // 256) * per_pass <= 64 * 16, x
    assert any(x[5] for x in r[1]["launches"]) == lanes and _batched_layers(r[1]) is None
    assert len([n for n in _names(r[1]) if "k_bat_gateup" in n]) == L * -(-B // 16)


def test_a_single_unit_has_kernels_of_its_own(fake):
    """Lone batched calls, and the units that go round the lanes, take their parameters directly; launches over several units
    take the arrays of their layers' weights."""
    r = run_steps(fake, [{"do": "ctx", "sizes": [5120, 13824, 16, 0, 0]}, {"do": "decode", "d": 4096, "F": 11008, "B": 16},
                   {"do": "stack", "d": 5120, "F": 13824, "L": 40, "B": 16}, {"do": "stack", "d": 4096, "F": 11008, "L": 3, "B": 4}])
    for res, args in ((r[1], "BatParams"), (r[2], "BatParams"), (r[3], "BatArgs")):
        bat = [n for n in _names(res) if "k_bat_gateup" in n or "k_bat_down" in n]
        assert bat and all(args in n for n in bat), bat[:2]


@pytest.mark.parametrize("d,F,B,tiles", [
    # 16 tokens a pass, or 32 in two tiles: from 17 tokens on, up to 4096 values and 16 d neurons; passes of nearly equal size
    (1024, 777, 16, [1]), (1024, 777, 17, [2]), (1024, 16384, 31, [2]), (1024, 16385, 20, [1, 1]), (2048, 300, 33, [2, 2]), (2560, 900, 49, [2, 2]),
    (3072, 500, 32, [2]), (4096, 255, 48, [2, 2]), (4096, 65536, 17, [2]), (5120, 900, 17, [1, 1]), (4096, 900, 64, [2, 2]), (4096, 900, 65, None),
    # the narrow and the odd widths, from the batch on that the matrix cores take
    (512, 600, 11, []), (512, 600, 12, [1]), (512, 1700, 32, [2]), (768, 900, 5, []), (768, 900, 6, [1]), (768, 3072, 33, [2, 2]), (1536, 3839, 4, []),
    (1536, 3840, 4, [1]), (1536, 2000, 31, [2]), (3584, 500, 2, []), (3584, 500, 3, [1]), (3584, 700, 33, [2, 2]),
    # the widest layers in two tiles, and one neuron past them
    (512, 8192, 32, [2]), (512, 8193, 32, [1, 1]), (768, 12288, 32, [2]), (1024, 16384, 32, [2]), (1536, 24576, 32, [2]), (2048, 32768, 32, [2]), (2560, 40960, 32, [2]),
    (3072, 49152, 32, [2]), (3584, 57344, 32, [2]), (3584, 57345, 32, [1, 1]), (4096, 65536, 32, [2]),
])
def test_passes_and_tiles_of_the_matrix_core_path(fake, d, F, B, tiles):
    """The instances by the mangled tail of their parameters: k_bat_gateup<.., tiles, Args>, k_bat_down<tiles, ..>."""
    r = run_steps(fake, [{"do": "ctx", "sizes": [d, F, min(B, 64), 0, 0]}, {"do": "decode", "d": d, "F": F, "B": B}])[1]
    if tiles is None:
        assert r["status"] != 0 and r["launches"] == []
        return
    up = [int(re.search(r"ELi([12])EN", n)[1]) for n in _names(r) if "k_bat_gateup" in n]
    down = [int(re.search(r"k_bat_downILi([12])E", n)[1]) for n in _names(r) if "k_bat_down" in n]
    assert r["status"] == 0 and up == down == tiles
    # two tiles: a pass's partial outputs, row groups x tokens, have 64 x 32 rows in front of its h
    for x in r["launches"]:
        assert "k_bat_downILi2E" not in x[0] or x[1] // -(-d // 256) * -(-B // len(tiles)) <= 64 * 32, x


@pytest.mark.parametrize("d,F,T,dtype,ladder,bisect", [
    # rows of one, two and up to four groups of 256 x 16 bytes; eight, four, two threads and one a token
    (512, 1200, 70, "f32", (4, 1, 256), 8), (768, 1500, 64, "bf16", (2, 1, 256), 8), (520, 2300, 128, "bf16", (2, 1, 256), 8), (1024, 2100, 129, "bf16", (2, 1, 256), 4),
    (2056, 2100, 256, "bf16", (2, 1, 512), 4), (512, 1100, 257, "bf16", (2, 1, 256), 2), (512, 1100, 512, "bf16", (2, 1, 256), 2), (512, 1100, 513, "bf16", (2, 1, 256), 1),
    (6144, 6200, 64, "bf16", (2, 2, 512), 8), (1028, 2100, 130, "f32", (4, 1, 512), 4), (3072, 3100, 100, "f32", (4, 2, 512), 8), (4096, 11008, 512, "bf16", (2, 1, 512), 2),
    # the narrowest window that is one (10 places of the sample: 29 entries of 44, 58 of 88, 117 of 176, 170 of 256), and past it; more tokens than a table has
    (256, 11878, 900, "bf16", (2, 1, 256), 1), (256, 11879, 900, "bf16", None, None), (4096, 23756, 300, "bf16", (2, 1, 512), 2), (4096, 23757, 300, "bf16", None, None),
    (512, 2100, 1024, "bf16", (2, 1, 256), 1), (512, 2100, 1025, "bf16", None, None),
])
def test_a_search_over_a_table_where_it_is_wide_enough(fake, d, F, T, dtype, ladder, bisect):
    r = run_steps(fake, [{"do": "ctx", "sizes": [d, F, 0, T, 0]}, {"do": "search", "d": d, "F": F, "T": T, "dtype": dtype}])[1]
    assert r["status"] == 0 and any("k_cett_curve" in n for n in _names(r))
    assert [tuple(map(int, re.search(r"k_cett_ladderILi(\d)ELi(\d)ELi(\d+)E", n).groups())) for n in _names(r) if "k_cett_ladder" in n] == [ladder] * 2 * (ladder is not None)
    assert [int(re.search(r"k_cett_bisectILi(\d)E", n)[1]) for n in _names(r) if "k_cett_bisect" in n] == [bisect] * 2 * (bisect is not None)


@pytest.mark.parametrize("d,F,B,dtype,kind,multi", [
    # rows of more than 1024 values
    (3584, 7168, 2, "bf16", "swiglu", True), (3584, 7168, 2, "bf16", "relu", True), (1032, 300, 2, "bf16", "swiglu", True),
    (1280, 3072, 2, "bf16", "relu", False), (1296, 3072, 2, "bf16", "relu", True), (1032, 3072, 3, "bf16", "relu", True),
    (1536, 3072, 4, "bf16", "relu", True), (1536, 3072, 5, "bf16", "relu", False), (1536, 3072, 9, "bf16", "relu", False), (4360, 400, 5, "bf16", "swiglu", True), (1028, 2000, 2, "f32", "geglu", True),
    # shorter rows: passes that are full enough, but bf16 ones of 768 values, whose fuller passes the matrix cores take
    (768, 3072, 4, "bf16", "swiglu", False), (768, 3072, 5, "bf16", "swiglu", True), (768, 3072, 8, "bf16", "swiglu", False),
    (768, 3072, 9, "bf16", "swiglu", False), (768, 3072, 16, "bf16", "swiglu", False), (776, 3072, 8, "bf16", "swiglu", True), (768, 3072, 8, "bf16", "relu", False), (1024, 4096, 2, "f32", "swiglu", False),
    (1024, 4096, 3, "f32", "swiglu", True), (1024, 4096, 9, "f32", "swiglu", True), (768, 4096, 9, "f32", "swiglu", False),
    (768, 4096, 33, "f32", "swiglu", True), (1024, 4096, 4, "f32", "relu", True), (1024, 4096, 5, "f32", "relu", False),
    # 512 values and fewer, fewer neurons than workgroups
    (512, 49152, 8, "bf16", "swiglu", False), (512, 2048, 4, "f32", "swiglu", False), (1536, 255, 8, "bf16", "swiglu", False),
    # one token
    (2052, 300, 1, "f32", "swiglu", True), (2052, 300, 1, "f32", "relu", False), (3584, 7168, 1, "bf16", "swiglu", False),
])
def test_decode_of_several_tokens_takes_the_faster_kernel(fake, d, F, B, dtype, kind, multi):
    r = run_steps(fake, [{"do": "ctx", "sizes": [d, F, B, 0, 0]}, {"do": "decode", "d": d, "F": F, "B": B, "dtype": dtype, "kind": kind}])
    assert any("k_ffn_multi" in n for n in _names(r[1])) == multi
    if (d, kind, dtype) in ((768, "swiglu", "bf16"), (1536, "relu", "bf16")) and B > 4:      # (the other side of the rule: the matrix cores)
        assert any("k_bat_gateup" in n for n in _names(r[1])) != multi


@pytest.mark.parametrize("d,dtype,kind,stack", [
    # every row length that only the launches over many layers take in a stack, and neighbours of theirs that the generic kernel runs either way
    (512, "bf16", "swiglu", True), (512, "bf16", "relu", True), (1536, "bf16", "relu", True), (2048, "bf16", "relu", True), (3072, "bf16", "geglu", True),
    (3072, "bf16", "relu", True), (3584, "bf16", "swiglu", True), (3584, "bf16", "relu", True), (6144, "bf16", "relu", True), (768, "f32", "swiglu", True),
    (1536, "bf16", "swiglu", False), (768, "f32", "relu", False), (1024, "f32", "geglu", False), (1536, "f32", "swiglu", False),
])
def test_a_lone_layer_is_the_batch_1_kernel_where_its_stack_is_one_launch(fake, d, dtype, kind, stack):
    """A stack has the bits of its layers' lone calls: single classes of 256 workgroups, never balanced, up to 1024 neurons a workgroup."""
    for F, dense in ((256, False), (16000, False), (60000, False), (60000, True), (255, False)):
        step = {"d": d, "F": F, "B": 1, "dtype": dtype, "kind": kind, "dense": dense}
        r = run_steps(fake, [{"do": "ctx", "sizes": [d, F, 1, 0, 0]}, dict(step, do="decode"), dict(step, do="stack", L=3)])
        assert any("k_ffn_decode_b1" in n for n in _names(r[1])) == (stack and F >= 256)
        assert [x[1] for x in r[1]["launches"] if "k_ffn_decode_b1" in x[0]] == [256] * (stack and F >= 256)
        assert (_stack_grid(r[2]) is not None) == (stack and F >= 256)


@pytest.mark.parametrize("d,F,T,kind,tiles,spare", [
    # gated, 128-token tiles (2 x neurons / 128), the units that are left take the norms of at most 16 + d / 64 rows a wave
    (4096, 11008, 129, "swiglu", 176, 80), (4096, 12288, 256, "swiglu", 192, 64), (4096, 14336, 129, "swiglu", 224, 0),
    (1024, 14336, 200, "swiglu", 224, 0), (1024, 12288, 200, "swiglu", 192, 0), (1024, 10240, 200, "swiglu", 160, 96),
    (5120, 13824, 129, "swiglu", 216, 0),
    # 256-token tiles, 24 + d / 32 rows, at most 57
    (4096, 11008, 512, "swiglu", 176, 80), (4096, 14336, 512, "swiglu", 224, 0), (512, 12288, 300, "swiglu", 192, 0),
    (512, 11264, 300, "swiglu", 176, 80), (5120, 13824, 384, "swiglu", 216, 0),
    # the non-gated family: one operand, 20 + d / 128 rows; tiles of 256 tokens x 256 neurons
    (2560, 10240, 129, "relu", 160, 96), (2560, 12288, 129, "relu", 192, 0), (4096, 12288, 129, "relu", 192, 64),
    (2048, 13312, 513, "relu", 160, 96),
])
def test_prefill_norms_on_spare_units_only_where_they_are_done_in_time(fake, d, F, T, kind, tiles, spare):
    r = run_steps(fake, [{"do": "ctx", "sizes": [d, F, 0, T, 0]}, {"do": "prefix", "d": d, "F": F, "T": T, "kind": kind}])
    assert [x[1] for x in r[1]["launches"] if "k_prefix_gateup" in x[0]] == [tiles + spare]
