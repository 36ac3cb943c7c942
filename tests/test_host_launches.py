"""Which kernels a call launches, and what a refused launch leaves behind: the library's host side on the CPU, over a runtime
that only writes the launches down (fake_hip.py)."""
import shutil

import pytest

from fake_hip import run_steps

pytestmark = pytest.mark.skipif(shutil.which("g++") is None, reason="no g++")


def _names(result):
    assert result["status"] == 0, result
    return [r[0] for r in result["launches"]]


def test_a_calibration_that_was_cut_short_does_not_reach_the_next_one(tmp_path):
    """The histograms are zero between calls only if the last kernel of a call ran: after a refused launch the next call clears
    them before it counts, and no call after that."""
    calib = {"do": "calibrate", "n": 1 << 20}
    clear = lambda r: [i for i, n in enumerate(_names(r)) if "k_calib_clear" in n]
    for refused in (0, 1, 2):                                # the first, second, third launch of the call
        r = run_steps([{"do": "ctx", "sizes": [0, 0, 0, 64, 0]}, calib, {"do": "fail", "in": refused}, calib, calib, calib], tmp_path)
        assert clear(r[1]) == [] and r[3]["status"] == 7     # CLADA_ERR_HIP
        assert len(r[3]["launches"]) == refused              # nothing is launched behind the refused one
        assert clear(r[4]) == [0] and clear(r[5]) == []
    # a clearing that was only recorded has not run: the next call clears again
    r = run_steps([{"do": "ctx", "sizes": [0, 0, 0, 64, 0]}, {"do": "fail", "in": 2}, calib, {"do": "capturing", "on": 1}, calib,
                   {"do": "capturing", "on": 0}, calib, calib], tmp_path)
    assert clear(r[4]) == [0] and clear(r[6]) == [0] and clear(r[7]) == []


def test_search_forms_the_mean_once_per_probe_above_1024_tokens(tmp_path):
    """In place (every workgroup reads all tokens' norms) only up to 1024 tokens."""
    d, F = 1024, 4096
    r = run_steps([{"do": "ctx", "sizes": [d, F, 0, 1025, 0]}] + [{"do": "search", "d": d, "F": F, "T": T} for T in (1024, 1025)], tmp_path)
    count = lambda res, name: sum(name in n for n in _names(res))
    assert (count(r[1], "k_cett_between"), count(r[1], "k_cett_take")) == (32, 0)
    assert (count(r[2], "k_cett_between"), count(r[2], "k_cett_take")) == (32, 31)


@pytest.mark.parametrize("T,d,F,dtype,large", [
    (4096, 256, 512, "bf16", True), (4097, 256, 512, "bf16", False), (16384, 64, 512, "bf16", False), (65536, 256, 1024, "bf16", False),
    (65536, 64, 2048, "bf16", True), (16384, 64, 512, "f32", True), (2048, 520, 512, "bf16", False), (2047, 512, 512, "bf16", False),
])
def test_search_over_many_tokens_of_a_narrow_layer_is_the_plain_bisection(tmp_path, T, d, F, dtype, large):
    """A probe inside the bracket costs a workgroup per token, which a bf16 projection of a few hundred neurons does not."""
    r = run_steps([{"do": "ctx", "sizes": [d, F, 0, T, 0]}, {"do": "search", "d": d, "F": F, "T": T, "dtype": dtype}], tmp_path)
    assert any("k_cett_between" in n for n in _names(r[1])) == large
