"""Weight gradients of narrow heads on both sides of the line between the 4x4x1 kernel and the tiled one
(pixels times channels, csrc/igemm_wgrad_small.hip), with ragged channel counts, against the oracle."""
import pytest

from paper_2402_14139_amd import binding as nf
from tests import gpu_common as G
from tests.test_gpu_parity import S

pytestmark = pytest.mark.gpu

# name -> (spec, B, kernel of the head's weight gradient)
CASES = {
    "a12_c136_above": (S(8, 16, 16, 136, 12), 93, "wgrad_small_4x4"),
    "a4_c260_above": (S(8, 9, 7, 260, 4), 200, "wgrad_small_4x4"),
    "a8_c132_above": (S(8, 16, 16, 132, 8), 95, "wgrad_small_4x4"),
    "a12_c136_below": (S(8, 16, 16, 136, 12), 90, "igemm_wgrad_fast_32x128"),
    "a16_c64_below": (S(8, 7, 5, 64, 16), 3, "igemm_wgrad_fast_32x128"),
}


@pytest.mark.parametrize("name", list(CASES))
def test_narrow_heads_match_oracle(name):
    spec, B, kernel = CASES[name]
    print(f"case {name}: B={B}", flush=True)
    nf.nf_prof_begin()
    out, final = G.run_step_both(spec, 10, B, seed=320, lr=0.05, mu=0.9, steps=1)
    got = {r["kernel"] for r in nf.nf_prof_end()}
    G.check_step_results(name, out, final)
    assert kernel in got, got


# The line lies lower where the 4x4x1 kernel fills its lanes (few filters beside 128 channels or more) or its waves (64s)
LOWER_CASES = {
    "a8_c200_above": (S(8, 8, 8, 200, 8), 102, "wgrad_small_4x4"),
    "a8_c200_below": (S(8, 8, 8, 200, 8), 101, "igemm_wgrad_fast_32x128"),
    "a16_c64_above": (S(8, 16, 16, 64, 16), 104, "wgrad_small_4x4"),
    "a16_c64_below_1_7m": (S(8, 16, 16, 64, 16), 103, "igemm_wgrad_fast_32x128"),
    # the tiled kernel with splits of at most 192 rows: the last one short, and nearly as many as the other kernel's
    "a12_c100": (S(8, 13, 11, 100, 12), 130, "igemm_wgrad_fast_32x128"),
    "a4_c36_many_splits": (S(8, 16, 16, 36, 4), 320, "igemm_wgrad_fast_32x128"),
}


@pytest.mark.parametrize("name", list(LOWER_CASES))
def test_the_line_where_the_lanes_are_full(name):
    spec, B, kernel = LOWER_CASES[name]
    print(f"case {name}: B={B}", flush=True)
    nf.nf_prof_begin()
    out, final = G.run_step_both(spec, 10, B, seed=321, lr=0.05, mu=0.9, steps=1)
    got = {r["kernel"] for r in nf.nf_prof_end()}
    G.check_step_results(name, out, final)
    assert kernel in got, got


def test_a_narrow_layer_keeps_the_tiled_kernel():
    """A layer of 8 filters (2.1 million pixels times channels) has that kernel's splits, a head of 8 would not."""
    nf.nf_prof_begin()
    out, final = G.run_step_both(S(256, 6, 6, 8, 80), 10, 226, seed=322, lr=0.05, mu=0.9, steps=1)
    got = {r["kernel"] for r in nf.nf_prof_end()}
    G.check_step_results("narrow_layer", out, final)
    assert "wgrad_small_4x4" not in got and "igemm_wgrad_fast_32x128" in got, got
