"""Heads of 256 and more features in one launch after the pooling or in two (csrc/head.hip, head_wide_applicable): both sides of the
choice, both poolings and losses, against the oracle."""
import pytest

from paper_2402_14139_amd import binding as nf
from tests import gpu_common as G
from tests.test_gpu_parity import S

pytestmark = pytest.mark.gpu

# name -> (spec, B, classes, one launch)
CASES = {
    "f240_c100": (S(8, 16, 16, 16, 60), 6, 100, False),
    "f256_c100_one_sample": (S(8, 6, 6, 16, 64), 1, 100, True),
    "f256_c100_many_samples": (S(8, 12, 12, 16, 64), 128, 100, True),
    "f256_c16_two_to_a_unit": (S(8, 16, 16, 16, 64), 32, 16, True),
    "f256_c17_two_to_a_unit": (S(8, 16, 16, 16, 64), 32, 17, False),
    "f292_c60_odd_filters": (S(8, 7, 7, 16, 73), 3, 60, True),
    "f320_c201": (S(8, 16, 16, 16, 80), 7, 201, True),
    "f320_c150_odd_map": (S(8, 13, 11, 16, 80), 9, 150, True),
    "f512_c37_ten_samples": (S(8, 14, 14, 16, 128), 10, 37, True),
    "f512_c37_thirty_samples": (S(8, 14, 14, 16, 128), 30, 37, False),
    "f1008_c24": (S(8, 16, 16, 16, 252), 9, 24, False),
    "f1008_c200": (S(8, 16, 16, 16, 252), 9, 200, True),
    "f1024_c1024": (S(8, 2, 2, 16, 256), 2, 1024, True),
    "f1024_c1025": (S(8, 2, 2, 16, 256), 2, 1025, False),
    "f1028_c200": (S(8, 2, 2, 16, 257), 2, 200, False),
}


@pytest.mark.parametrize("name", list(CASES))
@pytest.mark.parametrize("pmax,mse", [(0, 0), (1, 1)])
def test_the_line_of_one_launch(name, pmax, mse):
    spec, B, cls, one = CASES[name]
    print(f"case {name} head_pool={pmax}", flush=True)
    nf.nf_prof_begin()
    out, final = G.run_step_both(spec, cls, B, seed=370, lr=0.05, mu=0.9, steps=1, head_pool=pmax, loss_kind=mse)
    got = {r["kernel"] for r in nf.nf_prof_end()}
    G.check_step_results(name, out, final)
    assert ("head_wide" in got) == one, got
