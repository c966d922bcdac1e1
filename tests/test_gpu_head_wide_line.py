"""Heads of more than 16 384 weights in one launch (csrc/head.hip, head_wide_applicable): both sides of each line of the rule, both
poolings and losses, against the oracle."""
import pytest

from paper_2402_14139_amd import binding as nf
from tests import gpu_common as G
from tests.test_gpu_parity import S

pytestmark = pytest.mark.gpu

# name -> (spec, B, classes, one launch)
CASES = {
    "f256_c100_one_sample": (S(8, 6, 6, 16, 64), 1, 100, True),
    "f240_c100": (S(8, 16, 16, 16, 60), 6, 100, False),
    "f256_c100_many_samples": (S(8, 12, 12, 16, 64), 128, 100, True),
    "f256_c99": (S(8, 16, 16, 16, 64), 5, 99, False),
    "f320_c200": (S(8, 16, 16, 16, 80), 7, 200, True),
    "f320_c201": (S(8, 16, 16, 16, 80), 7, 201, False),
    "f336_c100": (S(8, 12, 12, 16, 84), 6, 100, False),
    "f256_c100_map_17x16": (S(8, 17, 16, 16, 64), 5, 100, False),
    "f320_c150_odd_map": (S(8, 13, 11, 16, 80), 9, 150, True),
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
