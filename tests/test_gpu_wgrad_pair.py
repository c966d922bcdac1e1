"""A layer's weight gradient and its head's in one launch (csrc/igemm_wgrad_fast.hip, wgrad_pair_kernel): the variants of either,
grids that are not whole multiples of eight workgroups.  That the launch is made, against the oracle, and bit for bit against the
same step while a measurement is on that has the two launched by themselves."""
import threading

import numpy as np
import pytest

from paper_2402_14139_amd import binding as nf
from paper_2402_14139_amd import layout
from tests import gpu_common as G
from tests.test_gpu_parity import S

pytestmark = pytest.mark.gpu

W64, W32, STEM = "igemm_wgrad_fast_64x64", "igemm_wgrad_fast_32x128", "stem_wgrad"
# name -> (spec, B, classes, kernels of the layer and the head, the launch they share; none where a projection's columns begin inside a tile
# or are 32 rows wide)
CASES = {
    "stem_narrow": (S(3, 9, 7, 16, 8), 3, 10, {STEM, W32}, "stem_32x128"),
    "stem_wide_head": (S(3, 8, 8, 100, 40, pool=(2, 2, 0)), 5, 10, {STEM, W64}, "stem_64x64"),
    "stem_head_position_rows": (S(3, 8, 8, 64, 40, pool=(2, 2, 0)), 5, 10, {STEM, W64}, "stem_64x64_rows"),
    "one_tile_each": (S(4, 2, 2, 4, 4), 1, 10, {W32}, "32x128_32x128"),
    "layer_64_head_32": (S(20, 7, 5, 72, 12, R=5, stride=2), 9, 37, {W64, W32}, "64x64_32x128"),
    "both_64": (S(20, 9, 9, 72, 40), 5, 10, {W64}, "64x64_64x64"),
    "layer_64_head_position_rows": (S(20, 5, 4, 64, 36), 6, 10, {W64}, "64x64_64x64_rows"),
    "layer_32_head_64": (S(24, 9, 8, 28, 36), 5, 10, {W32, W64}, "32x128_64x64"),
    "both_64_position_rows": (S(64, 2, 2, 128, 80), 17, 10, {W64}, "64x64_rows_64x64_rows"),
    "layer_64_position_rows_head_64": (S(64, 2, 2, 72, 40), 9, 10, {W64}, "64x64_rows_64x64"),
    "layer_64_position_rows_head_32": (S(128, 3, 3, 64, 20), 10, 10, {W64, W32}, "64x64_rows_32x128"),
    "layer_64_projection_mixed": (S(36, 4, 4, 60, 8, skip=2, skip_C=20), 7, 10, {W64, W32}, None),
    "layer_64_projection_whole": (S(64, 4, 4, 64, 36, skip=2, skip_C=64), 7, 10, {W64}, "64x64_proj_64x64_rows"),
    "layer_64_projection_whole_head_64": (S(64, 4, 4, 72, 36, skip=2, skip_C=64), 7, 10, {W64}, "64x64_proj_64x64"),
    "layer_32_projection_mixed": (S(12, 6, 5, 28, 68, skip=2, skip_C=8), 4, 10, {W32, W64}, None),
    "layer_32_projection_whole": (S(128, 5, 5, 32, 16, skip=2, skip_C=64), 6, 10, {W32}, None),
    "layer_64_projection_whole_narrow_head": (S(64, 5, 4, 68, 12, skip=2, skip_C=128), 5, 10, {W64, W32}, "64x64_proj_32x128"),
    "layer_32_identity_1x1": (S(24, 9, 9, 24, 4, R=1, pad=0, skip=1), 5, 10, {W32}, "32x128_32x128"),
}


def weight_gradients(records):
    return {r["kernel"] for r in records if "wgrad" in r["kernel"] and "reduce" not in r["kernel"]}


@pytest.mark.parametrize("name", list(CASES))
def test_pairs_match_oracle_and_single_launches(name):
    spec, B, cls, kernels, pair = CASES[name]
    print(f"case {name}: B={B}", flush=True)
    nf.nf_prof_begin_as_run()
    out, final = G.run_step_both(spec, cls, B, seed=360, lr=0.05, mu=0.9, steps=1)
    got = weight_gradients(nf.nf_prof_end())
    G.check_step_results(name, out, final)
    nf.nf_prof_begin()
    alone, _ = G.run_step_both(spec, cls, B, seed=360, lr=0.05, mu=0.9, steps=1)
    apart = weight_gradients(nf.nf_prof_end())
    if nf.nf_contraction() == nf.NF_CONTRACT_F32:
        assert got == ({"igemm_wgrad_pair_" + pair} if pair else kernels), got
        assert apart == kernels, apart
    for k, v in out[0][0][1].items():
        if v is not None:
            assert np.array_equal(v, alone[0][0][1][k]), k


def test_the_mode_may_change_while_a_step_is_enqueued():
    """Another thread sets the contraction mode all the while: every step succeeds, in the one or the other."""
    spec, B, cls = S(64, 2, 2, 128, 80), 17, 10
    x, xs, labels, p = G.make_inputs(spec, B, cls, 371)
    L = G.gpu_layer(spec, cls, p, B, 0.0)
    xd, ld = G.to_dev(layout.act_to_lib(x)), G.to_dev(labels)
    L.step(xd, None, ld, 0.0, 0.0)
    ref = {k: v.double().clone() for k, v in L.g.items() if v is not None}
    prev, stop, turns = nf.nf_contraction(), threading.Event(), [0]

    def toggle():
        while not stop.is_set():
            nf.nf_contraction(nf.NF_CONTRACT_BF16X6)
            nf.nf_contraction(nf.NF_CONTRACT_F32)
            turns[0] += 1

    t = threading.Thread(target=toggle)
    t.start()
    try:
        for _ in range(3000):
            L.step(xd, None, ld, 0.0, 0.0)
    finally:
        stop.set()
        t.join()
        nf.nf_contraction(prev)
    assert turns[0] > 100
    for k, v in ref.items():
        assert (L.g[k].double() - v).norm() <= G.REL * v.norm(), k
