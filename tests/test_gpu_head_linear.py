"""The head's linear layer and its gradients by the number of features and classes (csrc/head.hip): each form on both
sides of its line, pooling windows of one size and of several, against the oracle."""
import pytest

from tests import gpu_common as G
from tests.test_gpu_parity import S

pytestmark = pytest.mark.gpu

# name -> (spec, B, classes); 4 * A features
CASES = {
    "f124": (S(8, 12, 12, 16, 31), 9, 70),
    "f128_c16": (S(8, 32, 32, 16, 32), 5, 16),
    "f128_c17_odd_map": (S(8, 13, 11, 16, 32), 6, 17),
    "f132_c65_odd_filters": (S(8, 16, 16, 16, 33), 7, 65),
    "f128_c128": (S(8, 16, 16, 16, 32), 70, 128),  # a hundred and more classes: every range of a batch
    "f512_c31": (S(8, 9, 8, 16, 128), 3, 31),
    "f1024_c9": (S(16, 2, 2, 32, 256), 33, 9),
    "f260_c300": (S(8, 10, 10, 16, 65), 4, 300),
}


@pytest.mark.parametrize("name", list(CASES))
@pytest.mark.parametrize("pmax", [0, 1])
def test_linear_layers_match_oracle(name, pmax):
    spec, B, cls = CASES[name]
    print(f"case {name} head_pool={pmax}", flush=True)
    out, final = G.run_step_both(spec, cls, B, seed=340, lr=0.05, mu=0.9, steps=1, head_pool=pmax)
    G.check_step_results(name, out, final)
