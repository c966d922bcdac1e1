"""Direct contractions on small maps by output position (csrc/igemm_fwd_fast.hip, csrc/igemm_wgrad_fast.hip): taps over the padding are
left out.  Against the oracle, at the edges of the rule: batches around whole tiles, maps of one to eight pixels, strides,
5x5 filters, reductions cut in parts that begin and end between the taps of a channel chunk."""
import pytest
import torch

from paper_2402_14139_amd import binding as nf
from tests import gpu_common as G
from tests.test_gpu_parity import S

pytestmark = pytest.mark.gpu

# name -> (spec, B, classes)
CASES = {
    "map_1x1": (S(96, 1, 1, 132, 4), 64, 10),
    "map_2x2_wide_head": (S(64, 2, 2, 96, 64), 65, 10),
    "map_2x2_parts": (S(256, 2, 2, 64, 4), 129, 10),
    "map_3x2_identity": (S(160, 3, 2, 160, 8, skip=1), 64, 10),
    "map_4x4_5x5": (S(32, 4, 4, 68, 32, R=5), 70, 10),
    "map_4x4_stride2": (S(64, 4, 4, 72, 16, stride=2), 128, 10),
    "map_5x4_head_parts": (S(8, 5, 4, 288, 12), 128, 10),
    "map_2x2_pooled": (S(64, 4, 4, 64, 20, pool=(2, 2, 0)), 61, 10),
    "map_8x8_no_padding": (S(32, 8, 8, 36, 4, pad=0), 64, 10),
    "map_1x7_row": (S(64, 1, 7, 64, 32), 66, 10),
}


@pytest.mark.parametrize("name", list(CASES))
def test_small_maps_match_oracle(name):
    spec, B, cls = CASES[name]
    print(f"case {name}: B={B}", flush=True)
    out, final = G.run_step_both(spec, cls, B, seed=350, lr=0.05, mu=0.9, steps=1)
    G.check_step_results(name, out, final)


def test_padding_contributes_nothing():
    """An infinite weight reaches the pixels whose window holds a pixel under its tap, and no others."""
    B, C, H, K = 64, 32, 2, 64
    g = torch.Generator(device="cuda").manual_seed(6)
    x = torch.rand(B, H, H, C, generator=g, device="cuda") + 0.1
    w, b = torch.randn(K, 3, 3, C, generator=g, device="cuda") * 0.05, torch.full((K,), 50.0, device="cuda")
    w[9, 0, 0, 5] = float("inf")  # over a pixel for the last output position alone
    d = nf.LayerDesc(C_in=C, H_in=H, W_in=H, C_out=K, R=3, S=3, stride=1, pad=1)
    y = torch.empty(B, H, H, K, device="cuda")
    ws = torch.empty(max(256, nf.nf_workspace_bytes(d, None, B)), dtype=torch.uint8, device="cuda")
    nf.nf_layer_fwd(d, B, x, None, nf.layer_params(w, b, None), y, ws)
    if nf.nf_contraction() != nf.NF_CONTRACT_F32:
        pytest.skip("the split modes turn an infinity into NaN")
    inf = torch.zeros_like(y, dtype=torch.bool)
    inf[:, 1, 1, 9] = True
    assert torch.equal(torch.isinf(y), inf) and (y > 0).all()
