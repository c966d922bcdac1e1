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


@pytest.mark.parametrize("B,C,H,A", [(17, 64, 2, 80), (9, 128, 3, 40), (33, 64, 4, 64), (64, 128, 2, 200)])
def test_padding_contributes_nothing_to_weight_gradients(B, C, H, A):
    """An infinite gradient at the pixels that one pooling window alone sees: the taps that lie over the padding there stay finite."""
    g = torch.Generator(device="cuda").manual_seed(7)
    d = nf.LayerDesc(C_in=16, H_in=H, W_in=H, C_out=C, R=3, S=3, stride=1, pad=1)
    a = nf.AuxDesc(C_in=C, H_in=H, W_in=H, A=A, R=3, S=3, pad=1, relu=1, pool_oh=H, pool_ow=H, n_classes=4, loss_kind=1)
    x = torch.rand(B, H, H, 16, generator=g, device="cuda")
    y = torch.rand(B, H, H, C, generator=g, device="cuda") + 0.1
    labels = torch.zeros(B, device="cuda", dtype=torch.int32)
    Wa, Wf = torch.zeros(A, 3, 3, C, device="cuda"), torch.zeros(4, H * H * A, device="cuda")
    Wf[2, 5] = 3e38  # of filter 5 at pixel (0, 0): the logit is 3e8, its gradient infinite
    z = lambda *s: torch.zeros(*s, device="cuda")  # noqa: E731
    layer = [z(C, 3, 3, 16), z(C), z(C, 3, 3, 16), z(C)]
    head = [Wa, z(A) + 1e-30, Wf, z(4), z(A, 3, 3, C), z(A), z(4, H * H * A), z(4)]
    lp, gp, ap, ga = nf.layer_params(*layer[:2], None), nf.layer_params(*layer[2:], None), nf.aux_params(*head[:4]), nf.aux_params(*head[4:])
    loss, gWa = z(1), head[4]
    ws = torch.empty(nf.nf_workspace_bytes(d, a, B), dtype=torch.uint8, device="cuda")
    nf.nf_aux_fwd_loss(d, a, B, y, labels, ap, loss, ws)
    nf.nf_local_bwd_wgrad(d, a, B, x, None, y, lp, ap, gp, ga, ws)
    if nf.nf_contraction() != nf.NF_CONTRACT_F32:
        pytest.skip("the split modes turn an infinity into NaN")
    over = torch.zeros(3, 3, dtype=torch.bool, device="cuda")
    over[0, :] = over[:, 0] = True
    assert torch.isfinite(gWa[5][over]).all() and not torch.isfinite(gWa[5][~over]).any()
