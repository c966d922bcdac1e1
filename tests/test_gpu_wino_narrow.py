"""F(2x2, 3x3) in its variant of 32 filters (csrc/wino_fwd.hip): heads and layers of 17 ... 32 filters
against the CPU oracle, its sums for the head's pooling, and values that are not finite."""
import numpy as np
import pytest
import torch

from paper_2402_14139_amd import binding as nf
from tests import gpu_common as G
from tests.test_gpu_parity import S

pytestmark = pytest.mark.gpu

# name -> (spec, B, classes, launches of the variant)
CASES = {
    # pooling sums from the epilogue: rows of 16 pixels (two slots), of 32, of 64 (a ragged head)
    "pool_16": (S(16, 16, 16, 64, 32), 256, 10, 1),
    "pool_32": (S(64, 32, 32, 64, 32), 64, 10, 1),
    "pool_64_a20": (S(8, 6, 64, 64, 20), 170, 10, 1),
    # odd maps: pooled by a launch of its own; a ragged last tile block and channels that are no multiple of 8
    "odd_13x15_a28": (S(20, 13, 15, 68, 28), 260, 10, 1),
    # a layer and its data gradient of few filters, and the head
    "narrow_layer": (S(48, 28, 27, 28, 24), 80, 10, 2),
    # reduction in parts, which the pooling launch adds
    "parts": (S(8, 12, 12, 256, 32), 100, 10, 1),
}


@pytest.mark.parametrize("name", list(CASES))
def test_narrow_steps_match_oracle(name):
    spec, B, cls, launches = CASES[name]
    print(f"case {name}: B={B}", flush=True)
    nf.nf_prof_begin()
    out, final = G.run_step_both(spec, cls, B, seed=330, lr=0.05, mu=0.9, steps=1)
    got = {r["kernel"]: r["launches"] for r in nf.nf_prof_end()}
    G.check_step_results(name, out, final)
    assert got.get("wino_fwd_32", 0) >= launches, got


@pytest.mark.parametrize("W", [16, 32])
def test_pooling_sums_hold_results_formed_again(W):
    """An infinity in one pixel: the loss of that sample alone is not finite, all others keep theirs."""
    B, H, K, A, cls = 256, 16, 64, 32, 10
    g = torch.Generator(device="cuda").manual_seed(3)
    rn = lambda *s: torch.randn(*s, generator=g, device="cuda")  # noqa: E731
    d = nf.LayerDesc(C_in=8, H_in=H, W_in=W, C_out=K, R=3, S=3, stride=1, pad=1)
    a = nf.AuxDesc(C_in=K, H_in=H, W_in=W, A=A, R=3, S=3, pad=1, relu=1, pool_oh=2, pool_ow=2, n_classes=cls)
    y = rn(B, H, W, K).relu()
    labels = torch.randint(0, cls, (B,), generator=g, device="cuda", dtype=torch.int32)
    p = [rn(A, 3, 3, K) * 0.05, rn(A), rn(cls, 4 * A) * 0.2, rn(cls)]
    ap = nf.aux_params(*p)
    ws = torch.empty(nf.nf_workspace_bytes(d, a, B), dtype=torch.uint8, device="cuda")
    off, nbytes = nf.nf_workspace_region(d, a, B, nf.NF_WS_AUX_ACT)
    loss, acts = torch.zeros(1, device="cuda"), []
    for bad in (False, True):
        if bad:
            y[5, 4, 7, 3] = float("inf")
        nf.nf_prof_begin()
        nf.nf_aux_fwd_loss(d, a, B, y, labels, ap, loss, ws)
        names = {r["kernel"] for r in nf.nf_prof_end()}
        assert "wino_fwd_32" in names and "head_pool" not in names, names
        u = ws[off:off + nbytes].view(torch.float32).reshape(B, H, W, A).double()
        # the pooled features, logits and loss in 64 bits from the activation the kernel stored
        q = u.reshape(B, 2, H // 2, 2, W // 2, A).mean(dim=(2, 4)).reshape(B, -1)
        z = q @ p[2].double().t() + p[3].double()
        acts.append((u, torch.nn.functional.cross_entropy(z, labels.long(), reduction="none"), float(loss)))
    (u0, l0, got0), (u1, l1, got1) = acts
    assert abs(got0 - float(l0.mean())) <= 1e-5 * abs(float(l0.mean()))
    inf = torch.isinf(u1)
    at = torch.zeros_like(inf)
    at[5, 3:6, 6:9, :] = p[0].permute(1, 2, 0, 3)[..., 3].flip(0, 1) > 0  # positive taps on that pixel, the others' ReLU is 0
    assert torch.equal(inf, at) and not np.isfinite(got1)
    # 576-term sums in two orders where a neighbour was not finite: a few 1e-7 of the largest value
    seen = torch.zeros_like(inf)
    seen[5, 3:6, 6:9, :] = True
    assert (u1 - u0)[~seen].abs().max() <= 5e-6 * u0.max()
