"""F(2x2, 3x3) in its variant of 32 filters (csrc/wino_fwd.hip): data gradients onto layers of 17 ... 32 filters against the CPU
oracle, and the convolutions of that width, which do not run through it, for the accuracy of averages over their results."""
import pytest
import torch

from paper_2402_14139_amd import binding as nf
from paper_2402_14139_amd import layout
from tests import gpu_common as G
from tests.test_gpu_parity import S

pytestmark = pytest.mark.gpu

# name -> (spec, B, classes, launches of the variant)
CASES = {
    # not the layer and the head themselves
    "narrow_layer": (S(48, 28, 27, 28, 24), 80, 10, 1),
    # odd maps: a ragged last tile block, channels that are no multiple of 8
    "odd_13x15_k28": (S(68, 13, 15, 28, 20), 260, 10, 1),
    # reduction in parts
    "parts": (S(256, 12, 12, 32, 16), 100, 10, 1),
    "pooled_narrow": (S(64, 32, 32, 32, 32, pool=(2, 2, 0)), 200, 10, 1),
    # heads and layers of few filters keep the direct kernel
    "pool_16": (S(16, 16, 16, 64, 32), 256, 10, 0),
    "pool_32": (S(64, 32, 32, 64, 32), 64, 10, 0),
    "odd_13x15_a28": (S(20, 13, 15, 68, 28), 260, 10, 0),
    "head_parts": (S(8, 12, 12, 256, 32), 100, 10, 0),
}


@pytest.mark.parametrize("name", list(CASES))
def test_narrow_steps_match_oracle(name):
    spec, B, cls, launches = CASES[name]
    print(f"case {name}: B={B}", flush=True)
    nf.nf_prof_begin()
    out, final = G.run_step_both(spec, cls, B, seed=330, lr=0.05, mu=0.9, steps=1)
    got = {r["kernel"]: r["launches"] for r in nf.nf_prof_end()}
    G.check_step_results(name, out, final)
    n = got.get("wino_fwd_32", 0)
    assert n == launches, got


def filter_rounding_mean(x, w):
    """What the fp32 rounding of the transformed filter alone adds to a convolution's results (x [B,H,W,C], even sizes; w
    [K,3,3,C]), averaged over images and pixels [K]: everything else in 64 bits."""
    Gm = torch.tensor([[1, 0, 0], [.5, .5, .5], [.5, -.5, .5], [0, 0, 1]], device=w.device, dtype=torch.float64)
    Bt = torch.tensor([[1, 0, -1, 0], [0, 1, 1, 0], [0, -1, 1, 0], [0, 1, 0, -1]], device=w.device, dtype=torch.float64)
    At = torch.tensor([[1, 1, 1, 0], [0, 1, -1, -1]], device=w.device, dtype=torch.float64)
    U = torch.einsum("ar,krsc,bs->kabc", Gm, w.double(), Gm)
    dU = U.float().double() - U
    xp = torch.nn.functional.pad(x.double(), (0, 0, 1, 1, 1, 1))
    # the mean patch d[i][j] over all tiles: rows i, i + 2, ... of the padded image
    H, W = x.shape[1:3]
    d = torch.stack([torch.stack([xp[:, i:i + H:2, j:j + W:2].mean(dim=(0, 1, 2)) for j in range(4)]) for i in range(4)])
    V = torch.einsum("ai,ijc,bj->abc", Bt, d, Bt)
    return torch.einsum("pa,kab,qb->kpq", At, torch.einsum("kabc,abc->kab", dU, V), At).mean(dim=(1, 2))


@pytest.mark.parametrize("what", ["head", "layer"])
@pytest.mark.parametrize("C,H,A,B", [(64, 32, 32, 64), (128, 16, 20, 256), (64, 64, 32, 16)])
def test_averages_of_narrow_convolutions(C, H, A, B, what):
    """F_n averages an activation over pixels and the gradients sum over samples: rounding that is the same for all of them
    stays.  The direct sum's is not the same: its averages are off by a tenth of what a single rounding of a transformed filter
    leaves; the line lies at 0.6 of that.  (The layer's bias keeps its ReLU from cutting anything.)"""
    g = torch.Generator(device="cuda").manual_seed(C)
    rn = lambda *s: torch.randn(*s, generator=g, device="cuda")  # noqa: E731
    y, labels = rn(B, H, H, C).relu(), torch.zeros(B, device="cuda", dtype=torch.int32)
    Wa, bias, loss = rn(A, 3, 3, C) * (2.0 / (9 * C)) ** 0.5, 0.0, torch.zeros(1, device="cuda")
    if what == "layer":
        bias = 8.0  # the results' standard deviation is about 1.2
        b = torch.full((A,), bias, device="cuda")
        d = nf.LayerDesc(C_in=C, H_in=H, W_in=H, C_out=A, R=3, S=3, stride=1, pad=1)
        got = torch.empty(B, H, H, A, device="cuda")
        ws = torch.empty(max(256, nf.nf_workspace_bytes(d, None, B)), dtype=torch.uint8, device="cuda")
        nf.nf_layer_fwd(d, B, y, None, nf.layer_params(Wa, b, None), got, ws)
        assert (got > 0).all()
    else:
        d = nf.LayerDesc(C_in=16, H_in=H, W_in=H, C_out=C, R=3, S=3, stride=1, pad=1)
        a = nf.AuxDesc(C_in=C, H_in=H, W_in=H, A=A, R=3, S=3, pad=1, relu=0, pool_oh=2, pool_ow=2, n_classes=10)
        p = [Wa, torch.zeros(A, device="cuda"), rn(10, 4 * A) * 0.1, torch.zeros(10, device="cuda")]
        ws = torch.empty(nf.nf_workspace_bytes(d, a, B), dtype=torch.uint8, device="cuda")
        nf.nf_aux_fwd_loss(d, a, B, y, labels, nf.aux_params(*p), loss, ws)
        off, nbytes = nf.nf_workspace_region(d, a, B, nf.NF_WS_AUX_ACT)
        got = ws[off:off + nbytes].view(torch.float32)
    got = got.reshape(-1, A).double().mean(0) - bias
    yp = torch.nn.functional.pad(y.double(), (0, 0, 1, 1, 1, 1))
    mean = torch.stack([torch.stack([yp[:, r:r + H, s:s + H].mean(dim=(0, 1, 2)) for s in range(3)]) for r in range(3)])
    ref = torch.einsum("krsc,rsc->k", Wa.double(), mean)
    err, line = float((got - ref).norm()), 0.6 * float(filter_rounding_mean(y, Wa).norm())
    print(f"{what} {C} channels: {err:.3e}, line {line:.3e}", flush=True)
    assert err <= line


@pytest.mark.parametrize("B,classes,step,calls", [(192, 10, True, False), (193, 10, True, True), (3, 10, True, False), (3, 1200, True, True)])
def test_filter_of_the_data_gradient(B, classes, step, calls):
    """The transformed filter comes with a head launch of the step, or with the backward call's own; behind a forward call with
    the whole head in it, it takes a launch that pays from a certain size on."""
    spec = S(8, 16, 16, 28, 32)
    x, _, labels, p = G.make_inputs(spec, B, classes, 372)
    L = G.gpu_layer(spec, classes, p, B, 0.0)
    xd, ld = G.to_dev(layout.act_to_lib(x)), G.to_dev(labels)
    got = []
    for separate in (False, True):
        if separate:
            y = L.forward(xd, None)
            L.aux_loss(y, ld)
        nf.nf_prof_begin()
        if separate:
            L.backward(xd, None, y)
        else:
            L.step(xd, None, ld, 0.0, 0.0)
        got.append("wino_fwd_32" in {r["kernel"] for r in nf.nf_prof_end()})
    assert got == [step, calls]
