"""3x3 convolutions through F(2x2, 3x3) take fp32 products: rounded to nearest, so that errors of different results are
independent.  Matrix instructions on bf16 pieces round their running sums down, which shows in averages of sums that only grow."""
import math

import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(params=["F32", "BF16X6", "BF16X9"])
def mode(request):
    """All: layers of fewer than 128 filters take the same products in every mode."""
    from paper_2402_14139_amd import binding as nf

    before = nf.nf_contraction(getattr(nf, "NF_CONTRACT_" + request.param))
    yield request.param
    nf.nf_contraction(before)


def conv64(x, w):
    B, H, W, C = x.shape
    xp = torch.nn.functional.pad(x.double(), (0, 0, 1, 1, 1, 1))
    out = 0
    for r in range(3):
        for s in range(3):
            out = out + xp[:, r:r + H, s:s + W].reshape(-1, C) @ w[:, r, s].double().t()
    return out.reshape(B, H, W, -1)


def run(call):
    from paper_2402_14139_amd import binding as nf

    nf.nf_prof_begin()
    call()
    torch.cuda.synchronize()
    return {r["kernel"] for r in nf.nf_prof_end()}


def test_transformed_filters_leave_room_for_the_weight_gradient():
    """A step near the static array's size: 64 channels, a head of 128.  Transformed filters half as large again as in fp32 push the
    partial sums of the transformed weight gradient out of the plan."""
    from paper_2402_14139_amd import binding as nf
    from paper_2402_14139_amd.layer import LocalLayer

    B, H, C, A, cls = 64, 32, 64, 128, 10
    g = torch.Generator(device="cuda").manual_seed(4)
    rn = lambda *s: torch.randn(*s, generator=g, device="cuda")  # noqa: E731
    d = nf.LayerDesc(C_in=C, H_in=H, W_in=H, C_out=C, R=3, S=3, stride=1, pad=1)
    a = nf.AuxDesc(C_in=C, H_in=H, W_in=H, A=A, R=3, S=3, pad=1, relu=1, pool_oh=2, pool_ow=2, n_classes=cls)
    p = dict(W=rn(C, 3, 3, C) * 0.06, b=rn(C), Wp=None, Wa=rn(A, 3, 3, C) * 0.06, ba=rn(A), Wf=rn(cls, 4 * A) * 0.1, bf=rn(cls))
    L = LocalLayer(d, a, {k: None if v is None else v.cpu().numpy() for k, v in p.items()}, B, False)
    x, labels = rn(B, H, H, C).relu_(), torch.randint(0, cls, (B,), generator=g, device="cuda", dtype=torch.int32)
    names = run(lambda: L.step(x, None, labels, 0.01, 0.0))
    if nf.nf_contraction() != nf.NF_CONTRACT_F32:
        pytest.skip("the split modes have their own weight gradient of this head")
    assert {"wino_fwd", "wino_wgrad"} <= names, names


@pytest.mark.parametrize("C,H,K,B", [(512, 16, 100, 128), (512, 16, 64, 212)])
def test_averages_of_sums_that_only_grow(C, H, K, B, mode):
    averages(C, H, K, B)


@pytest.mark.parametrize("C,H,K,B", [(512, 4, 512, 512), (256, 8, 256, 256)])
def test_averages_of_sums_that_only_grow_wide_layers(C, H, K, B):
    averages(C, H, K, B)


def averages(C, H, K, B):
    """Rectified inputs, filters of one sign."""
    from paper_2402_14139_amd import binding as nf

    g = torch.Generator(device="cuda").manual_seed(C)
    x = torch.randn(B, H, H, C, generator=g, device="cuda").relu_()
    w = (torch.randn(K, 3, 3, C, generator=g, device="cuda") * math.sqrt(2 / (9 * C))).abs_()
    b, y = torch.zeros(K, device="cuda"), torch.empty(B, H, H, K, device="cuda")
    d = nf.LayerDesc(C_in=C, H_in=H, W_in=H, C_out=K, R=3, S=3, stride=1, pad=1)
    ws = torch.empty(nf.nf_workspace_bytes(d, None, B), dtype=torch.uint8, device="cuda")
    names = run(lambda: nf.nf_layer_fwd(d, B, x, None, nf.layer_params(w, b, None), y, ws))
    if K < 128 or nf.nf_contraction() == nf.NF_CONTRACT_F32:
        assert "wino_fwd" in names, names
    else:
        pytest.skip("the split modes have their own kernel here")
    ref = conv64(x, w).mean((0, 1, 2))
    off = float((y.double().mean((0, 1, 2)) - ref).norm() / ref.norm())
    # thousands of pixels' own errors average out; what all pixels share is the rounding of the transformed filters, 2^-24 each at
    # most and one of C: far below a quarter of 2^-24
    print(f"averages, C={C} K={K}: {off * 2 ** 24:.3f} of 2^-24", flush=True)
    assert off < 2.0 ** -26
