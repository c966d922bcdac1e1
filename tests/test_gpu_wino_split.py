"""F(2x2, 3x3) onto more than 32 filters (csrc/wino_fwd.hip): a layer's forward against its 64-bit sum where the kernel's blocks
end: 32 tiles, 8 channels a step, 64 filters, whole and split reductions, 2x2 pooling."""
import math

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# C, H, W, K, batch, pooled, shortcut, how the reduction runs: whole, in parts, or by the direct kernel (the estimate's choice)
CASES = [
    (20, 29, 27, 68, 165, 0, 0, "whole"), (24, 20, 21, 132, 64, 0, 1, "whole"), (28, 33, 31, 132, 16, 0, 0, "whole"),
    (36, 32, 32, 64, 64, 1, 0, "whole"), (60, 23, 26, 100, 60, 1, 1, "whole"), (64, 32, 32, 64, 65, 0, 1, "whole"),
    (68, 27, 25, 124, 64, 1, 0, "whole"), (100, 16, 16, 256, 33, 0, 0, "direct"), (100, 16, 16, 256, 63, 0, 0, "whole"),
    (128, 17, 17, 256, 21, 0, 0, "parts"), (256, 8, 8, 256, 256, 0, 1, "whole"), (512, 8, 8, 512, 16, 0, 0, "parts"),
    (512, 4, 4, 512, 107, 0, 0, "parts"),
]


@pytest.mark.parametrize("C,H,W,K,B,pool,skip,how", CASES)
def test_layer_forward_against_64_bits(C, H, W, K, B, pool, skip, how):
    from paper_2402_14139_amd import binding as nf
    from paper_2402_14139_amd.layer import LocalLayer

    g = torch.Generator(device="cuda").manual_seed(C * 131 + K)
    rn = lambda *s: torch.randn(*s, generator=g, device="cuda")  # noqa: E731
    Hp, Wp = (H // 2, W // 2) if pool else (H, W)
    d = nf.LayerDesc(C_in=C, H_in=H, W_in=W, C_out=K, R=3, S=3, stride=1, pad=1, pool_kind=pool, pool_k=2 * pool,
                     pool_stride=2 * pool, pool_pad=0, skip_kind=skip, skip_C=K * skip, skip_H=H * skip, skip_W=W * skip,
                     skip_stride=skip)
    a = nf.AuxDesc(C_in=K, H_in=Hp, W_in=Wp, A=4, R=3, S=3, pad=1, relu=1, pool_oh=2, pool_ow=2, n_classes=10)
    x, xs = rn(B, H, W, C).relu_(), rn(B, H, W, K).relu_() if skip else None
    W_, b = rn(K, 3, 3, C) * math.sqrt(2 / (9 * C)), rn(K) * 0.1
    host = dict(W=W_.cpu().numpy(), b=b.cpu().numpy(), Wp=None, Wa=np.zeros((4, 3, 3, K), np.float32), ba=np.zeros(4, np.float32),
                Wf=np.zeros((10, 16), np.float32), bf=np.zeros(10, np.float32))
    L = LocalLayer(d, a, host, B, False)
    nf.nf_prof_begin()
    y = L.forward(x, xs, y=L.new_output(B))
    names = {r["kernel"] for r in nf.nf_prof_end()}
    if nf.nf_contraction() == nf.NF_CONTRACT_F32:
        assert ("wino_fwd" in names) == (how != "direct") and (how == "direct" or ("fwd_finish" in names) == (how == "parts")), names
    ref = torch.nn.functional.conv2d(x.cpu().double().permute(0, 3, 1, 2), W_.cpu().double().permute(0, 3, 1, 2), b.cpu().double(), padding=1)
    if skip:
        ref = ref + xs.cpu().double().permute(0, 3, 1, 2)
    ref = ref.relu()
    if pool:
        ref = torch.nn.functional.max_pool2d(ref, 2)
    ref = ref.permute(0, 2, 3, 1).reshape(-1)
    err = y.cpu().double().reshape(-1) - ref
    # rounding errors of 2^-24: the transforms' (2 + 2 additions of values up to twice as large as the result's terms) and those of a
    # running sum of C terms, which grow with its root; the largest of up to 10^7 results is within 6 standard deviations of a
    # result's own error, itself up to 4 times the mean one on the largest partial sums
    u = 2.0 ** -24 * (8 + math.sqrt(C))
    assert float(err.norm() / ref.norm()) < u
    assert float(err.abs().max()) < 24 * u * float(ref.square().mean().sqrt())
