"""Which kernels carry out a wide 3x3 convolution in the split-operand modes."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mode,kernel", [("BF16X6", "igemm_fwd_split_128x128"), ("BF16X9", "igemm_fwd_split9_128x128")])
@pytest.mark.parametrize("C,H,K,B", [(512, 4, 512, 512), (256, 8, 256, 256), (64, 32, 128, 64), (144, 14, 132, 64)])
def test_wide_convolutions_keep_the_modes_own_kernel(C, H, K, B, mode, kernel):
    """Rectified values that are ties to within rounding fall as that mode's direct sums have them, though F(2x2, 3x3) would be
    planned for every one of these shapes (and runs in the default mode)."""
    from paper_2402_14139_amd import binding as nf

    d = nf.LayerDesc(C_in=C, H_in=H, W_in=H, C_out=K, R=3, S=3, stride=1, pad=1)
    g = torch.Generator(device="cuda").manual_seed(3)
    x, w = torch.randn(B, H, H, C, generator=g, device="cuda"), torch.randn(K, 3, 3, C, generator=g, device="cuda") * 0.05
    b, y = torch.zeros(K, device="cuda"), torch.empty(B, H, H, K, device="cuda")
    ws = torch.empty(nf.nf_workspace_bytes(d, None, B), dtype=torch.uint8, device="cuda")
    ran = {}
    for m in (nf.NF_CONTRACT_F32, getattr(nf, "NF_CONTRACT_" + mode)):
        before = nf.nf_contraction(m)
        try:
            nf.nf_prof_begin()
            nf.nf_layer_fwd(d, B, x, None, nf.layer_params(w, b, None), y, ws)
            ran[m] = {r["kernel"] for r in nf.nf_prof_end()}
        finally:
            nf.nf_contraction(before)
    assert "wino_fwd" in ran.pop(nf.NF_CONTRACT_F32)
    assert list(ran.values()) == [{kernel}], ran
