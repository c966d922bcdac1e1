"""2x2 max pooling: in the epilogue of F(2x2, 3x3) (csrc/wino_fwd.hip), and its backward by pooled cells
(csrc/elementwise.hip)."""
import pytest
import torch

from paper_2402_14139_amd import binding as nf
from tests import gpu_common as G
from tests.test_gpu_parity import S

pytestmark = pytest.mark.gpu


def forward(d, B, x, xs, w, b):
    Ho, Wo, Hp, Wp = nf.nf_layer_out_dims(d)
    y = torch.full((B, Hp, Wp, d.C_out), -1.0, device="cuda")
    ws = torch.empty(max(256, nf.nf_workspace_bytes(d, None, B)), dtype=torch.uint8, device="cuda")
    nf.nf_prof_begin()
    nf.nf_layer_fwd(d, B, x, xs, nf.layer_params(w, b, None), y, ws)
    names = {r["kernel"] for r in nf.nf_prof_end()}
    arg = None
    if d.pool_kind:
        off, nbytes = nf.nf_workspace_region(d, None, B, nf.NF_WS_POOL_ARG)
        arg = ws[off:off + nbytes].reshape(B, Hp, Wp, d.C_out).clone()
    return y, arg, names


# odd maps (a last row and column without a window), ragged tile blocks, filters that are no multiple of 64
@pytest.mark.parametrize("C,H,W,K,B,skip,bad", [(64, 32, 32, 128, 20, 0, False), (64, 13, 15, 124, 100, 0, True), (64, 9, 28, 36, 200, 0, True),
                                                (64, 16, 17, 40, 190, 1, False), (64, 5, 4, 256, 640, 1, True)])
def test_pooled_in_the_epilogue_as_by_itself(C, H, W, K, B, skip, bad):
    """Bit for bit the pooled result of the convolution without pooling, first maxima selected; infinities too."""
    g = torch.Generator(device="cuda").manual_seed(H * W)
    rn = lambda *s: torch.randn(*s, generator=g, device="cuda")  # noqa: E731
    x, w, b = rn(B, H, W, C), rn(K, 3, 3, C) * 0.05, rn(K)
    xs = rn(B, H, W, K) if skip else None
    if bad:
        x[3, 1, 2, 5] = float("inf")
    kw = dict(C_in=C, H_in=H, W_in=W, C_out=K, R=3, S=3, stride=1, pad=1)
    if skip:
        kw.update(skip_kind=1, skip_C=K, skip_H=H, skip_W=W, skip_stride=1)
    plain, _, n0 = forward(nf.LayerDesc(**kw), B, x, xs, w, b)
    y, arg, n1 = forward(nf.LayerDesc(**kw, pool_kind=1, pool_k=2, pool_stride=2, pool_pad=0), B, x, xs, w, b)
    if nf.nf_contraction() == nf.NF_CONTRACT_F32:
        assert any(k.startswith("wino_fwd") for k in n0) and "maxpool_fwd" not in n1, (n0, n1)
    Hp, Wp = H // 2, W // 2
    win = plain[:, :2 * Hp, :2 * Wp].reshape(B, Hp, 2, Wp, 2, K).permute(0, 1, 3, 2, 4, 5).reshape(B, Hp, Wp, 4, K)
    assert torch.equal(y, win.amax(3))
    first = (win == y.unsqueeze(3)).to(torch.uint8).argmax(3)  # (the first of equal values)
    assert torch.equal(arg.long(), first)


# name -> (spec, B): channels that are no multiple of 4, maps with a row and a column beside the windows
CASES = {
    "odd_both": (S(16, 7, 9, 20, 4, pool=(2, 2, 0)), 5),
    "odd_rows_k6": (S(8, 5, 6, 6, 5, pool=(2, 2, 0)), 3),
    "even": (S(64, 16, 16, 64, 8, pool=(2, 2, 0)), 40),
    "overlapping": (S(16, 9, 8, 20, 4, pool=(3, 2, 1)), 5),
}


@pytest.mark.parametrize("name", list(CASES))
def test_pool_backward_matches_oracle(name):
    spec, B = CASES[name]
    out, final = G.run_step_both(spec, 10, B, seed=360, lr=0.05, mu=0.9, steps=1)
    G.check_step_results(name, out, final)
