"""Tile sizes of the direct contraction kernels for more than 128 filters (csrc/igemm_fwd_fast.hip,
csrc/igemm_wgrad_fast.hip): the small tile where the large one would leave compute units idle."""
import pytest
import torch

from paper_2402_14139_amd import binding as nf
from tests import gpu_common as G
from tests.test_gpu_parity import S

pytestmark = pytest.mark.gpu

# name -> (spec, B, classes): filters, taps x channels and rows that end inside a 64-wide tile
SMALL = {
    "n132_rows_of_one_tile": (S(64, 5, 5, 132, 4, R=5), 2, 10),
    "n260_stride2": (S(36, 9, 9, 260, 4, stride=2), 13, 10),
    # both operands of the projection columns: a tile of taps and projection channels, whole tiles of each
    "projection_mixed": (S(36, 4, 4, 196, 4, skip=2, skip_C=20), 9, 10),
    "projection_whole": (S(64, 4, 4, 192, 4, skip=2, skip_C=64), 9, 10),
    "identity_1x1": (S(192, 6, 6, 192, 4, R=1, pad=0, skip=1), 11, 10),
    "wide_head_split": (S(256, 2, 2, 320, 144), 33, 10),
}


@pytest.mark.parametrize("name", list(SMALL))
def test_small_tiles_match_oracle(name):
    spec, B, cls = SMALL[name]
    print(f"case {name}: B={B}", flush=True)
    nf.nf_prof_begin()
    out, final = G.run_step_both(spec, cls, B, seed=320, lr=0.05, mu=0.9, steps=1)
    got = {r["kernel"] for r in nf.nf_prof_end()}
    G.check_step_results(name, out, final)
    if nf.nf_contraction() == nf.NF_CONTRACT_F32:
        assert {"igemm_fwd_fast_64x64", "igemm_wgrad_fast_64x64"} <= got, got


@pytest.mark.parametrize("B,K,kernel", [(128, 256, "igemm_fwd_fast_128x128"), (127, 256, "igemm_fwd_fast_64x64"),
                                        (128, 192, "igemm_fwd_fast_64x64")])
def test_both_sides_of_the_forward_rule(B, K, kernel):
    """512 large tiles take them, 508 or a column padded by half a tile do not."""
    H, C, R = 16, 84, 5
    g = torch.Generator(device="cuda").manual_seed(9)
    x = torch.randn(B, H, H, C, generator=g, device="cuda")
    w, b = torch.randn(K, R, R, C, generator=g, device="cuda") * 0.02, torch.randn(K, generator=g, device="cuda")
    d = nf.LayerDesc(C_in=C, H_in=H, W_in=H, C_out=K, R=R, S=R, stride=1, pad=2)
    y = torch.empty(B, H, H, K, device="cuda")
    ws = torch.empty(nf.nf_workspace_bytes(d, None, B), dtype=torch.uint8, device="cuda")
    nf.nf_prof_begin()
    nf.nf_layer_fwd(d, B, x, None, nf.layer_params(w, b, None), y, ws)
    got = {r["kernel"] for r in nf.nf_prof_end()}
    if nf.nf_contraction() == nf.NF_CONTRACT_F32:
        assert kernel in got, got
    n = 5  # images against the sum in double precision, the last ones included
    pad = torch.nn.functional.pad(x[-n:].double(), (0, 0, 2, 2, 2, 2))
    col = pad.unfold(1, R, 1).unfold(2, R, 1).permute(0, 1, 2, 4, 5, 3).reshape(n * H * H, R * R * C)
    ref = (col @ w.double().reshape(K, -1).t() + b.double()).clamp_min(0).reshape(n, H, H, K)
    # 2100 products in fp32: the suite's 1e-4 of the largest value
    assert (y[-n:].double() - ref).abs().max() <= 1e-4 * ref.abs().max()
