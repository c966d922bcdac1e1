"""The 3x3 convolutions that run through F(2x2, 3x3) (csrc/wino_fwd.hip) and the weight gradients that
run through F(3x3, 2x2) (csrc/wino_wgrad.hip): whole steps against the CPU oracle at the sizes where
the tiling can go wrong, and values that are not finite."""
import numpy as np
import pytest
import torch

import workloads
from paper_2402_14139_amd import binding as nf
from tests import gpu_common as G
from tests.test_gpu_parity import S

pytestmark = pytest.mark.gpu

# name -> (spec, B, classes, how many of layer / head / data gradient run as wino_fwd)
CASES = {
    # ragged last tile block, last filter block of 4, odd map (a half-empty tile in both directions)
    "odd_map_n260": (S(64, 5, 7, 260, 8), 221, 10, 1),
    # channel count not a multiple of the step (8), identity shortcut
    "c68_identity": (S(256, 8, 8, 256, 4, skip=1), 25, 10, 1),
    "c68": (S(68, 8, 8, 256, 4), 64, 10, 1),
    # the narrowest map it takes, an odd one
    "map_4x5": (S(64, 4, 5, 256, 8), 317, 10, 1),
    # split reductions: layer (pooled), and all three of layer, head and data gradient
    "split_pool": (S(256, 8, 8, 256, 4, pool=(2, 2, 0)), 25, 10, 1),
    "split_wide_head": (S(256, 4, 4, 256, 256), 94, 10, 3),
    # projection shortcut: a launch of its own, added in the epilogue
    "projection": (S(128, 8, 8, 256, 4, skip=2, skip_C=36), 260, 10, 1),
    # fewer filters than a workgroup's 64 columns
    "n60": (S(128, 16, 16, 60, 4), 100, 10, 1),
}


@pytest.mark.parametrize("name", list(CASES))
def test_wino_steps_match_oracle(name):
    wino_step(name, *CASES[name])


def wino_step(name, spec, B, cls, launches):
    print(f"case {name}: B={B}", flush=True)
    nf.nf_prof_begin()
    out, final = G.run_step_both(spec, cls, B, seed=310, lr=0.05, mu=0.9, steps=1)
    got = {r["kernel"]: r["launches"] for r in nf.nf_prof_end()}
    G.check_step_results(name, out, final)
    if nf.nf_contraction() == nf.NF_CONTRACT_F32:
        assert got.get("wino_fwd", 0) >= launches, got


# name -> (spec, B, whether the 3x3 part's reduction is split)
PROJECTIONS = {
    # its sums lie in the output, where fwd_finish adds the parts of the 3x3 convolution to them
    "split_4": (S(256, 8, 8, 256, 8, skip=2, skip_C=128), 64, True),
    "split_2_pool": (S(256, 8, 8, 256, 8, pool=(2, 2, 0), skip=2, skip_C=128), 128, True),
    # channels that are not a multiple of 4: the general kernel, the first-layer kernel
    "skip_c34_split": (S(512, 4, 4, 512, 4, skip=2, skip_C=34), 128, True),
    "skip_c10": (S(128, 8, 8, 256, 4, skip=2, skip_C=10), 260, False),
}


@pytest.mark.parametrize("name", list(PROJECTIONS))
def test_wino_beside_a_projection_matches_oracle(name):
    spec, B, split = PROJECTIONS[name]
    print(f"case {name}: B={B}", flush=True)
    nf.nf_prof_begin()
    out, final = G.run_step_both(spec, 10, B, seed=312, lr=0.05, mu=0.9, steps=1)
    got = {r["kernel"] for r in nf.nf_prof_end()}
    G.check_step_results(name, out, final)
    if nf.nf_contraction() == nf.NF_CONTRACT_F32:
        assert "wino_fwd" in got and ("fwd_finish" in got) == split, got


@pytest.mark.parametrize("where", ["input", "filter"])
def test_wino_values_that_are_not_finite(where):
    """An infinity reaches exactly the results whose direct sum contains it."""
    B, C, H, W, K = 83, 64, 9, 8, 256
    g = torch.Generator().manual_seed(5)
    x, w = torch.randn(B, H, W, C, generator=g), torch.randn(K, 3, 3, C, generator=g) * 0.06
    if where == "input":
        x[1, 4, 5, 7], x[2, 0, 0, 3] = float("inf"), float("nan")
    else:
        w[200, 1, 1, 9] = float("inf")  # the centre tap: never over the padding
    ref = torch.nn.functional.conv2d(x.permute(0, 3, 1, 2).double(), w.permute(0, 3, 1, 2).double(), padding=1)
    ref = ref.permute(0, 2, 3, 1).numpy()
    ref = np.where(ref > 0, ref, 0.0)  # ReLU as the library takes it: NaN is not positive
    d = nf.LayerDesc(C_in=C, H_in=H, W_in=W, C_out=K, R=3, S=3, stride=1, pad=1)
    xd, wd, bd = x.cuda(), w.cuda(), torch.zeros(K, device="cuda")
    y = torch.empty(B, H, W, K, device="cuda")
    ws = torch.empty(nf.nf_workspace_bytes(d, None, B), dtype=torch.uint8, device="cuda")
    nf.nf_prof_begin()
    nf.nf_layer_fwd(d, B, xd, None, nf.layer_params(wd, bd, None), y, ws)
    names = {r["kernel"] for r in nf.nf_prof_end()}
    if nf.nf_contraction() != nf.NF_CONTRACT_F32:
        pytest.skip("the split modes turn an infinity into NaN")
    assert "wino_fwd" in names
    got = y.cpu().numpy().astype(np.float64)
    inf = np.isinf(ref)
    assert inf.any() and np.array_equal(np.isinf(got), inf)
    # finite results: 576 products of unit variance scale; 1e-4 is the suite's bar
    assert np.abs(got[~inf] - ref[~inf]).max() <= 1e-4 * np.abs(ref[~inf]).max()


def test_wino_values_that_are_not_finite_beside_a_projection():
    """The projection's sums lie where the results go: a result formed again still has its own."""
    B, C, H, K, Cs = 260, 128, 8, 256, 36
    g = torch.Generator(device="cuda").manual_seed(13)
    rn = lambda *s: torch.randn(*s, generator=g, device="cuda")  # noqa: E731
    x, xs, w, b, wp = rn(B, H, H, C), rn(B, 2 * H, 2 * H, Cs), rn(K, 3, 3, C) * 0.04, rn(K), rn(K, Cs) * 0.2
    x[7, 3, 4, 5] = float("inf")
    d = nf.LayerDesc(C_in=C, H_in=H, W_in=H, C_out=K, R=3, S=3, stride=1, pad=1, skip_kind=2, skip_C=Cs,
                     skip_H=2 * H, skip_W=2 * H, skip_stride=2)
    need, ys, names = nf.nf_workspace_bytes(d, None, B), [], []
    for nbytes in (need, need - 256):  # the second one only holds the direct kernels
        ws = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
        y = torch.full((B, H, H, K), -1.0, device="cuda")
        nf.nf_prof_begin()
        nf.nf_layer_fwd(d, B, x, xs, nf.layer_params(w, b, wp), y, ws)
        names.append({r["kernel"] for r in nf.nf_prof_end()})
        ys.append(y)
    if nf.nf_contraction() != nf.NF_CONTRACT_F32:
        pytest.skip("the split modes turn an infinity into NaN")
    assert "wino_fwd" in names[0] and "wino_fwd" not in names[1], names
    inf = torch.isinf(ys[1])
    assert inf.any() and torch.equal(torch.isinf(ys[0]), inf) and not torch.isnan(ys[0]).any()
    # 1188-term sums in two orders: a few 1e-7 of the largest value
    assert (ys[0] - ys[1])[~inf].abs().max() <= 5e-6 * ys[1][~inf].abs().max()


def test_wino_results_of_filters_that_are_nan():
    """Whole filters of NaN, some beside finite ones in the group of four that a thread forms again."""
    B, C, H, K = 48, 64, 16, 256
    g = torch.Generator(device="cuda").manual_seed(12)
    x, w = torch.randn(B, H, H, C, generator=g, device="cuda"), torch.randn(K, 3, 3, C, generator=g, device="cuda") * 0.06
    d = nf.LayerDesc(C_in=C, H_in=H, W_in=H, C_out=K, R=3, S=3, stride=1, pad=1)
    b, ys = torch.full((K,), 30.0, device="cuda"), []  # every finite result positive: ReLU passes it
    ws = torch.empty(nf.nf_workspace_bytes(d, None, B), dtype=torch.uint8, device="cuda")
    bad = torch.zeros(K, dtype=torch.bool, device="cuda")
    bad[8:16], bad[21], bad[40:43] = True, True, True
    for nan in (False, True):
        if nan:
            w[bad] = float("nan")
        y = torch.empty(B, H, H, K, device="cuda")
        nf.nf_prof_begin()
        nf.nf_layer_fwd(d, B, x, None, nf.layer_params(w, b, None), y, ws)
        names = {r["kernel"] for r in nf.nf_prof_end()}
        ys.append(y)
    if nf.nf_contraction() == nf.NF_CONTRACT_F32:
        assert "wino_fwd" in names
    assert (ys[1][..., bad] == 0).all()  # ReLU as the library takes it: NaN is not positive
    assert (ys[0] > 0).all()
    # 576-term sums in two orders where a neighbour was NaN: a few 1e-7 of the largest value
    assert (ys[1] - ys[0])[..., ~bad].abs().max() <= 5e-6 * ys[0].abs().max()


def test_wino_padding_contributes_nothing():
    """An infinite weight at the rim of a filter reaches the pixels whose window holds a pixel under it, and no others."""
    B, C, H, K = 48, 64, 16, 256
    g = torch.Generator(device="cuda").manual_seed(15)
    x = torch.rand(B, H, H, C, generator=g, device="cuda") + 0.1
    w, b = torch.randn(K, 3, 3, C, generator=g, device="cuda") * 0.06, torch.full((K,), 50.0, device="cuda")
    w[200, 0, 2, 9] = float("inf")  # over the padding in the first row and the last column
    d = nf.LayerDesc(C_in=C, H_in=H, W_in=H, C_out=K, R=3, S=3, stride=1, pad=1)
    y = torch.empty(B, H, H, K, device="cuda")
    ws = torch.empty(nf.nf_workspace_bytes(d, None, B), dtype=torch.uint8, device="cuda")
    nf.nf_prof_begin()
    nf.nf_layer_fwd(d, B, x, None, nf.layer_params(w, b, None), y, ws)
    names = {r["kernel"] for r in nf.nf_prof_end()}
    if nf.nf_contraction() != nf.NF_CONTRACT_F32:
        pytest.skip("the split modes turn an infinity into NaN")
    assert "wino_fwd" in names
    inf = torch.zeros_like(y, dtype=torch.bool)
    inf[:, 1:, :-1, 200] = True
    assert torch.equal(torch.isinf(y), inf) and (y > 0).all()


def test_wino_wgrad_padding_contributes_nothing():
    """An infinite gradient at one corner pixel: the taps that lie over the padding there stay zero."""
    B, C, H, K, A = 64, 64, 16, 128, 8
    g = torch.Generator(device="cuda").manual_seed(16)
    z = lambda *s: torch.zeros(*s, device="cuda")  # noqa: E731
    d = nf.LayerDesc(C_in=C, H_in=H, W_in=H, C_out=K, R=3, S=3, stride=1, pad=1)
    a = nf.AuxDesc(C_in=K, H_in=H, W_in=H, A=A, R=3, S=3, pad=1, relu=1, pool_oh=2, pool_ow=2, n_classes=4, loss_kind=1)
    x, y = torch.rand(B, H, H, C, generator=g, device="cuda") + 0.1, z(B, H, H, K)
    y[3, 0, 0] = 1e-28  # the one pixel that passes the ReLU
    p = [z(K, 3, 3, C), z(K), z(A, 3, 3, K), z(A) + 1e-30, z(4, 4 * A), z(4)]
    p[2][5] = 0.01
    p[4][2, 5] = 3e38  # filter 5, first quadrant: a finite logit, an infinite gradient
    gr, labels, loss = [torch.zeros_like(t) for t in p], torch.zeros(B, device="cuda", dtype=torch.int32), z(1)
    lp, ap, gp, ga = nf.layer_params(*p[:2], None), nf.aux_params(*p[2:]), nf.layer_params(*gr[:2], None), nf.aux_params(*gr[2:])
    ws = torch.empty(nf.nf_workspace_bytes(d, a, B), dtype=torch.uint8, device="cuda")
    nf.nf_aux_fwd_loss(d, a, B, y, labels, ap, loss, ws)
    nf.nf_prof_begin()
    nf.nf_local_bwd_wgrad(d, a, B, x, None, y, lp, ap, gp, ga, ws)
    names = {r["kernel"] for r in nf.nf_prof_end()}
    if nf.nf_contraction() != nf.NF_CONTRACT_F32:
        pytest.skip("the split modes turn an infinity into NaN")
    assert "wino_wgrad" in names
    seen = torch.zeros(K, 3, 3, C, dtype=torch.bool, device="cuda")
    seen[:, 1:, 1:] = True
    assert torch.isinf(gr[0][seen]).all() and (gr[0][~seen] == 0).all()


# data gradients whose transformed filter comes from a head launch: the per-sample head, the wide one and the
# backward of a wide linear layer; channels of the head and of the layer that are not multiples of 8 and 64
DGRAD_CASES = {
    "head_sample_a20_k132": (S(8, 7, 7, 132, 20), 453, 10, 1),
    "head_wide_a20_k60": (S(8, 16, 16, 60, 20), 240, 10, 1),
    "head_wide_a32_k200_pool": (S(8, 20, 20, 200, 32, pool=(2, 2, 0)), 80, 10, 1),
    "head_bwd_a36_k68": (S(8, 12, 12, 68, 36), 200, 130, 1),
}


@pytest.mark.parametrize("name", list(DGRAD_CASES))
def test_wino_data_gradients_match_oracle(name):
    wino_step(name, *DGRAD_CASES[name])


def test_backward_in_a_larger_workspace_than_the_forward_call():
    """A head call whose workspace holds the direct kernels alone leaves no transformed filter; the
    backward call in one that holds everything forms its own."""
    B, H, K, A, cls = 128, 16, 64, 32, 10
    g = torch.Generator(device="cuda").manual_seed(8)
    rn = lambda *s: torch.randn(*s, generator=g, device="cuda")  # noqa: E731
    d = nf.LayerDesc(C_in=8, H_in=H, W_in=H, C_out=K, R=3, S=3, stride=1, pad=1)
    a = nf.AuxDesc(C_in=K, H_in=H, W_in=H, A=A, R=3, S=3, pad=1, relu=1, pool_oh=2, pool_ow=2, n_classes=cls)
    x, y = rn(B, H, H, 8), rn(B, H, H, K).relu()
    labels = torch.randint(0, cls, (B,), generator=g, device="cuda", dtype=torch.int32)
    p = [rn(K, 3, 3, 8) * 0.1, rn(K), rn(A, 3, 3, K) * 0.05, rn(A), rn(cls, 4 * A) * 0.2, rn(cls)]
    lp, ap = nf.layer_params(p[0], p[1], None), nf.aux_params(*p[2:])
    need = nf.nf_workspace_bytes(d, a, B)
    loss, res = torch.zeros(1, device="cuda"), []
    for fwd_bytes in (need, need - 16 * 64 * 32 * 4):
        ws = torch.full((need,), 0xFF, dtype=torch.uint8, device="cuda")  # NaN wherever nothing is written
        gr = [torch.zeros_like(t) for t in p]
        nf.nf_aux_fwd_loss(d, a, B, y, labels, ap, loss, ws[:fwd_bytes])
        nf.nf_local_bwd_wgrad(d, a, B, x, None, y, lp, ap, nf.layer_params(gr[0], gr[1], None), nf.aux_params(*gr[2:]), ws)
        res.append(gr[0].cpu().numpy().copy())
    assert np.abs(res[0]).max() > 0
    # (the head's sums may be cut differently: 1e-4 is the suite's bar)
    assert np.abs(res[1] - res[0]).max() <= 1e-4 * np.abs(res[0]).max()


WGRAD_CASES = {
    # odd maps (half-empty tiles), tiles of an image not a multiple of a step's four
    "odd_map_13x11": (S(64, 13, 11, 128, 4), 90, 10),
    # ragged channel (32) and filter (64) blocks, identity shortcut, pooled
    "c36_p132_pool": (S(36, 10, 9, 132, 4, pool=(2, 2, 0)), 574, 10),
    # narrowest map it takes, a last split shorter than the others
    "map_4x4_last_split": (S(96, 4, 4, 256, 4), 517, 10),
    # projection shortcut (its columns are a launch of their own)
    "projection": (S(128, 8, 8, 192, 4, skip=2, skip_C=68), 200, 10),
    # more than one addition to the result per split
    "several_periods": (S(256, 8, 8, 256, 4, skip=1), 160, 10),
}


@pytest.mark.parametrize("name", list(WGRAD_CASES))
def test_wino_weight_gradients_match_oracle(name):
    spec, B, cls = WGRAD_CASES[name]
    print(f"case {name}: B={B}", flush=True)
    nf.nf_prof_begin()
    out, final = G.run_step_both(spec, cls, B, seed=311, lr=0.05, mu=0.9, steps=1)
    got = {r["kernel"] for r in nf.nf_prof_end()}
    G.check_step_results(name, out, final)
    if nf.nf_contraction() == nf.NF_CONTRACT_F32:
        assert "wino_wgrad" in got, got


def test_wino_weight_gradient_of_an_infinite_input():
    """An infinity in the corner pixel reaches the four taps that see it, in its channel alone."""
    B, C, H, K, cls = 64, 64, 16, 128, 10
    g = torch.Generator(device="cuda").manual_seed(6)
    rn = lambda *s: torch.randn(*s, generator=g, device="cuda")  # noqa: E731
    d = nf.LayerDesc(C_in=C, H_in=H, W_in=H, C_out=K, R=3, S=3, stride=1, pad=1)
    a = nf.AuxDesc(C_in=K, H_in=H, W_in=H, A=8, R=3, S=3, pad=1, relu=0, pool_oh=2, pool_ow=2, n_classes=cls)
    x, y = rn(B, H, H, C), rn(B, H, H, K).abs() + 0.1  # every pixel passes the ReLU: no zero in dL/dZ
    labels = torch.randint(0, cls, (B,), generator=g, device="cuda", dtype=torch.int32)
    p = [rn(K, 3, 3, C) * 0.05, rn(K), rn(8, 3, 3, K) * 0.05, rn(8), rn(cls, 32) * 0.2, rn(cls)]
    gr = [torch.zeros_like(t) for t in p]
    lp, ap = nf.layer_params(p[0], p[1], None), nf.aux_params(*p[2:])
    gp, ga = nf.layer_params(gr[0], gr[1], None), nf.aux_params(*gr[2:])
    ws = torch.empty(nf.nf_workspace_bytes(d, a, B), dtype=torch.uint8, device="cuda")
    loss = torch.zeros(1, device="cuda")
    res = []
    for bad in (0.0, float("inf")):
        if bad:
            x[3, 0, 0, 37] = bad
        nf.nf_aux_fwd_loss(d, a, B, y, labels, ap, loss, ws)
        nf.nf_prof_begin()
        nf.nf_local_bwd_wgrad(d, a, B, x, None, y, lp, ap, gp, ga, ws)
        names = {r["kernel"] for r in nf.nf_prof_end()}
        res.append(gr[0].cpu().numpy().copy())
    if nf.nf_contraction() != nf.NF_CONTRACT_F32:
        pytest.skip("the split modes turn an infinity into NaN")
    assert "wino_wgrad" in names
    inf = np.zeros((K, 3, 3, C), bool)
    inf[:, :2, :2, 37] = True
    assert np.array_equal(np.isinf(res[1]), inf) and not np.isnan(res[1]).any()
    # the taps of that channel that do not see it lose the pixel's old value in neither run: compare all
    # other channels (1e-4: the suite's bar)
    keep = np.arange(C) != 37
    ref = res[0][..., keep]
    assert np.abs(res[1][..., keep] - ref).max() <= 1e-4 * np.abs(ref).max()
    tail = res[0][:, 2, :, 37]
    assert np.abs(res[1][:, 2, :, 37] - tail).max() <= 1e-4 * np.abs(ref).max()


def test_a_workspace_for_the_direct_kernels_alone_is_enough():
    """A workspace that holds no transformed filter runs the direct kernels, same result to rounding."""
    B, C, H, K = 64, 64, 16, 128
    g = torch.Generator(device="cuda").manual_seed(8)
    rn = lambda *s: torch.randn(*s, generator=g, device="cuda")  # noqa: E731
    x, w, b = rn(B, H, H, C), rn(K, 3, 3, C) * 0.06, rn(K)
    d = nf.LayerDesc(C_in=C, H_in=H, W_in=H, C_out=K, R=3, S=3, stride=1, pad=1)
    ys, names = [], []
    for nbytes in (nf.nf_workspace_bytes(d, None, B), 256):
        ws = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
        y = torch.empty(B, H, H, K, device="cuda")
        nf.nf_prof_begin()
        nf.nf_layer_fwd(d, B, x, None, nf.layer_params(w, b, None), y, ws)
        names.append({r["kernel"] for r in nf.nf_prof_end()})
        ys.append(y.cpu().numpy())
    if nf.nf_contraction() == nf.NF_CONTRACT_F32:
        assert "wino_fwd" in names[0] and "wino_fwd" not in names[1], names
    # 576-term sums in two orders: a few 1e-7 of the largest value
    assert np.abs(ys[0] - ys[1]).max() <= 5e-6 * np.abs(ys[0]).max()


def test_workspaces_between_the_least_and_the_full_plan():
    """Each gives up what does not fit and no more, and all give the same gradients to rounding.  (Wanted
    here: 122 MB, as much as lets the step stay in the static array; the direct kernels need 111 MB.)"""
    B, H, C, A, cls = 176, 32, 64, 32, 100
    g = torch.Generator(device="cuda").manual_seed(14)
    rn = lambda *s: torch.randn(*s, generator=g, device="cuda")  # noqa: E731
    d = nf.LayerDesc(C_in=C, H_in=H, W_in=H, C_out=C, R=3, S=3, stride=1, pad=1)
    # no ReLU in the head and a given activation: no decision that rounding could turn
    a = nf.AuxDesc(C_in=C, H_in=H, W_in=H, A=A, R=3, S=3, pad=1, relu=0, pool_oh=2, pool_ow=2, n_classes=cls)
    x, y = rn(B, H, H, C).relu(), rn(B, H, H, C).relu()
    labels = torch.randint(0, cls, (B,), generator=g, device="cuda", dtype=torch.int32)
    p = [rn(C, 3, 3, C) * 0.06, rn(C), rn(A, 3, 3, C) * 0.06, rn(A), rn(cls, 4 * A) * 0.2, rn(cls)]
    lp, ap, loss = nf.layer_params(p[0], p[1], None), nf.aux_params(*p[2:]), torch.zeros(1, device="cuda")
    want = nf.nf_workspace_bytes(d, a, B)
    names, grads = [], []
    for nbytes in (want, want - 256, 111600000 // 256 * 256, 111288576, 111288576 - 256):
        ws = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
        gr = [torch.zeros_like(t) for t in p]
        if nbytes < 111288576:
            with pytest.raises(Exception, match="workspace"):
                nf.nf_aux_fwd_loss(d, a, B, y, labels, ap, loss, ws)
            break
        nf.nf_prof_begin()
        nf.nf_aux_fwd_loss(d, a, B, y, labels, ap, loss, ws)
        nf.nf_local_bwd_wgrad(d, a, B, x, None, y, lp, ap, nf.layer_params(gr[0], gr[1], None), nf.aux_params(*gr[2:]), ws)
        names.append({r["kernel"] for r in nf.nf_prof_end()})
        grads.append([t.double() for t in gr])
    if nf.nf_contraction() == nf.NF_CONTRACT_F32:
        assert [[k in n for k in ("wino_wgrad", "wino_fwd")] for n in names] == [[True, True], [False, True], [False, True],
                                                                                [False, False]], names
    for other in grads[1:]:
        for u, v in zip(grads[0], other):
            # sums of 180 224 products in other orders: some 1e-7 of the norm each
            assert (u - v).norm() <= 2e-6 * u.norm()


@pytest.mark.parametrize("B,H,K,A,cls", [(128, 16, 64, 32, 10), (453, 7, 132, 20, 10)])
def test_a_head_call_of_its_own_leaves_no_transformed_filter(B, H, K, A, cls):
    """Nothing would read it: the backward call forms its own.  (The wide head and the per-sample one.)"""
    g = torch.Generator(device="cuda").manual_seed(15)
    rn = lambda *s: torch.randn(*s, generator=g, device="cuda")  # noqa: E731
    d = nf.LayerDesc(C_in=8, H_in=H, W_in=H, C_out=K, R=3, S=3, stride=1, pad=1)
    a = nf.AuxDesc(C_in=K, H_in=H, W_in=H, A=A, R=3, S=3, pad=1, relu=1, pool_oh=2, pool_ow=2, n_classes=cls)
    labels = torch.randint(0, cls, (B,), generator=g, device="cuda", dtype=torch.int32)
    ap = nf.aux_params(rn(A, 3, 3, K) * 0.05, rn(A), rn(cls, 4 * A) * 0.2, rn(cls))
    y, written = rn(B, H, H, K).relu(), []
    need = nf.nf_workspace_bytes(d, a, B)
    for nbytes in (need, need - 16 * 64 * -(-K // 64) * 8 * -(-A // 8) * 4):  # the second one has no room for it
        ws = torch.full((nbytes,), 0xFF, dtype=torch.uint8, device="cuda")
        nf.nf_aux_fwd_loss(d, a, B, y, labels, ap, torch.zeros(1, device="cuda"), ws)
        written.append(int((ws.view(torch.int32) != -1).sum()))
    assert written[0] == written[1], written
