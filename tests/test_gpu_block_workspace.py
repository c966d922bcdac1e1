"""A block call in a workspace larger than its plan: the layers get all of it and nothing beyond it."""
import pytest
import torch

from paper_2402_14139_amd import binding as nf
from paper_2402_14139_amd.layer import LocalLayer

pytestmark = pytest.mark.gpu
CLS, A, GUARD = 10, 8, 1 << 16


def layers(n, C, H, B, momentum=False):
    g = torch.Generator().manual_seed(C + n)
    rn = lambda *s: torch.randn(*s, generator=g)  # noqa: E731
    out = []
    for _ in range(n):
        d = nf.LayerDesc(C_in=C, H_in=H, W_in=H, C_out=C, R=3, S=3, stride=1, pad=1)
        a = nf.AuxDesc(C_in=C, H_in=H, W_in=H, A=A, R=3, S=3, pad=1, relu=1, pool_oh=2, pool_ow=2, n_classes=CLS)
        p = dict(W=rn(C, 3, 3, C) * (2 / (9 * C)) ** 0.5, b=rn(C) * 0.1, Wp=None, Wa=rn(A, 3, 3, C) * 0.05, ba=rn(A) * 0.1,
                 Wf=rn(CLS, 4 * A) * 0.2, bf=rn(CLS) * 0.1)
        out.append(LocalLayer(d, a, {k: None if v is None else v.numpy() for k, v in p.items()}, B, momentum))
    return out


def block(ls, train):
    col = lambda name: [getattr(l, name) for l in ls]  # noqa: E731
    return nf.make_block(col("d"), col("a") if train else None, [-1] * len(ls), col("sp"), col("sa") if train else None,
                         col("sgp") if train else None, col("sga") if train else None)


def guarded(nbytes):
    """(workspace of nbytes filled with NaN, the bytes behind it)"""
    buf = torch.full(((nbytes + GUARD + 3) // 4 * 4,), 0xFF, dtype=torch.uint8, device="cuda")
    return buf[:nbytes], buf[nbytes:]


ROOMY = 200 << 20


# a batch of 256 and one of 88, whose reduction is cut where its scratch has room (8 MiB more hold its direct kernel only); and a
# partial batch of one sample
@pytest.mark.parametrize("C,H,B,items,extra", [(256, 8, 256, 344, 8 << 20), (256, 8, 256, 344, (24 << 20) + 12), (256, 8, 256, 344, ROOMY),
                                               (128, 16, 96, 97, 0), (128, 16, 96, 97, 256), (128, 16, 96, 97, ROOMY)])
def test_sweep_gives_its_layers_the_whole_workspace(C, H, B, items, extra):
    ls = layers(2, C, H, B)
    blk = block(ls, False)
    x = torch.randn(items, H, H, C, generator=torch.Generator(device="cuda").manual_seed(1), device="cuda").relu_()
    labels = torch.zeros(items, dtype=torch.int32, device="cuda")
    out, lab = torch.empty(items, H * H * C, device="cuda"), torch.empty(items, dtype=torch.int32, device="cuda")
    ws, behind = guarded(nf.nf_block_workspace_bytes(blk, B) + extra)
    nf.nf_prof_begin()
    nf.nf_block_fill_cache(blk, B, items, x, labels, items, out, lab, items, ws)
    names = {r["kernel"]: r["launches"] for r in nf.nf_prof_end()}
    assert bool((behind == 0xFF).all())
    t = x[items // B * B:]
    nf.nf_prof_begin()
    for l in ls:  # each in a workspace of its own that its plan asks for
        t = l.forward(t)
    alone = {r["kernel"]: r["launches"] for r in nf.nf_prof_end()}
    got, own = out[items // B * B:], t.reshape(items % B, -1)
    if extra == ROOMY:  # room for everything: the same kernels, the same bits
        assert torch.equal(got, own)
        assert all(names.get(k, 0) >= n for k, n in alone.items()), (names, alone)
    # sums of 9 C products in other orders, two layers: a few 1e-7 of the norm
    assert float((got - own).norm()) <= 4e-6 * float(own.norm())


@pytest.mark.parametrize("extra", [0, (24 << 20) + 12])
def test_epoch_in_a_larger_workspace(extra):
    C, H, B, items = 256, 8, 256, 344
    ls = layers(2, C, H, B)
    blk = block(ls, True)
    g = torch.Generator(device="cuda").manual_seed(2)
    x = torch.randn(items, H * H * C, generator=g, device="cuda").relu_()
    labels = torch.randint(0, CLS, (items,), generator=g, device="cuda", dtype=torch.int32)
    losses = torch.zeros(2, len(ls), device="cuda")
    ws, behind = guarded(nf.nf_block_workspace_bytes(blk, B) + extra)
    nf.nf_block_train_epoch(blk, 0.01, 0.0, B, items, x, labels, items, None, losses, ws)
    assert bool((behind == 0xFF).all())
    ref = layers(2, C, H, B)
    for b in range(2):
        t = x[b * B:(b + 1) * B].reshape(-1, H, H, C)
        for i, l in enumerate(ref):
            t = l.step(t, None, labels[b * B:(b + 1) * B], 0.01, 0.0)
            assert abs(float(l.loss) - float(losses[b, i])) <= 1e-5 * abs(float(l.loss))
    for l, r in zip(ls, ref):
        for k in ("W", "Wa", "Wf"):
            # one update of 0.01 times a gradient whose sums ran in another order
            assert float((l.p[k] - r.p[k]).norm()) <= 1e-5 * float(r.p[k].norm())
