"""Logits that nf_aux_predict reports, against 64 bits: one sum of F products per class, over pooled features that
are exact (a 1x1 head convolution that copies channels, pooling windows of one pixel)."""
import numpy as np
import pytest
import torch

from paper_2402_14139_amd import binding as nf

pytestmark = pytest.mark.gpu


def emulated(q, w, b):
    """The same sums in float32: 64 running sums of every 64th product, then a tree (products rounded: the
    kernel, which fuses them, has no more roundings)."""
    prod = (q[:, None, :] * w[None]).astype(np.float32)
    pad = np.zeros((*prod.shape[:2], -prod.shape[2] % 64), np.float32)
    prod = np.concatenate([prod, pad], 2).reshape(*prod.shape[:2], -1, 64)
    acc = np.zeros_like(prod[:, :, 0])
    for i in range(prod.shape[2]):
        acc = acc + prod[:, :, i]
    while acc.shape[2] > 1:
        acc = acc[..., 0::2] + acc[..., 1::2]
    return acc[..., 0] + b


# (filters, pooled map, classes): features a multiple of 4 or not, fewer and more than 64, classes around 64 and 256
@pytest.mark.parametrize("A,o,cls", [(256, 2, 100), (512, 2, 200), (256, 2, 300), (129, 2, 37), (67, 1, 65), (321, 1, 10),
                                     (3, 1, 1), (16, 2, 64)])
def test_exit_logits_keep_short_sums(A, o, cls):
    B, C = 33, 4
    g = torch.Generator(device="cuda").manual_seed(A + cls)
    rn = lambda *s: torch.randn(*s, generator=g, device="cuda")  # noqa: E731
    d = nf.LayerDesc(C_in=C, H_in=o, W_in=o, C_out=C, R=3, S=3, stride=1, pad=1)
    a = nf.AuxDesc(C_in=C, H_in=o, W_in=o, A=A, R=1, S=1, pad=0, relu=0, pool_oh=o, pool_ow=o, n_classes=cls)
    F, y = o * o * A, rn(B, o, o, C)
    copied = torch.arange(A, device="cuda") % C
    Wa = torch.zeros(A, 1, 1, C, device="cuda")
    Wa[torch.arange(A), 0, 0, copied] = 1.0
    Wf, bf = rn(cls, F) * (2.0 / F) ** 0.5, rn(cls) * 0.1
    logits, pred = torch.empty(B, cls, device="cuda"), torch.empty(B, dtype=torch.int32, device="cuda")
    ws = torch.empty(nf.nf_workspace_bytes(d, a, B), dtype=torch.uint8, device="cuda")
    nf.nf_aux_predict(d, a, B, y, None, nf.aux_params(Wa, torch.zeros(A, device="cuda"), Wf, bf), pred, None, False, logits, ws)
    q, w, b = y[..., copied].reshape(B, F).cpu().numpy(), Wf.cpu().numpy(), bf.cpu().numpy()
    ref = q.astype(np.float64) @ w.T.astype(np.float64) + b
    got = logits.cpu().numpy()
    rel = lambda v: np.linalg.norm(v - ref) / np.linalg.norm(ref)  # noqa: E731
    # the emulation's error, a quarter more for the spread of B * cls results with other roundings; few results: twice
    assert rel(got) <= (1.25 if B * cls > 1000 else 2.0) * rel(emulated(q, w, b))
    assert np.array_equal(pred.cpu().numpy(), got.argmax(1))
