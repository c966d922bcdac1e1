"""Workspace sizes of the layers of every configuration (host functions only)."""
import pytest

import workloads
from paper_2402_14139_amd import binding as nf


@pytest.mark.parametrize("cfg_name", ["cfg2", "cfg3", "cfg4", "cfg5"])
def test_workspaces_of_smaller_batches_fit(cfg_name):
    """A block's workspace is sized at its batch size; the pass over a partial last batch must fit it
    (the planned kernels, and with them the scratch, depend on the batch)."""
    cfg = workloads.config(cfg_name)
    for blk in cfg.blocks:
        for i in blk.layers:
            spec = cfg.layers[i]
            d = nf.LayerDesc(**spec.layer_desc_fields())
            a = nf.AuxDesc(**spec.aux_desc_fields(cfg.n_classes))
            full = nf.nf_workspace_bytes(d, a, blk.batch)
            for b in {1, 3, blk.batch // 8, blk.batch // 4, blk.batch // 2, blk.batch - 1}:
                assert nf.nf_workspace_bytes(d, a, max(b, 1)) <= full, (cfg_name, spec.name, b)


@pytest.mark.parametrize("cfg_name", ["cfg2", "cfg3", "cfg4", "cfg5"])
def test_no_layer_is_pushed_out_of_the_static_scratch(cfg_name):
    """All layers of the configurations run through nf_local_step_static (115 MiB at most without the
    scratch of the transformed contractions)."""
    cfg = workloads.config(cfg_name)
    for blk in cfg.blocks:
        for i in blk.layers:
            spec = cfg.layers[i]
            d = nf.LayerDesc(**spec.layer_desc_fields())
            a = nf.AuxDesc(**spec.aux_desc_fields(cfg.n_classes))
            assert nf.nf_workspace_bytes(d, a, blk.batch) <= nf.NF_STATIC_SCRATCH_BYTES, (cfg_name, spec.name)


def layer(C, H, W, K, A, R, pool, skip, classes):
    """(layer, head) descriptors; pool 0 / 2 (2x2) / 3 (3x3, stride 2), skip 0 / 1 (identity) / 2 (projection of C/2)."""
    pk, ps, pp = {0: (0, 0, 0), 2: (2, 2, 0), 3: (3, 2, 1)}[pool]
    Hp, Wp = ((n + 2 * pp - pk) // ps + 1 if pool else n for n in (H, W))
    sk = {0: (0, 0, 0, 0), 1: (K, H, W, 1), 2: (C // 2, 2 * H, 2 * W, 2)}[skip]
    d = nf.LayerDesc(C_in=C, H_in=H, W_in=W, C_out=K, R=R, S=R, stride=1, pad=R // 2, pool_kind=int(pool > 0), pool_k=pk,
                     pool_stride=ps, pool_pad=pp, skip_kind=skip, skip_C=sk[0], skip_H=sk[1], skip_W=sk[2], skip_stride=sk[3])
    return d, nf.AuxDesc(C_in=K, H_in=Hp, W_in=Wp, A=A, R=3, S=3, pad=1, relu=1, pool_oh=2, pool_ow=2, n_classes=classes)


# (layer, batch) whose direct kernels' scratch, the last figure, is just below the static array's size and whose
# transformed contractions would need more
NEAR_THE_LIMIT = [
    ((64, 22, 22, 192, 64, 3, 0, 0, 10), 166, 134197248),
    ((192, 10, 10, 96, 128, 3, 0, 0, 10), 535, 134217472),
    ((32, 6, 6, 384, 5, 3, 0, 0, 100), 1839, 134175232),
    ((64, 4, 4, 512, 8, 3, 0, 1, 200), 2728, 134205440),
    ((32, 7, 7, 512, 5, 3, 2, 0, 10), 871, 134208256),
    ((32, 20, 20, 256, 16, 3, 3, 2, 10), 178, 134206208),
    # heads of few filters, whose weight gradient takes more splits than it needs
    ((512, 56, 56, 4, 16, 5, 2, 0, 200), 641, 134208512),
    ((28, 31, 32, 4, 16, 5, 3, 0, 10), 2319, 134188288),
    ((32, 59, 59, 4, 12, 3, 2, 0, 200), 850, 134099456),
]


@pytest.mark.parametrize("shape,B,direct", NEAR_THE_LIMIT)
def test_what_the_direct_kernels_fit_is_not_pushed_out(shape, B, direct):
    assert direct <= nf.NF_STATIC_SCRATCH_BYTES
    assert nf.nf_workspace_bytes(*layer(*shape), B) <= nf.NF_STATIC_SCRATCH_BYTES


# (layer, batch) whose full plan is larger than the static array: what fits of it stays (the last figure: the
# scratch of the direct kernels)
BETWEEN = [
    ((64, 56, 56, 64, 32, 3, 0, 0, 100), 64, 118730752),
    ((64, 32, 32, 64, 32, 3, 0, 0, 100), 176, 111288576),
    ((64, 32, 32, 64, 32, 3, 0, 0, 100), 216, 132972800),
    ((64, 32, 32, 64, 64, 3, 0, 0, 100), 128, 117668352),
]


@pytest.mark.parametrize("shape,B,direct", BETWEEN)
def test_a_plan_that_does_not_fit_gives_up_a_part(shape, B, direct):
    assert direct < nf.nf_workspace_bytes(*layer(*shape), B) <= nf.NF_STATIC_SCRATCH_BYTES


@pytest.mark.parametrize("shape,B,direct", [((512, 16, 16, 64, 4, 3, 0, 2, 10), 39, 11084544),
                                            ((384, 6, 6, 60, 5, 3, 0, 2, 100), 380, 12166144),
                                            ((512, 33, 33, 64, 4, 3, 0, 0, 10), 9, 11777024)])
def test_scratch_at_most_doubles(shape, B, direct):
    """Partial sums of the transformed weight gradient against what the direct kernels need."""
    assert nf.nf_workspace_bytes(*layer(*shape), B) <= 2 * direct


@pytest.mark.parametrize("shape,B,planned", [((180, 34, 34, 128, 4, 3, 0, 0, 10), 62, 78599936),
                                             ((336, 13, 13, 128, 4, 3, 0, 0, 10), 52, 41464320),
                                             ((72, 21, 21, 48, 4, 3, 0, 0, 10), 167, 39490304)])
def test_splits_of_the_weight_gradient_fill_whole_rounds(shape, B, planned):
    """12, 22 and 3 blocks of filters and channels: 42, 11 and 170 splits make 504, 242 and 510 workgroups for
    512 or 256 places.  One more split (the scratch would show it) leaves a second round to a handful."""
    assert nf.nf_workspace_bytes(*layer(*shape), B) <= planned


def test_a_head_takes_no_more_parts_than_its_direct_kernel():
    """7 samples of 32x31: the direct head convolution is not cut, and a pooling launch with 28 windows would add the
    parts of a cut one (the scratch would show them)."""
    assert nf.nf_workspace_bytes(*layer(4, 32, 31, 128, 80, 1, 0, 0, 10), 7) <= 28820480
