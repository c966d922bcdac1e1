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
