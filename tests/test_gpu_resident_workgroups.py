"""Workgroups that the per-source kernels keep on a compute unit: sixteen
waves, whatever the kind of call and the workgroup's size (a register more
than the share of a wave halves them)."""
import numpy as np
import pytest
import torch

import graphgen as gg
import paper_1403_3005_amd as nk
from nkutil import ivec, upload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("block", [256, 512, 1024])
def test_sixteen_waves_a_compute_unit(block):
    g = gg.erdos_renyi(20000, 80000, 3)
    rp, ci = upload(g)
    k = 4200
    s = ivec(np.arange(k))
    wt = torch.ones(g.m, dtype=torch.int32, device="cuda:0")
    units = torch.cuda.get_device_properties(0).multi_processor_count
    calls = {
        "sources": lambda: nk.nk_bc_sources(rp, ci, s, 1.0), "edges": lambda: nk.nk_edge_bc(rp, ci, s, 1.0),
        "directed": lambda: nk.nk_bc_directed(rp, ci, s, 1.0, rp, ci),
        "bisect": lambda: nk.nk_bc_sources_bisect(rp, ci, s, 1.0),
        "weighted": lambda: nk.nk_bc_weighted(rp, ci, wt, s, 1.0),
        "path counts": lambda: nk.nk_sssp_counts(rp, ci, s),
    }
    for name, call in calls.items():
        nk.nk_set_tuning(block=block, flags=4)                       # (not the kernels with the state in LDS)
        try:
            call()
        finally:
            nk.nk_set_tuning()
        st = nk.nk_last_stats()
        assert (st["block"], st["workgroups"]) == (block, units * 1024 // block), (name, st)
