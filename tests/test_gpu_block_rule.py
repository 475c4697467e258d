"""The automatic block size at both sides of each of its lines -- vertices,
arcs a vertex, sources -- against the CPU oracle and against the other
sizes."""
import numpy as np
import pytest
import torch

import graphgen as gg
import oracle
import paper_1403_3005_amd as nk
from nkutil import assert_scores_close, ivec, upload

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _default_tuning():
    nk.nk_set_tuning()
    yield
    nk.nk_set_tuning()


CASES = [  # graph, sources, block of the edge run, of the weighted run
    (lambda: gg.erdos_renyi(999, 6000, 1), 4, 256, 256), (lambda: gg.erdos_renyi(1000, 6000, 1), 4, 512, 512),
    (lambda: gg.erdos_renyi(1999, 9000, 2), 300, 256, 256), (lambda: gg.erdos_renyi(2000, 9000, 2), 300, 512, 512),
    (lambda: gg.erdos_renyi(2000, 9000, 2), 600, 512, 256),
    (lambda: gg.erdos_renyi(4000, 12000, 3), 8, 1024, 1024), (lambda: gg.erdos_renyi(4000, 11999, 3), 8, 256, 256),
    (lambda: gg.erdos_renyi(4000, 12000, 3), 257, 512, 512),
    (lambda: gg.erdos_renyi(20000, 120000, 4), 8, 1024, 1024), (lambda: gg.erdos_renyi(20000, 119999, 4), 260, 512, 512),
    (lambda: gg.erdos_renyi(20000, 120000, 4), 260, 1024, 1024), (lambda: gg.random_tree(20000, 5), 8, 512, 512),
]


@pytest.mark.parametrize("make,k,edge_block,weighted_block", CASES)
def test_block_and_scores(make, k, edge_block, weighted_block):
    g = make()
    rp, ci = upload(g)
    src = gg.sample_sources(g.n, k, 7)
    ebc, _ = nk.nk_edge_bc(rp, ci, ivec(src), 1.5)
    assert nk.nk_last_stats()["block"] == edge_block
    assert_scores_close(ebc.cpu().numpy(), oracle.edge_bc(g.rowptr, g.colidx, src, 1.5, nthreads=8)[0], "edges")
    w = gg.edge_weights(g, 20, 8, symmetric=True)
    wt = torch.from_numpy(np.ascontiguousarray(w, dtype=np.int32)).to("cuda:0")
    got = nk.nk_bc_weighted(rp, ci, wt, ivec(src), 1.5)
    assert nk.nk_last_stats()["block"] == weighted_block
    if k < 100:
        assert_scores_close(got.cpu().numpy(), oracle.bc_weighted(g.rowptr, g.colidx, w, src, 1.5, nthreads=8), "weighted")
    d1, s1 = nk.nk_sssp_counts(rp, ci, ivec(src[:300]))
    for block in (256, 512, 1024):
        nk.nk_set_tuning(block=block)
        assert_scores_close(nk.nk_bc_weighted(rp, ci, wt, ivec(src), 1.5).cpu().numpy(), got.cpu().numpy(), f"{block}")
        d, s = nk.nk_sssp_counts(rp, ci, ivec(src[:300]))
        assert torch.equal(d, d1) and torch.equal(s, s1)
