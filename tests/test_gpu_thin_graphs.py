"""Graphs of many narrow levels under the launch shapes chosen for wide ones:
the launch leaves and the call starts over, with the scores and counters of
the second run alone -- every kind of call, thin graphs, a thin component
among others, and both sides of the line (vertices found in 32 levels)."""
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


def _cliques(count, size):
    """Cliques in a chain: a level holds one vertex, then size - 1, in turn."""
    i, j = np.triu_indices(size, 1)
    base = np.arange(count)[:, None] * size
    ends = np.arange(1, count) * size
    return gg.from_edges(count * size, np.concatenate([(base + i).ravel(), ends - 1]),
                         np.concatenate([(base + j).ravel(), ends]), f"{count} cliques of {size}")


WIDE = gg.rmat(13, 16, 3)
GRAPHS = [   # graph, whether the launch leaves
    (lambda: _cliques(400, 8), True), (lambda: _cliques(150, 16), True),
    (lambda: _cliques(60, 96), False),                               # 32 levels hold over 1024 vertices
    (lambda: gg.disjoint_union([WIDE, _cliques(300, 8)]), True), (lambda: WIDE, False),
]


def _auto(g, k):
    """The block size by the vertices alone."""
    return 256 if g.n < 20000 else 512


@pytest.mark.parametrize("make,leaves", GRAPHS)
@pytest.mark.parametrize("k", [40, 700])
def test_calls(make, leaves, k):
    g = make()
    rp, ci = upload(g)
    src = gg.sample_sources(g.n, k, 7)
    src[:8] = g.n - 1 - 9 * np.arange(8)                             # (in the chain, where there is one)
    s = ivec(src)

    nk.nk_set_tuning(flags=4)                                        # (not the all-in-LDS kernel)

    def same(counters=True):
        st = nk.nk_last_stats()
        assert (st["block"] == _auto(g, k)) == leaves, st
        if counters:
            reached, arcs, _, _ = oracle.work_counts(g.rowptr, g.colidx, src)
            assert (st["sources"], st["reached"], st["arcs_reached"]) == (k, reached, arcs)

    ebc, bc = nk.nk_edge_bc(rp, ci, s, 1.5)
    same()
    ref_e, ref_v = oracle.edge_bc(g.rowptr, g.colidx, src, 1.5, nthreads=16)
    assert_scores_close(ebc.cpu().numpy(), ref_e, "edges")
    assert_scores_close(bc.cpu().numpy(), ref_v, "vertices of the edge run")
    assert_scores_close(nk.nk_bc_directed(rp, ci, s, 1.5, rp, ci).cpu().numpy(), ref_v, "directed")
    same()
    assert_scores_close(nk.nk_bc_sources_bisect(rp, ci, s, 2.0).cpu().numpy(),
                        oracle.bc_sources_bisect(g.rowptr, g.colidx, src, 2.0, nthreads=16), "bisect")
    same()
    d, sg = nk.nk_sssp_counts(rp, ci, s[:60])
    for i in range(0, min(k, 60), 7):
        od, os_ = oracle.sssp_counts(g.rowptr, g.colidx, int(src[i]))
        assert np.array_equal(d[i].cpu().numpy(), od)
        assert np.array_equal(sg[i].cpu().numpy().view(np.uint64), os_)
    w = gg.edge_weights(g, 1_000_000, 8, symmetric=True)                # (few ties: few paths)
    wt = torch.from_numpy(np.ascontiguousarray(w, dtype=np.int32)).to("cuda:0")
    assert_scores_close(nk.nk_bc_weighted(rp, ci, wt, s, 1.5).cpu().numpy(),
                        oracle.bc_weighted(g.rowptr, g.colidx, w, src, 1.5, nthreads=16), "weighted")
    nk.nk_set_tuning(scratch_mib=1, flags=4)                                  # (too little for the bit-parallel searches)
    got = nk.nk_closeness_sampled(rp, ci, s).cpu().numpy()
    assert np.allclose(got, oracle.closeness_approx(g.rowptr, g.colidx, src)[0], rtol=1e-14, atol=0.0)


@pytest.mark.parametrize("make,k,where", [
    (lambda: _cliques(8300, 8), 16, 1), (lambda: _cliques(8300, 8), 128, 1),
    (lambda: gg.disjoint_union([gg.rmat(17, 8, 1), _cliques(100, 8)]), 40, 1),
    (lambda: gg.disjoint_union([gg.rmat(17, 8, 1), _cliques(15, 8)]), 40, 6),   # 32 levels or fewer
])
def test_few_sources(make, k, where):
    g = make()
    rp, ci = upload(g)
    src = gg.sample_sources(g.n, k, 7)
    src[:3] = g.n - 1 - np.arange(3)
    got = nk.nk_bc_sources(rp, ci, ivec(src), 1.25).cpu().numpy()
    st = nk.nk_last_stats()
    assert st["bitmap_lds"] == where
    reached, arcs, dag, depth = oracle.work_counts(g.rowptr, g.colidx, src)
    assert (st["sources"], st["reached"], st["arcs_reached"], st["dag_arcs"]) == (k, reached, arcs, dag)
    assert st["levels_td"] + st["levels_bu"] == depth + k
    assert_scores_close(got, oracle.bc_sources(g.rowptr, g.colidx, src, 1.25, nthreads=16), "few")


def test_errors_of_the_second_run():
    g = _cliques(400, 8)
    rp, ci = upload(g)
    with pytest.raises(nk.NkError) as e:
        nk.nk_edge_bc(rp, ci, ivec([5] * 40 + [g.n]), 1.0)
    assert e.value.code == nk.NK_E_INVALID_ARG
    ci2 = ci.clone()
    ci2[0] = 9                                                       # the reverse of arc 0 is missing
    with pytest.raises(nk.NkError) as e:
        nk.nk_edge_bc(rp, ci2, ivec(np.arange(40)), 1.0)
    assert e.value.code == nk.NK_E_INVALID_GRAPH
