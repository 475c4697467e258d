"""Statistics of closeness calls, on both kernels: vertices reached and their
arcs as the oracle counts them (repeated sources once per occurrence, several
passes, small and other components), the levels run, and the placement."""
import numpy as np
import pytest

import graphgen as gg
import oracle
import paper_1403_3005_amd as nk
from nkutil import ivec, upload

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _default_tuning():
    nk.nk_set_tuning()
    yield
    nk.nk_set_tuning()


CASES = [   # graph, sources (0: the exact form), placement, passes
    (lambda: gg.rmat(13, 16, 1), 40, 8, 1), (lambda: gg.barabasi_albert(20011, 6, 3), 1025, 8, 2),
    (lambda: gg.disjoint_union([gg.rmat(12, 16, 7), gg.cycle(40), gg.path(1), gg.star(700), gg.complete(60)]), 2100, 8, 3),
    (lambda: gg.erdos_renyi(3000, 40000, 10), 0, 8, 3),
    (lambda: gg.rmat(12, 16, 1), 8, 1, 0), (lambda: gg.path(4000), 1024, 1, 0),
]


@pytest.mark.parametrize("make,k,where,passes", CASES)
def test_counters(make, k, where, passes):
    g = make()
    rp, ci = upload(g)
    if k:
        src = np.concatenate([gg.sample_sources(g.n, k - 2, 8), [0, 0]])
        nk.nk_closeness_sampled(rp, ci, ivec(src))
    else:
        src = np.arange(g.n)
        nk.nk_closeness(rp, ci)
    st = nk.nk_last_stats()
    reached, arcs, _, _ = oracle.work_counts(g.rowptr, g.colidx, src)
    assert (st["bitmap_lds"], st["sources"], st["reached"], st["arcs_reached"]) == (where, len(src), reached, arcs)
    if where == 8:
        depth = sum(max(oracle.work_counts(g.rowptr, g.colidx, np.array([s]))[3] for s in src[a:a + 1024])
                    for a in range(0, len(src), 1024))
        assert st["levels_bu"] == depth + passes          # each pass runs the level that finds nothing
        # a level of a pass looks at an arc once, and one of those it looks at finds each vertex
        assert g.m > 0 and st["arcs_fwd"] <= g.m * st["levels_bu"] and st["arcs_fwd"] > 0


def test_a_bad_graph_leaves_no_counts():
    g = gg.rmat(13, 16, 2)
    rp, ci = upload(g)
    ci[7] = g.n
    with pytest.raises(nk.NkError) as e:
        nk.nk_closeness_sampled(rp, ci, ivec(np.arange(200)))
    assert e.value.code == nk.NK_E_INVALID_GRAPH and nk.nk_last_stats()["reached"] == 0
