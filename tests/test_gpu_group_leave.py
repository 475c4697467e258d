"""A group launch whose workgroups leave before they start (another launch
holds the device): the call must end on another kernel with the right scores
and the counters of that run alone, whatever part of the grid had registered
by then -- few sources, the sparse mid-size range and the kernel asked for by
flag."""
import pytest

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


@pytest.mark.parametrize("make,k,flags", [
    (lambda: gg.rmat(17, 8, 1), 8, 0),
    (lambda: gg.erdos_renyi(100_000, 400_000, 2), 300, 0),
    (lambda: gg.rmat(13, 12, 6), 24, 4 | 8),
])
@pytest.mark.parametrize("block", [0, 512])
def test_leave(make, k, flags, block):
    g = make()
    if block and not flags:
        flags = 8            # (a set block leaves the automatic choice to the one-source kernel)
    rp, ci = upload(g)
    src = gg.sample_sources(g.n, k, 5)
    ref = oracle.bc_sources(g.rowptr, g.colidx, src, 1.0, nthreads=16)
    reached, arcs, dag, _ = oracle.work_counts(g.rowptr, g.colidx, src)
    for leave, where in ((0, 6), (128, 1), (0, 6)):
        nk.nk_set_tuning(flags=flags | leave, block=block)
        got = nk.nk_bc_sources(rp, ci, ivec(src), 1.0).cpu().numpy()
        st = nk.nk_last_stats()
        assert st["bitmap_lds"] == where, (leave, st)
        assert (st["sources"], st["reached"], st["arcs_reached"], st["dag_arcs"]) == (k, reached, arcs, dag)
        assert_scores_close(got, ref, f"leave {leave}")
