"""State-in-LDS kernel on a graph whose arcs lead into vertices without arcs of
their own (not symmetric, so outside the undirected forms' contract): every
kernel treats such vertices as reached by nothing, which leaves the scores of
the symmetric part, and no access leaves the state's arrays."""
import numpy as np
import pytest

import graphgen as gg
import oracle
import paper_1403_3005_amd as nk
from nkutil import assert_scores_close, ivec

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _default_tuning():
    nk.nk_set_tuning()
    yield
    nk.nk_set_tuning()


@pytest.mark.parametrize("n,live", [(9000, 8995), (9000, 7000), (40000, 9000), (40000, 20000), (40000, 39999),
                                    (65534, 40000)])
@pytest.mark.parametrize("flags", [0, 2])
def test_arcs_into_bare_vertices(n, live, flags):
    core = gg.erdos_renyi(live, 2 * live, 5)
    r = np.random.default_rng(n + live)
    # a third of the core's vertices with arcs get one into a vertex past it
    extra = (core.degrees() > 0) & (r.random(live) < 0.34)
    deg = np.concatenate([core.degrees() + extra, np.zeros(n - live, dtype=np.int64)])
    rowptr = np.concatenate([[0], np.cumsum(deg)]).astype(np.int32)
    colidx = np.empty(rowptr[-1], dtype=np.int32)
    last = rowptr[1:live + 1][extra] - 1
    own = np.ones(len(colidx), dtype=bool)
    own[last] = False
    colidx[own] = core.colidx
    colidx[last] = r.integers(live, n, int(extra.sum()))
    rp, ci = ivec(rowptr), ivec(colidx)
    src = r.choice(live, 40, replace=False)
    src = src[core.degrees()[src] > 0]
    want = np.zeros(n)
    want[:live] = oracle.bc_sources(core.rowptr, core.colidx, src, 1.5, nthreads=16)
    for bu in (16.0, 0.0):
        nk.nk_set_tuning(flags=flags, bu_ratio=bu)
        got = nk.nk_bc_sources(rp, ci, ivec(src), 1.5).cpu().numpy()
        assert nk.nk_last_stats()["bitmap_lds"] == 1
        assert_scores_close(got, want, "scores")
