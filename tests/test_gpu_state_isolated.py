"""State-in-LDS kernel on graphs with isolated vertices, which it leaves out of
its passes: at the end, between the others and nearly all of them, counts
around the workgroup's pieces, isolated sources, all forms (state in LDS, part
of it global, own ids) -- scores and counters against the oracle."""
import numpy as np
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


def _graph(n, live, kind):
    """n vertices, arcs among `live` of them: the first, the last or spread."""
    r = np.random.default_rng(n + live)
    core = gg.erdos_renyi(live, 2 * live, 3) if kind == "sparse" else gg.path(live)
    ids = {0: np.arange(live), 1: np.arange(n - live, n), 2: np.sort(r.permutation(n)[:live])}[(n + live) % 3]
    t = np.repeat(np.arange(live), core.degrees())
    return gg.from_edges(n, ids[t], ids[core.colidx]), ids


@pytest.mark.parametrize("n,live,kind", [
    (9000, 8999, "sparse"), (9000, 5000, "sparse"), (9000, 2, "path"), (9000, 300, "path"), (40000, 20000, "sparse"),
    (40000, 39990, "sparse"), (40000, 10239, "sparse"), (40000, 10240, "sparse"), (40000, 10241, "sparse"),
    (65534, 1023, "path"), (65534, 1024, "path"), (65534, 1025, "path"), (65534, 33000, "sparse"), (65534, 65533, "sparse"),
])
@pytest.mark.parametrize("flags", [0, 2])
def test_isolated(n, live, kind, flags):
    g, ids = _graph(n, live, kind)
    rp, ci = upload(g)
    r = np.random.default_rng(1)
    rest = np.setdiff1d(np.arange(n), ids)
    src = np.concatenate([ids[[0, -1]], r.choice(ids, min(live, 30)), r.choice(rest, min(len(rest), 20)), [0, n - 1]])
    for block in (0, 256):
        nk.nk_set_tuning(flags=flags, block=block)
        got = nk.nk_bc_sources(rp, ci, ivec(src), 1.5).cpu().numpy()
        st = nk.nk_last_stats()
        reached, arcs, dag, depth = oracle.work_counts(g.rowptr, g.colidx, src)
        assert st["bitmap_lds"] == 1 or (n == 9000 and st["bitmap_lds"] == 2)
        assert (st["sources"], st["reached"], st["arcs_reached"], st["dag_arcs"]) == (len(src), reached, arcs, dag)
        if st["bitmap_lds"] == 1:
            assert st["levels_td"] + st["levels_bu"] == depth + len(src)
        assert_scores_close(got, oracle.bc_sources(g.rowptr, g.colidx, src, 1.5, nthreads=16), "scores")
    lin = nk.nk_bc_sources_linear(rp, ci, ivec(src), 1.5).cpu().numpy()
    assert_scores_close(lin, oracle.bc_sources_linear(g.rowptr, g.colidx, src, 1.5, nthreads=16), "linear")


def test_no_arcs_and_bad_sources():
    g = gg.from_edges(30000, [], [])
    rp, ci = upload(g)
    assert not nk.nk_bc_sources(rp, ci, ivec([0, 5, 29999]), 1.0).cpu().numpy().any()
    g, ids = _graph(40000, 300, "path")
    rp, ci = upload(g)
    for bad in (-1, 40000):
        with pytest.raises(nk.NkError) as e:
            nk.nk_bc_sources(rp, ci, ivec([0, bad]), 1.0)
        assert e.value.code == nk.NK_E_INVALID_ARG
