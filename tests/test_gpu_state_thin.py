"""Thin graphs of up to 2 * 10^4 vertices with many sources: they leave the
state-in-LDS kernel for the one-source kernel (four 256-thread workgroups a
compute unit), single and in batches, and only they; invalid graphs are
refused as before."""
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
    i, j = np.triu_indices(size, 1)
    base = np.arange(count)[:, None] * size
    ends = np.arange(1, count) * size
    return gg.from_edges(count * size, np.concatenate([(base + i).ravel(), ends - 1]),
                         np.concatenate([(base + j).ravel(), ends]), f"{count} cliques of {size}")


def _tail(g, length):
    t = np.repeat(np.arange(g.n), g.degrees())
    keep = t < g.colidx
    ends = np.concatenate([[0], g.n + np.arange(length - 1)])
    return gg.from_edges(g.n + length, np.concatenate([t[keep], ends]),
                         np.concatenate([g.colidx[keep], g.n + np.arange(length)]), "tail")


THIN = [lambda: gg.cycle(9000), lambda: _cliques(900, 9), lambda: gg.cycle(19999), lambda: gg.grid(4, 2300)]
WIDE = [lambda: gg.barabasi_albert(9973, 4, 2), lambda: gg.erdos_renyi(12000, 18000, 3), lambda: gg.random_tree(9000, 4),
        lambda: gg.star(12000), lambda: _cliques(300, 40), lambda: _tail(gg.barabasi_albert(9000, 4, 2), 900),
        lambda: gg.disjoint_union([gg.path(12)] * 1000), lambda: gg.cycle(20000)]


def _big(g):
    """Long runs are left to the counters; the oracle scores some sources."""
    return gg.sample_sources(g.n, 800, 6)


@pytest.mark.parametrize("make,thin", [(m, True) for m in THIN] + [(m, False) for m in WIDE])
def test_single(make, thin):
    g = make()
    rp, ci = upload(g)
    src = _big(g)
    try:
        got = nk.nk_bc_sources(rp, ci, ivec(src), 1.0).cpu().numpy()
    except nk.NkError as e:                      # (a long grid's path counts)
        assert e.code == nk.NK_E_SIGMA_OVERFLOW and g.n == 9200
        return
    st = nk.nk_last_stats()
    assert (st["bitmap_lds"], st["block"]) == (1, 256 if thin else 1024), g.name
    reached, arcs, dag, depth = oracle.work_counts(g.rowptr, g.colidx, src)
    assert (st["sources"], st["reached"], st["arcs_reached"], st["dag_arcs"]) == (800, reached, arcs, dag)
    assert_scores_close(got, oracle.bc_sources(g.rowptr, g.colidx, src, 1.0, nthreads=16), g.name)
    nk.nk_bc_sources(rp, ci, ivec(src[:700]), 1.0)
    assert nk.nk_last_stats()["block"] == 1024
    nk.nk_set_tuning(block=512)
    nk.nk_bc_sources(rp, ci, ivec(src), 1.0)
    assert nk.nk_last_stats()["block"] == 512


def test_batch():
    graphs = [gg.barabasi_albert(9973, 4, 2), gg.cycle(9000), gg.erdos_renyi(500, 900, 1), _cliques(900, 9), gg.star(12000)]
    vtx = np.cumsum([0] + [g.n for g in graphs]).astype(np.int64)
    arc = np.cumsum([0] + [g.m for g in graphs]).astype(np.int64)
    rp = torch.from_numpy(np.concatenate([g.rowptr for g in graphs]).astype(np.int32)).cuda()
    ci = torch.from_numpy(np.concatenate([g.colidx for g in graphs]).astype(np.int32)).cuda()
    ref = np.concatenate([oracle.bc_exact(g.rowptr, g.colidx, nthreads=16) for g in graphs])
    assert_scores_close(nk.nk_bc_exact_batched(vtx, arc, rp, ci).cpu().numpy(), ref, "batch")
    with nk.NkBatchPlan(vtx, arc, rp, ci) as plan:
        for _ in range(2):
            assert_scores_close(plan.run().cpu().numpy(), ref, "plan")
            st = nk.nk_last_stats()
            assert st["block"] == 256 and st["sources"] == vtx[-1]     # (the thin graphs' launch is the one shown)


@pytest.mark.parametrize("spoil", ["head", "low", "rows", "end"])
def test_invalid(spoil):
    g = gg.cycle(9000)
    rp, ci = upload(g)
    if spoil == "head":
        ci[::3] = 1 << 30
    elif spoil == "low":
        ci[::3] = -5
    elif spoil == "rows":
        rp[1:-1:2] = -7
    else:
        rp[2:-1] = 1 << 30
    with pytest.raises(nk.NkError) as e:
        nk.nk_bc_exact(rp, ci)
    assert e.value.code == nk.NK_E_INVALID_GRAPH
    vtx, arc = np.array([0, g.n], dtype=np.int64), np.array([0, g.m], dtype=np.int64)
    with pytest.raises(nk.NkError) as e:
        nk.nk_bc_exact_batched(vtx, arc, rp, ci)
    assert e.value.code == nk.NK_E_INVALID_GRAPH
