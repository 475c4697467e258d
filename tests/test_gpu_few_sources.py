"""Runs with fewer sources than compute units, several workgroups a source:
both sides of each line of the automatic choice (sources, vertices, arcs a
vertex, a set block size, a scratch limit), pushed and pulled backward
levels, every group size -- scores against the CPU oracle and the work
counters against its own; and a call that finds the device held by another
launch."""
import threading

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


def _run(g, k, where, ref=True, **tuning):
    nk.nk_set_tuning(**tuning)
    rp, ci = upload(g)
    src = gg.sample_sources(g.n, k, 5)
    got = nk.nk_bc_sources(rp, ci, ivec(src), 1.25).cpu().numpy()
    st = nk.nk_last_stats()
    assert st["bitmap_lds"] == where and st["sources"] == k, st
    if ref:
        assert_scores_close(got, oracle.bc_sources(g.rowptr, g.colidx, src, 1.25, nthreads=16), g.name)
    return got, st, src


@pytest.mark.parametrize("make,k,where", [
    (lambda: gg.rmat(17, 8, 1), 1, 6), (lambda: gg.rmat(17, 8, 1), 8, 6), (lambda: gg.rmat(17, 8, 1), 9, 6),
    (lambda: gg.rmat(17, 8, 1), 128, 6), (lambda: gg.rmat(17, 8, 1), 129, 1),
    (lambda: gg.erdos_renyi(65534, 200000, 2), 4, 1), (lambda: gg.erdos_renyi(65535, 200000, 2), 4, 6),
    (lambda: gg.erdos_renyi(70000, 210000, 3), 20, 6), (lambda: gg.erdos_renyi(70000, 209999, 3), 20, 1),
])
def test_choice(make, k, where):
    g = make()
    _, st, src = _run(g, k, where)
    reached, arcs, dag, depth = oracle.work_counts(g.rowptr, g.colidx, src)
    assert (st["reached"], st["arcs_reached"], st["dag_arcs"]) == (reached, arcs, dag)
    assert st["levels_td"] + st["levels_bu"] == depth + k


def test_choice_left_to_the_caller():
    g = gg.rmat(17, 8, 1)
    for tuning in (dict(block=1024), dict(block=256), dict(wg_per_cu=1), dict(flags=1), dict(flags=16), dict(scratch_mib=16)):
        _run(g, 4, 0 if tuning.get("flags") == 1 else 1, ref=False, **tuning)


@pytest.mark.parametrize("bw_ratio", [0.0, 0.5, 1e9])
@pytest.mark.parametrize("group", [0, 1, 2, 8, 32])
def test_push_and_pull(group, bw_ratio):
    for g in (gg.rmat(13, 12, 6), gg.disjoint_union([gg.grid(9, 11), gg.star(3000), gg.path(1), gg.cycle(901)])):
        _, st, src = _run(g, 24, 6, flags=12, group=group, bw_ratio=bw_ratio)
        assert (st["levels_bw_push"] > 0) == (bw_ratio > 0)
        rp, ci = upload(g)
        got = nk.nk_bc_sources_linear(rp, ci, ivec(src), 2.0).cpu().numpy()
        assert_scores_close(got, oracle.bc_sources_linear(g.rowptr, g.colidx, src, 2.0, nthreads=8), "linear")


def test_beside_another_launch():
    """Sixteen long searches hold their compute units from another thread and
    stream; the call ends right whichever kernel it ends on."""
    long_rp, long_ci = upload(gg.path(4000))
    g = gg.rmat(17, 8, 1)
    rp, ci = upload(g)
    src = gg.sample_sources(g.n, 8, 5)
    ref = oracle.bc_sources(g.rowptr, g.colidx, src, 1.0, nthreads=16)
    started = threading.Event()
    out = []

    def hold():
        with torch.cuda.stream(torch.cuda.Stream()):
            started.set()
            out.append(nk.nk_bc_sources_bisect(long_rp, long_ci, ivec(np.arange(16)), 1.0).cpu().numpy())

    th = threading.Thread(target=hold)
    th.start()
    started.wait()
    with torch.cuda.stream(torch.cuda.Stream()):
        for _ in range(3):
            got = nk.nk_bc_sources(rp, ci, ivec(src), 1.0).cpu().numpy()
            assert nk.nk_last_stats()["bitmap_lds"] in (1, 6)
            assert_scores_close(got, ref, "beside another launch")
    th.join()
    assert len(out) == 1 and np.isfinite(out[0]).all()
