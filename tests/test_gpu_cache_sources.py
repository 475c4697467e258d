"""Registered autotuner entries and the number of sources: few sources go to the
group kernel whatever the entry of their graph's shape says, more run under
the entry, and the caller's own tuning comes first."""
import json

import numpy as np
import pytest

import graphgen as gg
import oracle
import paper_1403_3005_amd as nk
from nkutil import assert_scores_close, ivec, upload

pytestmark = pytest.mark.gpu


def bucket(g):
    mean = g.m / g.n
    return "n%d_d%d_s%d" % (int(np.floor(np.log2(g.n))), int(np.round(np.log2(mean))),
                            int(np.round(np.log2(g.degrees().max() / mean))))


@pytest.fixture(autouse=True)
def _defaults():
    nk.nk_set_tuning()
    yield
    nk.nk_set_tuning_cache(None)
    nk.nk_set_tuning()


@pytest.mark.parametrize("entry,many", [
    ([512, 16, 0.1, 0, 1, 10.0, 16, 0], (1, 512)),      # the one-source kernel
    ([1024, 16, 0.1, 0, 1, 10.0, 8, 2], (6, 1024)),     # the group kernel, two workgroups a source
    ([256, 16, 0.1, 0, 8, 10.0], (4, 256)),             # eight sources a task (no kernel choice)
    ([256, 16, 0.1, 10.0], (1, 256)),
])
def test_few_and_many(tmp_path, entry, many):
    g = gg.rmat(17, 8, 1)
    rp, ci = upload(g)
    cache = tmp_path / "tune.json"
    cache.write_text(json.dumps({bucket(g): entry}))
    nk.nk_set_tuning_cache(str(cache))
    for k, few in ((16, True), (128, True), (129, False)):
        src = gg.sample_sources(g.n, k, 5)
        for call, ref in ((nk.nk_bc_sources, oracle.bc_sources), (nk.nk_bc_sources_linear, oracle.bc_sources_linear)):
            got = call(rp, ci, ivec(src), 1.0).cpu().numpy()
            st = nk.nk_last_stats()
            assert (st["bitmap_lds"], st["block"]) == ((6, 1024) if few else many), (k, st)
            if k == 16:
                assert_scores_close(got, ref(g.rowptr, g.colidx, src, 1.0, nthreads=16), "few")
    # the caller's own choice is not few sources' to make
    nk.nk_set_tuning(flags=16)
    nk.nk_bc_sources(rp, ci, ivec(src[:16]), 1.0)
    assert (nk.nk_last_stats()["bitmap_lds"], nk.nk_last_stats()["block"]) == many


def test_other_calls_keep_the_entry(tmp_path):
    g = gg.rmat(17, 8, 1)
    rp, ci = upload(g)
    cache = tmp_path / "tune.json"
    cache.write_text(json.dumps({bucket(g): [256, 16, 0.1, 0, 1, 10.0, 16, 0]}))
    nk.nk_set_tuning_cache(str(cache))
    s = ivec(gg.sample_sources(g.n, 8, 5))
    for call in (lambda: nk.nk_edge_bc(rp, ci, s, 1.0), lambda: nk.nk_bc_directed(rp, ci, s, 1.0, rp, ci),
                 lambda: nk.nk_bc_sources_bisect(rp, ci, s, 1.0)):
        call()
        assert nk.nk_last_stats()["block"] == 256
