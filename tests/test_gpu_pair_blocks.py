"""Pair sampling's record blocks carry nothing of the graph that used them
last: a block left by one call serves a later call on another graph of any
vertex count it is large enough for.  Graphs of different strides and arc
counts take turns on one pool; every call's counts must equal the CPU
oracle's."""
import numpy as np
import pytest

import graphgen as gg
import oracle
import paper_1403_3005_amd as nk
from nkutil import upload

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _default_tuning():
    nk.nk_shutdown()            # the first call takes a fresh block
    nk.nk_set_tuning(flags=32)  # one record per vertex
    yield
    nk.nk_set_tuning()


@pytest.mark.parametrize("sizes", [(6000, 4100, 6000, 5999), (64, 700, 65, 3)])
def test_one_block_for_graphs_of_many_sizes(sizes):
    for i, n in enumerate(sizes):
        g = gg.chung_lu(n, 2.4, 7.0, 50 + i) if i % 2 else gg.erdos_renyi(n, min(3 * n, n * (n - 1) // 2), 60 + i)
        rp, ci = upload(g)
        for seed in (1, 2):
            got = nk.nk_pair_counts(rp, ci, 500, seed).cpu().numpy()
            assert np.array_equal(got, oracle.pair_counts(g.rowptr, g.colidx, 500, seed, nthreads=8)), (n, seed)
