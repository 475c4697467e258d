"""Path counts past 2^64 where every step of a path has parallel arcs (levels
stay one vertex wide): reported by the kernel with the graph in LDS and by
the one with the source's state there, top-down and bottom-up; one step
below the limit the scores are those of the path without them."""
import numpy as np
import pytest
import torch

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


def _chain(steps, arcs, tail):
    """A path of `steps` steps with `arcs` parallel arcs each, then `tail`'s graph."""
    rows = [[x for x in (i - 1, i + 1) if 0 <= x <= steps for _ in range(arcs)] for i in range(steps + 1)]
    base = len(rows)
    deg = np.concatenate([[len(r) for r in rows], tail.degrees()])
    ci = np.concatenate([np.concatenate(rows), tail.colidx.astype(np.int64) + base])
    return np.concatenate([[0], np.cumsum(deg)]).astype(np.int32), ci.astype(np.int32)


@pytest.mark.parametrize("arcs,most", [(16, 15), (2, 63), (65536, 3)])
@pytest.mark.parametrize("tail,where", [(lambda: gg.path(1), 2), (lambda: gg.from_edges(30000, [], []), 1),
                                        (lambda: gg.erdos_renyi(40000, 200000, 3), 1)])
@pytest.mark.parametrize("bu_ratio", [0.0, 16.0, 1e9])
def test_parallel_arcs(arcs, most, tail, where, bu_ratio):
    tail = tail()
    if arcs == 65536:
        where = 1                                   # too many arcs for the LDS
    nk.nk_set_tuning(bu_ratio=bu_ratio)
    for steps in (most, most + 1):
        rp, ci = (torch.from_numpy(a).to("cuda:0") for a in _chain(steps, arcs, tail))
        src = ivec([0, steps, steps // 2])
        if steps > most:
            with pytest.raises(nk.NkError) as e:
                nk.nk_bc_sources(rp, ci, src, 1.0)
            assert e.value.code == nk.NK_E_SIGMA_OVERFLOW
        else:
            got = nk.nk_bc_sources(rp, ci, src, 1.0).cpu().numpy()
            assert nk.nk_last_stats()["bitmap_lds"] == where
            simple = gg.path(steps + 1)
            ref = oracle.bc_sources(simple.rowptr, simple.colidx, np.array([0, steps, steps // 2]), 1.0)
            assert_scores_close(got[:steps + 1], ref, "chain")
            assert not got[steps + 1:].any()
