"""Arc loops over tiles whose rows begin and end at the edges of a thread's
four arcs, a wave's 256 and a block's pass: rows of 0, 1, 255 ... 4097 arcs,
long runs of empty rows (more than a wave's marks can number), in every
order a list holds them -- each kernel that walks tiles against the CPU
oracle."""
import numpy as np
import pytest
import torch

import graphgen as gg
import oracle
import paper_1403_3005_amd as nk
from nkutil import assert_scores_close, ivec, upload

pytestmark = pytest.mark.gpu

DEGREES = [0] * 300 + [1] * 257 + [2, 3, 4, 5, 63, 64, 65, 255, 0, 256, 0, 0, 257, 259] + [0] * 700 + \
          [1] * 3 + [1021, 1023, 1024, 1025, 0, 4095, 4096, 4097] + [7] * 90 + [0] * 1100 + [513, 1]


@pytest.fixture(autouse=True)
def _default_tuning():
    nk.nk_set_tuning()
    yield
    nk.nk_set_tuning()


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.int32)).to("cuda:0")


def _arcs(seed):
    """Source 0 -> one vertex a degree (their order shuffled, seed > 0) -> a
    pool of 5000 -> 40 vertices."""
    rng = np.random.default_rng(seed)
    deg = np.array(DEGREES)
    if seed:
        rng.shuffle(deg)
    a = 1 + np.arange(deg.size)
    pool = 1 + deg.size + np.arange(5000)
    last = pool[-1] + 1 + np.arange(40)
    v = np.concatenate([rng.choice(pool, d, replace=False) for d in deg])
    return (last[-1] + 1, np.concatenate([np.zeros(deg.size, np.int64), np.repeat(a, deg), pool]),
            np.concatenate([a, v, rng.choice(last, pool.size)]))


@pytest.mark.parametrize("flags", [4, 6])          # 2: under the caller's ids
@pytest.mark.parametrize("block", [256, 512, 1024])
@pytest.mark.parametrize("seed", [0, 1])
def test_rows_directed(seed, block, flags):
    n, u, v = _arcs(seed)
    g = gg.directed_from_arcs(n, u, v, "rows")
    t = gg.transpose(g)
    rp, ci = upload(g)
    src = [0, 1, 700, n - 1]
    ref = oracle.bc_directed(g.rowptr, g.colidx, src, 2.0)
    for bu in (0.0, 1e9):
        nk.nk_set_tuning(block=block, flags=flags, bu_ratio=bu)
        got = nk.nk_bc_directed(rp, ci, ivec(src), 2.0, _dev(t.rowptr), _dev(t.colidx)).cpu().numpy()
        assert_scores_close(got, ref, f"bu {bu}")
    w = gg.edge_weights(g, 9, 3, symmetric=False)
    nk.nk_set_tuning(block=block, flags=flags)
    got = nk.nk_bc_weighted(rp, ci, _dev(w), ivec(src), 2.0).cpu().numpy()
    assert_scores_close(got, oracle.bc_weighted(g.rowptr, g.colidx, w, src, 2.0), "weighted")


@pytest.mark.parametrize("flags", [4, 6, 8, 10])   # one source a workgroup; several workgroups a source
@pytest.mark.parametrize("bu_ratio", [0.0, 16.0, 1e9])
@pytest.mark.parametrize("seed", [0, 1])
def test_rows_both_ways(seed, bu_ratio, flags):
    n, u, v = _arcs(seed)
    g = gg.from_edges(n, u, v, "rows")
    rp, ci = upload(g)
    src = [0, 1, 700, n - 1]
    nk.nk_set_tuning(flags=flags, bu_ratio=bu_ratio)
    got = nk.nk_bc_sources(rp, ci, ivec(src), 2.0).cpu().numpy()
    st = nk.nk_last_stats()
    assert (st["bitmap_lds"] == 6) == bool(flags & 8), st
    assert_scores_close(got, oracle.bc_sources(g.rowptr, g.colidx, src, 2.0), "scores")
    if not flags & 8:
        ebc, _ = nk.nk_edge_bc(rp, ci, ivec(src), 2.0)
        assert_scores_close(ebc.cpu().numpy(), oracle.edge_bc(g.rowptr, g.colidx, src, 2.0)[0], "edges")
