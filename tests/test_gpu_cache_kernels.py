"""Autotuner entries belong to the kernel they were timed on: an entry made with
the source's state in LDS applies to plain calls there and not to edge,
directed and bisection calls, an older one the other way round; and the
autotuner leaves alone the ratio that its kernel does not look at."""
import json

import pytest

import graphgen as gg
import oracle
import paper_1403_3005_amd as nk
from nkutil import assert_scores_close, ivec, upload

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _defaults():
    nk.nk_set_tuning()
    yield
    nk.nk_set_tuning_cache(None)
    nk.nk_set_tuning()


def _others(rp, ci, s):
    return (lambda: nk.nk_edge_bc(rp, ci, s, 1.0), lambda: nk.nk_bc_directed(rp, ci, s, 1.0, rp, ci),
            lambda: nk.nk_bc_sources_bisect(rp, ci, s, 1.0))


@pytest.mark.parametrize("bw_ratio", [0.1, 0.7])
def test_entry_made_in_lds(tmp_path, bw_ratio):
    g = gg.barabasi_albert(20000, 4, 123)
    rp, ci = upload(g)
    src = gg.sample_sources(g.n, 32, 124)
    s = ivec(src)
    cache = tmp_path / "tune.json"
    nk.nk_set_tuning(bw_ratio=bw_ratio)
    best = nk.nk_autotune(rp, ci, s, str(cache))
    nk.nk_set_tuning()
    assert best["bw_ratio"] == pytest.approx(bw_ratio)
    entries = json.loads(cache.read_text())
    (key, entry), = entries.items()
    assert entry[6] in (256 + 8, 256 + 16) and entry[2] == pytest.approx(bw_ratio)
    # a distinctive one
    cache.write_text(json.dumps({key: [256, 0.0, bw_ratio, 0, 1, 1.0, 256 + 16, 0]}))
    nk.nk_set_tuning_cache(str(cache))
    got = nk.nk_bc_sources(rp, ci, s, 1.0).cpu().numpy()
    st = nk.nk_last_stats()
    assert (st["bitmap_lds"], st["block"], st["levels_bu"]) == (1, 256, 0)
    assert_scores_close(got, oracle.bc_sources(g.rowptr, g.colidx, src, 1.0, nthreads=16), "entry")
    for call in _others(rp, ci, s):
        call()
        st = nk.nk_last_stats()
        assert st["block"] == 1024 and st["levels_bu"] > 0        # the automatic choice
    # the same without the mark: timed on the other kernels
    cache.write_text(json.dumps({key: [256, 0.0, bw_ratio, 0, 1, 1.0, 16, 0]}))
    nk.nk_set_tuning_cache(str(cache))
    nk.nk_bc_sources(rp, ci, s, 1.0)
    st = nk.nk_last_stats()
    assert (st["bitmap_lds"], st["block"]) == (1, 1024) and st["levels_bu"] > 0
    for call in _others(rp, ci, s):
        call()
        st = nk.nk_last_stats()
        assert (st["block"], st["levels_bu"]) == (256, 0)


def test_graph_in_lds(tmp_path):
    g = gg.erdos_renyi(1200, 5000, 3)
    rp, ci = upload(g)
    cache = tmp_path / "tune.json"
    best = nk.nk_autotune(rp, ci, ivec(gg.sample_sources(g.n, 64, 4)), str(cache))
    assert (best["bu_ratio"], best["bw_ratio"]) == (16.0, pytest.approx(0.1))
    (key, _), = json.loads(cache.read_text()).items()
    for mark in (0, 256):
        cache.write_text(json.dumps({key: [256, 16, 0.1, 0, 1, 1.0, 16 + mark, 0]}))
        nk.nk_set_tuning_cache(str(cache))
        nk.nk_bc_exact(rp, ci)
        st = nk.nk_last_stats()
        assert (st["bitmap_lds"], st["block"]) == (2, 256)


def test_batch_under_a_larger_graph_s_entry(tmp_path):
    """The entry of the largest graph (too large for LDS) leaves the launch of
    the others alone."""
    import numpy as np
    import torch

    small, big = gg.barabasi_albert(16000, 4, 5), gg.erdos_renyi(66000, 132000, 6)
    vtx = np.array([0, small.n, small.n + big.n], dtype=np.int64)
    arc = np.array([0, small.m, small.m + big.m], dtype=np.int64)
    rp = torch.from_numpy(np.concatenate([small.rowptr, big.rowptr]).astype(np.int32)).cuda()
    ci = torch.from_numpy(np.concatenate([small.colidx, big.colidx]).astype(np.int32)).cuda()
    deg = big.degrees()
    mean = big.m / big.n
    key = "n%d_d%d_s%d" % (int(np.floor(np.log2(big.n))), int(np.round(np.log2(mean))),
                           int(np.round(np.log2(deg.max() / mean))))
    cache = tmp_path / "tune.json"
    cache.write_text(json.dumps({key: [256, 0.0, 0.1, 0, 1, 1.0, 16, 0]}))
    nk.nk_set_tuning_cache(str(cache))
    with nk.NkBatchPlan(vtx, arc, rp, ci) as plan:
        out = plan.run().cpu().numpy()
        st = nk.nk_last_stats()
    assert st["block"] == 256 and st["levels_bu"] > 0             # the small graph's levels
    assert_scores_close(out[:small.n], oracle.bc_exact(small.rowptr, small.colidx, nthreads=16), "small")
