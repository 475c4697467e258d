"""The kernel that keeps a source's levels and path counts in LDS (graphs of
up to 65,534 vertices whose CSR does not fit LDS): every lanes-per-row form,
rows scanned by a whole wave, more levels than the kept offsets, path counts
split between LDS and global memory, direction mixes, both estimators, the
unchecked and the overflow-checked counting, and batches that mix its forms
-- scores against the CPU oracle."""
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


def _with_spare(g, n):
    """g plus isolated vertices up to n in all."""
    rp = np.concatenate([g.rowptr, np.full(n - g.n, g.rowptr[-1], dtype=np.int32)])
    return gg.Graph(n, rp, g.colidx, f"{g.name}+{n - g.n}")


GRAPHS = [
    lambda: gg.erdos_renyi(11000, 22000, 1),            # 4 lanes a row
    lambda: gg.erdos_renyi(9001, 90000, 2),             # 8
    lambda: gg.rmat(13, 40, 3),                         # 16, hubs
    lambda: gg.complete(400),                           # every row a wave's
    lambda: gg.star(20000), lambda: gg.path(12001),     # one hub; levels far past the kept offsets
    lambda: gg.barabasi_albert(13500, 4, 4), lambda: gg.barabasi_albert(13700, 4, 5),   # either side of the LDS limit
    lambda: gg.random_tree(30011, 6), lambda: gg.rmat(15, 8, 7), lambda: gg.barabasi_albert(65534, 3, 8),
    lambda: gg.disjoint_union([gg.grid(6, 1500), gg.star(5000), gg.path(1), gg.cycle(999)]),
]


@pytest.mark.parametrize("make", GRAPHS)
@pytest.mark.parametrize("bu_ratio", [0.0, 16.0, 1e9])
def test_scores(make, bu_ratio):
    g = make()
    nk.nk_set_tuning(bu_ratio=bu_ratio)
    src = gg.sample_sources(g.n, 12, 9)
    rp, ci = upload(g)
    got = nk.nk_bc_sources(rp, ci, ivec(src), 1.5).cpu().numpy()
    st = nk.nk_last_stats()
    assert st["bitmap_lds"] == 1 and st["sources"] == 12, st
    assert st["levels_bw_push"] == 0                    # (the other kernel of this placement pushes levels)
    reached, arcs, dag, depth = oracle.work_counts(g.rowptr, g.colidx, src)
    assert (st["reached"], st["arcs_reached"], st["dag_arcs"]) == (reached, arcs, dag)
    assert st["levels_td"] + st["levels_bu"] == depth + 12
    assert_scores_close(got, oracle.bc_sources(g.rowptr, g.colidx, src, 1.5, nthreads=8), g.name)
    if bu_ratio == 16.0:
        got = nk.nk_bc_sources_linear(rp, ci, ivec(src), 2.0).cpu().numpy()
        assert_scores_close(got, oracle.bc_sources_linear(g.rowptr, g.colidx, src, 2.0, nthreads=8), g.name)


@pytest.mark.parametrize("n", [12000, 40000])
def test_counts_to_the_last_bit(n):
    rp, ci = upload(_with_spare(gg.diamond_chain(63), n))       # 2^63 paths end to end
    g = gg.diamond_chain(63)
    got = nk.nk_bc_sources(rp, ci, ivec([0, 3 * 63]), 1.0).cpu().numpy()
    assert_scores_close(got[:g.n], oracle.bc_sources(g.rowptr, g.colidx, [0, 3 * 63]), "2^63")
    assert not got[g.n:].any()
    rp, ci = upload(_with_spare(gg.diamond_chain(64), n))
    with pytest.raises(nk.NkError) as e:
        nk.nk_bc_sources(rp, ci, ivec([0]), 1.0)
    assert e.value.code == nk.NK_E_SIGMA_OVERFLOW
    with pytest.raises(nk.NkError) as e:
        nk.nk_bc_sources(rp, ci, ivec([0, n]), 1.0)
    assert e.value.code in (nk.NK_E_INVALID_ARG, nk.NK_E_SIGMA_OVERFLOW)


def test_batch_of_every_form():
    graphs = [gg.erdos_renyi(500, 2000, 11), gg.barabasi_albert(7000, 3, 12), gg.path(4), gg.erdos_renyi(15001, 30000, 13),
              gg.barabasi_albert(14500, 2, 14), gg.star(6000), gg.rmat(9, 60, 15)]
    vtx = np.cumsum([0] + [g.n for g in graphs])
    arc = np.cumsum([0] + [g.m for g in graphs])
    rp = torch.from_numpy(np.concatenate([g.rowptr for g in graphs]).astype(np.int32)).cuda()
    ci = torch.from_numpy(np.concatenate([g.colidx for g in graphs]).astype(np.int32)).cuda()
    refs = [oracle.bc_exact(g.rowptr, g.colidx, nthreads=16) for g in graphs]
    with nk.NkBatchPlan(vtx, arc, rp, ci) as plan:
        for got in (nk.nk_bc_exact_batched(vtx, arc, rp, ci), plan.run(), plan.run()):
            got = got.cpu().numpy()
            assert nk.nk_last_stats()["sources"] == int(vtx[-1])
            for i, g in enumerate(graphs):
                assert_scores_close(got[vtx[i]:vtx[i + 1]], refs[i], f"graph {i}")
