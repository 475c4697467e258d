"""Closeness where the bit-parallel searches look at their growth: the kernel
that ends the call at both sides of each line (lattices, chains, small
worlds, a tail behind the peak, a later pass deeper than the first), and its
scores against the oracle."""
import numpy as np
import pytest

import graphgen as gg
import oracle
import paper_1403_3005_amd as nk
from nkutil import ivec, upload

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _default_tuning():
    nk.nk_set_tuning()
    yield
    nk.nk_set_tuning()


def _lattice(*dims):
    ids = np.arange(int(np.prod(dims))).reshape(dims)
    u, v = [], []
    for a in range(len(dims)):
        u.append(np.moveaxis(ids, a, 0)[:-1].ravel())
        v.append(np.moveaxis(ids, a, 0)[1:].ravel())
    return gg.from_edges(ids.size, np.concatenate(u), np.concatenate(v), "x".join(map(str, dims)))


def _cliques(count, size):
    i, j = np.triu_indices(size, 1)
    base = np.arange(count)[:, None] * size
    ends = np.arange(1, count) * size
    return gg.from_edges(count * size, np.concatenate([(base + i).ravel(), ends - 1]),
                         np.concatenate([(base + j).ravel(), ends]), "chain of cliques")


def _small_world(n, half, seed):
    r = np.random.default_rng(seed)
    u = np.tile(np.arange(n), half)
    v = np.concatenate([(np.arange(n) + d + 1) % n for d in range(half)])
    far = r.random(u.size) < 0.02
    v[far] = r.integers(0, n, int(far.sum()))
    keep = u != v
    return gg.from_edges(n, u[keep], v[keep], "small world")


def _tail(g, length):
    """g with a path of `length` vertices hung on vertex 0."""
    t = np.repeat(np.arange(g.n), g.degrees())
    keep = t < g.colidx
    ends = np.concatenate([[0], g.n + np.arange(length - 1)])
    return gg.from_edges(g.n + length, np.concatenate([t[keep], ends]),
                         np.concatenate([g.colidx[keep], g.n + np.arange(length)]), "tail")


CASES = [   # graph, sources, whether the bit-parallel searches end the call
    (lambda: _lattice(400, 300), 40, False), (lambda: _lattice(60, 60), 700, False),
    (lambda: _lattice(24, 24, 24), 200, True), (lambda: _lattice(40, 40, 40), 64, True),
    (lambda: _cliques(1200, 8), 300, False), (lambda: _small_world(20000, 4, 1), 300, True),
    (lambda: gg.path(4000), 1024, False), (lambda: gg.random_tree(40000, 2), 400, True),
    (lambda: _tail(gg.rmat(13, 16, 3), 60), 300, True),      # levels of one vertex behind the peak
    (lambda: _tail(gg.rmat(13, 16, 3), 400), 300, False),    # too many of them
    (lambda: gg.disjoint_union([gg.rmat(11, 16, 4), gg.from_edges(60000, [], [])]), 1024, True),
]


@pytest.mark.parametrize("make,k,bits", CASES)
def test_sampled(make, k, bits):
    g = make()
    rp, ci = upload(g)
    src = gg.sample_sources(g.n, k, 8)
    got = nk.nk_closeness_sampled(rp, ci, ivec(src)).cpu().numpy()
    blocks = nk.nk_last_stats()["workgroups"] == (g.n + 63) // 64
    ref, _ = oracle.closeness_approx(g.rowptr, g.colidx, src)
    assert np.allclose(got, ref, rtol=1e-14, atol=0.0), g.name
    assert blocks == bits, g.name


@pytest.mark.parametrize("deep", [lambda: gg.path(700), lambda: _lattice(90, 40)])
def test_a_later_pass_is_deep(deep):
    """The first 1024 sources are done in a few levels; the others' pass needs
    hundreds (past the 128 levels whose masks are kept)."""
    g = gg.disjoint_union([gg.erdos_renyi(2000, 16000, 5), deep(), gg.star(300)])
    rp, ci = upload(g)
    got = nk.nk_closeness(rp, ci).cpu().numpy()
    assert nk.nk_last_stats()["workgroups"] == (g.n + 63) // 64
    assert np.allclose(got, oracle.closeness(g.rowptr, g.colidx), rtol=1e-14, atol=0.0)
