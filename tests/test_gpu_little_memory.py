"""Calls on a device whose memory is nearly all taken by others end as they
would with less of it asked for: fewer slots, one copy of the scores."""
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
    torch.cuda.empty_cache()
    nk.nk_shutdown()


def _leave(mib):
    """Takes all device memory but `mib` MiB."""
    nk.nk_shutdown()
    torch.cuda.empty_cache()
    taken = []
    for _ in range(3):                                     # (a large allocation can leave more than was asked for)
        free = torch.cuda.mem_get_info()[0] - (mib << 20)
        if free > 2 << 20:
            taken.append(torch.empty(free, dtype=torch.uint8, device="cuda"))
    assert torch.cuda.mem_get_info()[0] <= (mib + 32) << 20
    return taken


def test_copies_of_the_scores():
    """2^25 vertices: 2 GiB of score copies beside 1.4 GiB of scratch a slot."""
    n, leaves = 1 << 25, 1000
    rp = torch.full((n + 1,), 2 * leaves, dtype=torch.int32, device="cuda")
    rp[:leaves + 1] = torch.arange(leaves + 1, dtype=torch.int32, device="cuda")
    ci = torch.cat([torch.full((leaves,), leaves, dtype=torch.int32), torch.arange(leaves, dtype=torch.int32)]).cuda()
    src = ivec([0, leaves])
    bc = torch.empty(n, dtype=torch.float64, device="cuda")
    nk.nk_bc_sources(rp, ci, src, 1.0, bc=bc)              # with memory at hand
    taken = _leave(4400)
    bc.fill_(-1.0)
    nk.nk_bc_sources(rp, ci, src, 1.0, bc=bc)
    del taken
    assert bc[leaves].item() == leaves - 1                 # the star's centre, from leaf 0
    bc[leaves] = 0.0
    assert int(torch.count_nonzero(bc)) == 0


def test_state_in_lds():
    """Up to 65,534 vertices part of a slot's state is in device memory, 200 MB
    for a slot on every compute unit; with less the grid shrinks."""
    g = gg.barabasi_albert(65000, 4, 3)
    rp, ci = upload(g)
    src = gg.sample_sources(g.n, 600, 4)
    ref = oracle.bc_sources(g.rowptr, g.colidx, src, 1.0, nthreads=16)
    assert_scores_close(nk.nk_bc_sources(rp, ci, ivec(src), 1.0).cpu().numpy(), ref, "memory at hand")
    grid = nk.nk_last_stats()["workgroups"]
    s, bc = ivec(src), torch.empty(g.n, dtype=torch.float64, device="cuda")
    taken = _leave(128)
    nk.nk_bc_sources(rp, ci, s, 1.0, bc=bc)
    st = nk.nk_last_stats()
    del taken
    assert st["bitmap_lds"] == 1 and 0 < st["workgroups"] < grid
    assert_scores_close(bc.cpu().numpy(), ref, "128 MiB left")


def test_closeness_that_gives_up():
    """A path of 200 vertices beside a star and isolated vertices, 10^6 in all,
    has too many levels for the bit-parallel searches; their 400 MB of bits do
    not count against the kernel that takes over (44 MB a slot)."""
    g = gg.disjoint_union([gg.path(200), gg.star(5200), gg.from_edges(994_600, [], [])])
    rp, ci = upload(g)
    src = np.concatenate([np.arange(200), np.arange(200, 1024) + 3000])
    ref, _ = oracle.closeness_approx(g.rowptr, g.colidx, src)
    s, out = ivec(src), torch.empty(g.n, dtype=torch.float64, device="cuda")
    nk.nk_closeness_sampled(rp, ci, s, out=out)            # with memory at hand
    taken = _leave(650)
    nk.nk_closeness_sampled(rp, ci, s, out=out)
    st = nk.nk_last_stats()
    del taken
    assert st["reached"] > 0 and 6 <= st["workgroups"] < 20, st
    assert np.allclose(out.cpu().numpy(), ref, rtol=1e-14, atol=0.0)
