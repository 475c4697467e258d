"""Sampled closeness at both sides of the most vertices a bit-parallel level's
launch can hold (2^29), and where the launch would pass 2^32 threads: a star
among the last million vertices, every other vertex isolated, the source the
star's centre -- the last id."""
import pytest
import torch

import paper_1403_3005_amd as nk

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,bits", [(2**29, True), (2**29 + 1, False), (2**30 + 12345, False)])
def test_star_of_the_last_vertices(n, bits):
    if torch.cuda.mem_get_info()[0] < 200 << 30:
        pytest.skip("needs 200 GiB of free device memory")
    leaves = 1_000_000
    first = n - 1 - leaves
    try:
        rp = torch.zeros(n + 1, dtype=torch.int32, device="cuda")
        rp[first:n] = torch.arange(0, leaves + 1, dtype=torch.int32, device="cuda")
        rp[n] = 2 * leaves
        ci = torch.full((2 * leaves,), n - 1, dtype=torch.int32, device="cuda")
        ci[leaves:] = torch.arange(first, n - 1, dtype=torch.int32, device="cuda")
        out = nk.nk_closeness_sampled(rp, ci, torch.tensor([n - 1], dtype=torch.int32, device="cuda"))
        st = nk.nk_last_stats()
        assert int(torch.count_nonzero(out)) == leaves
        # farness n / 1 * 1 of every leaf
        assert torch.allclose(out[first:n - 1], torch.full((leaves,), (n - 1) / n, dtype=torch.float64, device="cuda"),
                              rtol=1e-14, atol=0.0)
        # (one source is one workgroup of the other kernel, a block of 64 vertices here)
        assert (st["workgroups"] > 1) == bits, st
    finally:
        rp = ci = out = None
        torch.cuda.empty_cache()
        nk.nk_shutdown()
