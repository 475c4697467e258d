"""Pair sampling on both forms of its kernel (four workgroups a compute unit, or
two with more registers) at both sides of the line between them, with records
and with hash tables, and under a scratch cap that leaves few slots: counts
equal the oracle's."""
import numpy as np
import pytest

import graphgen as gg
import oracle
import paper_1403_3005_amd as nk
from nkutil import upload

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _default_tuning():
    nk.nk_set_tuning()
    yield
    nk.nk_set_tuning()


@pytest.mark.parametrize("make", [lambda: gg.chung_lu(70000, 2.4, 9.0, 3), lambda: gg.grid(30, 41),
                                  lambda: gg.disjoint_union([gg.rmat(10, 8, 2), gg.star(400), gg.path(30)])])
@pytest.mark.parametrize("flags", [32, 64])
def test_counts(make, flags):
    g = make()
    rp, ci = upload(g)
    for r, tuning in ((1, {}), (512, {}), (513, {}), (2500, {}), (2500, dict(wg_per_cu=1)), (2500, dict(wg_per_cu=3)),
                      (2500, dict(scratch_mib=64))):
        nk.nk_set_tuning(flags=flags, **tuning)
        got = nk.nk_pair_counts(rp, ci, r, 11).cpu().numpy()
        assert np.array_equal(got, oracle.pair_counts(g.rowptr, g.colidx, r, 11)), (r, tuning)
