"""Work tables of batches on both sides of the plan kernel's sizes: one
cluster per thread with 256 threads up to 64 clusters, with 1024 threads in
one pass up to 1024, and in several passes above."""

import pytest

import oracle
import workloads
from tests.test_gpu_batch import Batch, check_rows, i_block, oracle_rows, predicted

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ncl,n_hi", [(1, 600), (64, 600), (65, 600), (1024, 40), (1025, 600), (2100, 40)])
def test_batch_plan_sizes(ncl, n_hi):
    """Every row against the oracle at the suite's tolerances; n_hi 600 gives
    wide, narrow and cut blocks, so all three queue classes hold items."""
    import paper_0902_4463_amd as g6
    cb = workloads.config_c4(seed=5000 + ncl, nclusters=ncl, n_lo=16, n_hi=n_hi)
    xp, vp = predicted(oracle, cb)
    xi, vi, h2 = i_block(cb, xp, vp)
    ref = oracle_rows(oracle, cb, xp, vp, xi, vi, h2)
    with g6.Session(2) as s:
        s.load(cb.jm)
        g6.check(s.id, g6.g6mi_set_precision(s.id, "ds"))
        g6.check(s.id, g6.g6mi_batch_set_tuning(s.id, dict(g6.g6mi_batch_get_tuning(s.id), wide_min=257)))
        b = Batch(g6, cb, xi, vi, h2)
        try:
            g6.check(s.id, b.run(s.id))
            check_rows(g6, s.id, b.fetch(), ref, cb, xp, xi, f"{ncl} clusters")
            assert g6.g6mi_last_status(s.id) & ~g6.FLAG_NB_OVERFLOW == 0
        finally:
            g6.check(s.id, g6.g6mi_batch_set_tuning(s.id, None))
