"""First device-path calls on a caller's stream after particles were set on
the host: the j-memory is allocated and cleared, or regrown, on the handle's
stream and filled on the caller's, in that order."""

import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batch", [False, True])
def test_first_call_on_another_stream(batch):
    import torch

    import paper_0902_4463_amd as g6
    n, ni, hid = 150000, 40, 4
    jm = workloads.random_cluster(n, seed=5100)
    rows = np.linspace(0, 4999, ni).astype(np.int32)
    dev = [torch.from_numpy(np.ascontiguousarray(q)).cuda()
           for q in (rows, jm.x[rows], jm.v[rows], np.full(ni, 1e-4))]
    out = [torch.zeros(ni, k, dtype=torch.float64, device="cuda") for k in (3, 3, 1)]
    stream = torch.cuda.Stream()
    ti = float(jm.t.max())

    def store(lo, hi):
        g6.check(hid, g6.g6mi_set_j_particles(hid, hi - lo, np.arange(lo, hi), jm.index[lo:hi], jm.t[lo:hi], None,
                                              jm.m[lo:hi], jm.j6[lo:hi], jm.a2[lo:hi], jm.v[lo:hi], jm.x[lo:hi]))

    def call(nj):
        for q in out:
            q.fill_(float("nan"))
        torch.cuda.synchronize()
        g6.g6_set_ti(hid, ti)
        if batch:
            cl = g6.clusters([0], [nj], [0], [ni], [ti], [1e-4])
            g6.check(hid, g6.g6mi_batch_calc(hid, cl, ni, *dev, *out, stream=stream))
        else:
            g6.check(hid, g6.g6mi_calc_device(hid, nj, ni, dev[0], dev[1], dev[2], 1e-4, dev[3], *out, stream=stream))
        stream.synchronize()
        return [q.cpu().numpy() for q in out]

    for _ in range(4):
        g6.check(hid, g6.g6_open(hid))
        try:
            store(0, 5000)
            first = call(5000)   # allocates and clears
            again = call(5000)   # settled
            store(5000, n)
            grown = call(n)      # regrows and clears
            settled = call(n)
        finally:
            g6.g6_close(hid)
        for a, b in zip(first + grown, again + settled):
            assert np.isfinite(a).all() and np.array_equal(a, b)
