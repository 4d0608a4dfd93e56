"""What a handle leaves behind and what its switches promise, beside the
results: device memory after g6_close, neighbour lists switched off."""

import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu


def _device_inputs(torch, jm, rows, h2):
    return [torch.from_numpy(np.ascontiguousarray(q)).cuda()
            for q in (rows.astype(np.int32), jm.x[rows], jm.v[rows], np.full(len(rows), h2))]


def test_close_returns_device_memory():
    """Every kind of calculation (fused, pieces, one and two i-particles per
    lane, ordered, batched, block steps) between open and close: once the
    runtime holds its own memory, 64 further cycles take less than half of the
    library's smallest buffer (64 KiB) each."""
    import torch

    import paper_0902_4463_amd as g6
    n, hid = 20000, 4
    jm = workloads.random_cluster(n, seed=5200)
    dev = _device_inputs(torch, jm, np.arange(n), 1e-4)
    out = [torch.zeros(n, k, dtype=torch.float64, device="cuda") for k in (3, 3, 1)]

    def cycle():
        g6.check(hid, g6.g6_open(hid))
        try:
            g6.check(hid, g6.g6mi_set_j_particles(hid, n, np.arange(n), jm.index, np.zeros(n), None, jm.m, jm.j6, jm.a2,
                                                  jm.v, jm.x))
            for ni, spatial in ((4, 1), (200, 1), (1000, 1), (n, 2)):
                g6.check(hid, g6.g6mi_set_spatial(hid, spatial))
                g6.check(hid, g6.g6mi_calc_device(hid, n, ni, *dev[:3], 1e-4, dev[3], *out))
            cl = g6.clusters([0], [n], [0], [300], [0.0], [1e-4])
            g6.check(hid, g6.g6mi_batch_calc(hid, cl, 300, *dev, *out))
            g6.check(hid, g6.g6_read_neighbour_list(hid))
            g6.check(hid, g6.g6mi_hermite_init(hid, 1000, 1e-4, 0.0, 0.01, 0.01, 2.0 ** -7, 2.0 ** -40))
            g6.check(hid, g6.g6mi_hermite_advance(hid, 1e30, 2)[0])
            g6.g6mi_hermite_state(hid, 1000)
        finally:
            g6.g6_close(hid)
        torch.cuda.synchronize()
        return torch.cuda.mem_get_info()[0]

    free = [cycle() for _ in range(4)][-1]
    for _ in range(64):
        last = cycle()
    assert free - last < 64 * 2 ** 15


@pytest.mark.parametrize("ni", [300, 1500])
def test_lists_off_report_no_neighbours(ni):
    """After calculations with lists on, a calculation with lists off reports
    zero neighbours: device calls and batches, few and many rows."""
    import torch

    import paper_0902_4463_amd as g6
    n, hid = 2000, 4
    jm = workloads.random_cluster(n, seed=5300)
    rows = np.arange(ni)
    dev = _device_inputs(torch, jm, rows, 1.0)
    out = [torch.zeros(ni, k, dtype=torch.float64, device="cuda") for k in (3, 3, 1)]
    ti = float(jm.t.max())
    cl = g6.clusters([0, 0], [n, n], [0, 100], [100, ni - 100], [ti] * 2, [1e-4] * 2)

    def counts(batch):
        torch.cuda.synchronize()
        g6.g6_set_ti(hid, ti)
        if batch:
            g6.check(hid, g6.g6mi_batch_calc(hid, cl, ni, *dev, *out))
        else:
            g6.check(hid, g6.g6mi_calc_device(hid, n, ni, *dev[:3], 1e-4, dev[3], *out))
        rc = g6.check(hid, g6.g6_read_neighbour_list(hid))
        ln, buf, got = np.zeros(1, dtype=np.int32), np.zeros(g6.NB_MAX, dtype=np.int32), []
        for i in range(ni):
            g6.check(hid, g6.g6_get_neighbour_list(hid, i, g6.NB_MAX, ln, buf))
            got.append(int(ln[0]))
        return rc, np.array(got)

    with g6.Session(hid) as s:
        s.load(jm)
        for batch in (False, True):
            g6.check(hid, g6.g6mi_set_neighbour_lists(hid, True))
            assert (counts(batch)[1] > 0).any()
            g6.check(hid, g6.g6mi_set_neighbour_lists(hid, False))
            for other in (batch, not batch):
                rc, got = counts(other)
                assert rc == g6.OK and not got.any(), (batch, other)
