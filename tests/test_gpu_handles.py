"""What a handle leaves behind: device memory after g6_close."""

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
