"""Block steps make no neighbour lists: with lists switched on, neighbour
radii, particle indices that are no slot numbers and listed calculations on
the same handle before and between the steps, the states are those with lists
off, bit for bit.  (A step that finished the lists an earlier calculation left
behind would look its particle indices up as slots.)"""

import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu

N, EPS2, H2 = 1500, 2.0 ** -12, 0.05
INDEX = np.where(np.arange(N) % 7, 10 ** 8 + 3 * np.arange(N), -5 - np.arange(N)).astype(np.int32)


def listed_calls(g6, hid, state):
    """A batch of two clusters, then a device calculation, on the handle's
    j-memory, with neighbours to list; the lists read back."""
    import torch
    rows = np.arange(0, N, 5, dtype=np.int32)
    dev = [torch.from_numpy(np.ascontiguousarray(q)).cuda()
           for q in (rows, state["x"][rows], state["v"][rows], np.full(len(rows), H2))]
    out = [torch.zeros(len(rows), 3, dtype=torch.float64, device="cuda") for _ in range(2)]
    pot = torch.zeros(len(rows), dtype=torch.float64, device="cuda")
    torch.cuda.synchronize()
    g6.g6_set_ti(hid, float(state["t"].max()))
    for batch in (True, False):
        if batch:
            cl = g6.clusters([0, 0], [N, N], [0, 100], [100, len(rows) - 100], [float(state["t"].max())] * 2, [EPS2] * 2)
            g6.check(hid, g6.g6mi_batch_calc(hid, cl, len(rows), *dev, *out, pot))
        else:
            g6.check(hid, g6.g6mi_calc_device(hid, N, len(rows), dev[0], dev[1], dev[2], EPS2, dev[3], *out, pot))
        g6.check(hid, g6.g6_read_neighbour_list(hid))
        ln, buf, listed = np.zeros(1, dtype=np.int32), np.zeros(g6.NB_MAX, dtype=np.int32), 0
        for i in range(len(rows)):
            g6.check(hid, g6.g6_get_neighbour_list(hid, i, g6.NB_MAX, ln, buf))
            assert np.isin(buf[:min(ln[0], g6.NB_MAX)], INDEX).all()
            listed += ln[0]
        assert listed > len(rows)


def steps(g6, prec, lists_init, lists_steps, h2, calls):
    """Three advances of 1, 4 and 18 block steps; the states after each."""
    hid = 5
    x, v = workloads.plummer(N, 77)
    m, z = np.full(N, 1.0 / N), np.zeros((N, 3))
    states = []
    g6.check(hid, g6.g6_open(hid))
    try:
        g6.check(hid, g6.g6mi_set_precision(hid, prec))
        g6.check(hid, g6.g6mi_set_j_particles(hid, N, np.arange(N), INDEX, np.zeros(N), None, m, z, z, v, x))
        g6.check(hid, g6.g6mi_set_neighbour_lists(hid, lists_init))
        g6.check(hid, g6.g6mi_hermite_init(hid, N, EPS2, h2, 0.01, 0.01, 2.0 ** -7, 2.0 ** -40), allow_warn=False)
        g6.check(hid, g6.g6mi_set_neighbour_lists(hid, lists_steps))
        for count in (1, 4, 18):
            if calls:
                listed_calls(g6, hid, states[-1] if states else g6.g6mi_hermite_state(hid, N))
            rc, _, _, _ = g6.g6mi_hermite_advance(hid, 1e30, count)
            g6.check(hid, rc, allow_warn=False)
            assert g6.g6_read_neighbour_list(hid) == g6.ESTATE  # no lists of a block step
            states.append(g6.g6mi_hermite_state(hid, N))
    finally:
        g6.g6_close(hid)
    return states


@pytest.mark.parametrize("prec", ["ds", "fp32", "fp64"])
@pytest.mark.parametrize("lists_init,lists_steps,h2,calls", [(True, True, H2, False), (True, True, 0.0, True),
                                                             (False, True, H2, True)])
def test_block_steps_ignore_neighbour_lists(prec, lists_init, lists_steps, h2, calls):
    import paper_0902_4463_amd as g6
    ref = steps(g6, prec, False, False, 0.0, False)
    got = steps(g6, prec, lists_init, lists_steps, h2, calls)
    for a, b in zip(ref, got):
        for k in a:
            assert np.array_equal(a[k], b[k]), k
