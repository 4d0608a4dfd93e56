"""Forces of one block step against a batch of one cluster on the same
predicted states: narrow blocks, and blocks wide enough (some 5700 active
particles of 16384) for two i-particles per lane, with and without a ragged
last tile.

Both add the same float32 sums; the float64 additions of at most 64 split
partials above them may go in another order: 64 * 2^-53 of their absolute sum,
which is at most some 10^3 times the result."""

import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu

RTOL = 1e-11
EPS2 = 2.0 ** -12


@pytest.mark.parametrize("prec", ["ds", "fp32", "fp64"])
@pytest.mark.parametrize("n", [300, 1500, 16384, 16385])
def test_block_forces_match_one_cluster_batch(n, prec):
    import torch

    import paper_0902_4463_amd as g6
    x, v = workloads.plummer(n, 60 + n)
    m, z, idx = np.full(n, 1.0 / n), np.zeros((n, 3)), np.arange(n)
    with g6.Session(5, precision=prec, neighbour_lists=False):
        g6.check(5, g6.g6mi_set_j_particles(5, n, idx, idx, np.zeros(n), None, m, z, z, v, x))
        g6.check(5, g6.g6mi_hermite_init(5, n, EPS2, 0.0, 0.01, 0.01, 2.0 ** -13, 2.0 ** -13), allow_warn=False)
        g6.check(5, g6.g6mi_hermite_advance(5, 1e30, 1)[0], allow_warn=False)
        before = g6.g6mi_hermite_state(5, n)
        rc, tb, _, _ = g6.g6mi_hermite_advance(5, 1e30, 1)
        g6.check(5, rc, allow_warn=False)
        after = g6.g6mi_hermite_state(5, n)
    rows = np.flatnonzero(after["t"] == tb).astype(np.int32)
    assert len(rows) == n  # dt_min = dt_max: every particle in every block
    # the block's particles predicted as the library predicts them
    tau = (tb - before["t"])[:, None]
    a2, j6 = 0.5 * before["acc"], before["jerk"] / 6.0
    xp = before["x"] + tau * (before["v"] + tau * (a2 + tau * j6))
    vp = before["v"] + tau * (2.0 * a2 + tau * (3.0 * j6))
    dev = [torch.from_numpy(np.ascontiguousarray(q)).cuda() for q in (rows, xp[rows], vp[rows], np.zeros(len(rows)))]
    out = [torch.zeros(len(rows), k, dtype=torch.float64, device="cuda") for k in (3, 3, 1)]
    torch.cuda.synchronize()
    with g6.Session(5, precision=prec, neighbour_lists=False):
        g6.check(5, g6.g6mi_set_j_particles(5, n, idx, idx, before["t"], None, m, before["jerk"] / 6.0,
                                            before["acc"] / 2.0, before["v"], before["x"]))
        cl = g6.clusters([0], [n], [0], [len(rows)], [tb], [EPS2])
        g6.check(5, g6.g6mi_batch_calc(5, cl, len(rows), *dev, *out))
        assert g6.g6mi_last_status(5) == 0
        torch.cuda.synchronize()
    for k, q in zip(("acc", "jerk", "pot"), out):
        got, want = after[k][rows].reshape(len(rows), -1), q.cpu().numpy()
        d = np.linalg.norm(got - want, axis=1)
        print(f"n={n} {prec} {k}: active {len(rows)} rel {np.max(d / np.linalg.norm(want, axis=1)):.2e}", flush=True)
        assert np.all(d <= RTOL * np.linalg.norm(want, axis=1)), k
