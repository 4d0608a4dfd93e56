"""Block steps inside the library at sizes and step counts where their
kernels change path: ragged last tiles, blocks of 512 and more (two
i-particles per lane), step counts that mix graphs of 16, 4 and 1 steps."""

import numpy as np
import pytest

import workloads
from hermite.driver import G6Backend
from tests.hermite_oracle import OracleBackend
from tests.test_gpu_hermite_device import device_run, host_run

pytestmark = pytest.mark.gpu


def start(n):
    x, v = workloads.plummer(n, 40 + n)
    return x, v, np.full(n, 1.0 / n)


# states within the float64 rounding of the force sums over the given steps
TOL = (("x", "x", 1e-12), ("v", "v", 1e-11), ("acc", "a", 1e-10), ("jerk", "j", 1e-9))


@pytest.mark.parametrize("n,dt_max,steps", [(2, 0.125, 3), (257, 0.125, 21), (700, 0.125, 37), (1500, 2.0 ** -9, 5)])
def test_steps_against_oracle(n, dt_max, steps):
    import paper_0902_4463_amd as g6
    x, v, m = start(n)
    eps2 = 2.0 ** -12
    dev = device_run(g6, 5, x, v, m, eps2, 0.01, dt_max, max_steps=steps, prec="fp64")
    it, st = host_run(OracleBackend(n, eps2), x, v, m, 0.01, dt_max, steps=steps)
    s = dev["state"]
    assert dev["block_steps"] == steps == it.steps and dev["particle_steps"] == it.particle_steps
    assert np.array_equal(s["t"], st.t) and np.array_equal(s["dt"], st.dt)
    for k, attr, tol in TOL:
        ref = getattr(st, attr)
        err = np.abs(s[k] - ref).max() / np.abs(ref).max()
        print(f"n={n} {k}: {err:.2e}", flush=True)
        assert err < tol, k


@pytest.mark.parametrize("n,dt_max,steps", [(257, 0.125, 21), (1500, 2.0 ** -9, 5)])
@pytest.mark.parametrize("prec", ["ds", "fp32"])
def test_float32_forces_of_a_step(n, dt_max, steps, prec):
    """The accelerations of the particles of the last block, against the
    host path's forces on the same predicted states: both within the pair
    terms' float32 rounding of the truth (1e-5 of the largest)."""
    import paper_0902_4463_amd as g6
    x, v, m = start(n)
    eps2 = 2.0 ** -12
    dev = device_run(g6, 5, x, v, m, eps2, 0.01, dt_max, max_steps=steps, prec=prec)
    back = G6Backend(n, eps2, precision=prec, handle=6)
    try:
        _, st = host_run(back, x, v, m, 0.01, dt_max, steps=steps)
    finally:
        back.close()
    s = dev["state"]
    same = s["t"] == st.t
    assert same.mean() > 0.99
    for k, attr in (("acc", "a"), ("jerk", "j")):
        ref = getattr(st, attr)[same]
        assert np.abs(s[k][same] - ref).max() <= 1e-5 * np.abs(ref).max(), k
