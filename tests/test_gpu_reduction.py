"""GPU reduction of the split partials: rows per workgroup and splits per
lane at their edges, and neighbour lists of every length the two list sorts
meet (a team of four lanes up to 16 entries, a wave up to 256)."""

import numpy as np
import pytest

import workloads
from tests import parity

pytestmark = pytest.mark.gpu

LENGTHS = (0, 1, 2, 4, 5, 15, 16, 17, 63, 64, 65, 255, 256, 257)


@pytest.fixture(scope="module")
def system():
    import oracle
    n = 6000
    rng = np.random.default_rng(17)
    idx = (rng.permutation(n) * 3 - n).astype(np.int32)
    jm = workloads.make_jmemory(rng.uniform(-1.0, 1.0, (n, 3)), rng.normal(size=(n, 3)), np.full(n, 1.0 / n),
                                index=idx, meta=dict(ti=0.0))
    return oracle, jm


@pytest.mark.parametrize("ni", [1, 2, 63, 64, 65, 257])
@pytest.mark.parametrize("splits", [1, 2, 9, 23])
def test_rows_splits_and_list_lengths(system, ni, splits):
    """Float64 forces to the oracle's tolerance of that variant, the nearest
    neighbour exact, and each list exact: its radius lies halfway between two
    neighbours' distances."""
    import paper_0902_4463_amd as g6
    orc, jm = system
    slots = workloads.active_set(jm.n, ni, seed=ni)
    h2 = np.empty(ni)
    for r, s in enumerate(slots):
        d2 = np.sort(((jm.x - jm.x[s]) ** 2).sum(axis=1))[1:]
        k = LENGTHS[r % len(LENGTHS)]
        h2[r] = 0.5 * (d2[k - 1] + d2[k]) if k else 0.5 * d2[0]
    ref = orc.evaluate(jm, 0.0, slots, 1e-6, h2, conditioning=True)
    with g6.Session(3, precision="fp64") as s:
        s.load(jm)
        g6.check(s.id, g6.g6mi_set_shape(s.id, 0, splits))
        gpu = s.calc(jm.n, 0.0, jm.index[slots], ref["xi"], ref["vi"], 1e-6, h2)
        assert g6.g6mi_get_shape(s.id)["j_splits"] == splits
    rep = parity.force_report(gpu, ref)
    print(f"ni={ni} splits={splits}: acc={rep['acc_max']:.1e} jerk={rep['jerk_max']:.1e}", flush=True)
    assert rep["acc_max"] < 1e-12 and rep["jerk_max"] < 1e-11 and rep["pot_max"] < 1e-13
    assert np.array_equal(gpu["nn_index"], ref["nn_index"])
    assert np.array_equal(gpu["nb_count"], ref["nb_count"])
    assert np.array_equal(gpu["nb_count"], [LENGTHS[r % len(LENGTHS)] for r in range(ni)])
    assert np.array_equal(gpu["nb_list"], ref["nb_list"])
