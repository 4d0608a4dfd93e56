"""Launch shapes chosen by the library against shapes set by hand that take
the general kernels: where a split of the j-range or the i-particles per lane
must not change the float32 sums, the results differ only by the order of the
float64 additions above them."""

import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu

# at most about 10^4 float64 additions in another order, of terms whose sum
# cancels by less than 10^3: 10^4 * 10^3 * 1e-16
RTOL = 1e-9


def evaluate(g6, s, jm, slots, xi, vi, eps2, h2, shape):
    g6.check(s.id, g6.g6mi_set_shape(s.id, *shape))
    return s.calc(jm.n, jm.meta["ti"], jm.index[slots], xi, vi, eps2, h2)


def assert_same_sums(a, b):
    for k in ("acc", "jerk", "pot"):
        d = np.linalg.norm((a[k] - b[k]).reshape(len(a[k]), -1), axis=1)
        assert np.all(d <= RTOL * np.linalg.norm(b[k].reshape(len(b[k]), -1), axis=1)), k
    for k in ("nn_index", "nn_r2", "nb_count", "nb_list"):
        assert np.array_equal(a[k], b[k]), k


@pytest.mark.parametrize("prec", ["ds", "fp32", "fp64"])
@pytest.mark.parametrize("n,ni", [(700, 512), (600, 600), (2049, 513), (4096, 767), (20001, 1025), (70000, 3000)])
def test_one_particle_per_lane_matches_two(prec, n, ni):
    """force_one (chosen from 512 i-particles on; float64 from 257) against
    force_wide (512 i-particles per workgroup asked for)."""
    import paper_0902_4463_amd as g6
    jm = workloads.random_cluster(n, seed=4000 + n)
    slots = workloads.active_set(n, ni, seed=ni)
    with g6.Session(4, precision=prec) as s:
        s.load(jm)
        xi, vi = jm.x[slots], jm.v[slots]
        a = evaluate(g6, s, jm, slots, xi, vi, 1e-4, 0.02, (0, 0))
        assert g6.g6mi_get_shape(s.id)["i_per_group"] == 256
        b = evaluate(g6, s, jm, slots, xi, vi, 1e-4, 0.02, (512, 3))
        assert g6.g6mi_get_shape(s.id)["i_per_group"] == 512
    assert_same_sums(a, b)


@pytest.mark.parametrize("prec,ni", [("ds", 1), ("ds", 2), ("ds", 9), ("ds", 16), ("fp32", 16), ("fp64", 1),
                                     ("fp64", 33), ("fp64", 256), ("fp64", 257), ("fp64", 400)])
@pytest.mark.parametrize("n", [1, 256, 257, 5000])
def test_split_count_of_small_blocks(prec, ni, n):
    """The chosen split count (down to one tile per split) against one
    split."""
    import paper_0902_4463_amd as g6
    jm = workloads.random_cluster(n, seed=4100 + n)
    rng = np.random.default_rng(ni)
    slots = np.sort(rng.permutation(n)[:ni]) if ni <= n else rng.integers(0, n, ni)
    with g6.Session(4, precision=prec) as s:
        s.load(jm)
        xi, vi = jm.x[slots], jm.v[slots]
        a = evaluate(g6, s, jm, slots, xi, vi, 1e-4, 0.02, (0, 0))
        b = evaluate(g6, s, jm, slots, xi, vi, 1e-4, 0.02, (0, 1))
        assert g6.g6mi_get_shape(s.id)["j_splits"] == 1
    assert_same_sums(a, b)


@pytest.mark.parametrize("prec", ["ds", "fp32"])
@pytest.mark.parametrize("n,ni", [(n, ni) for n in (257, 600, 1024, 4097, 5100, 33000)
                                  for ni in (17, 33, 100, 256, 300, 511)] + [(140000, 20), (140001, 100)])
def test_pieces_match_whole_splits(prec, n, ni):
    """Blocks of 17 to 511 in pieces of their j-splits, with one, two and four
    sets of lanes per workgroup (many pieces, more than one per compute unit,
    few), each starting from the minima of its split's earlier tiles, against the same splits walked whole
    (a shape set by hand).  Ragged last tiles, own slots in nearly every tile,
    no softening, lists near and far."""
    import paper_0902_4463_amd as g6
    jm = workloads.random_cluster(n, seed=4200 + n)
    ni = min(ni, n)
    slots = workloads.active_set(n, ni, seed=ni)
    ntiles = (n + 255) // 256
    ipw = 32
    while ipw < min(ni, 256):
        ipw *= 2
    with g6.Session(4, precision=prec) as s:
        s.load(jm)
        xi, vi = jm.x[slots], jm.v[slots]
        a = evaluate(g6, s, jm, slots, xi, vi, 0.0, 0.02, (0, 0))
        got = g6.g6mi_get_shape(s.id)
        # one tile per piece; the last split's pieces may be empty; a split of
        # two tiles against few i-particles stays whole
        assert got["i_per_group"] == ipw
        if ntiles == 2 and ipw <= 64:
            assert got["j_splits"] == 1
        else:
            assert ntiles <= got["j_splits"] < ntiles + max(1, ntiles // 8)
        b = evaluate(g6, s, jm, slots, xi, vi, 0.0, 0.02, (ipw, max(1, ntiles // 8)))
    assert_same_sums(a, b)


@pytest.mark.parametrize("prec", ["ds", "fp32", "fp64"])
@pytest.mark.parametrize("ni", [129, 192, 257, 300, 341, 449, 512, 513, 640, 1025])
def test_waves_dealt_over_i_blocks(prec, ni):
    """i-blocks of 256 share the block's waves of 64 rows evenly: the same
    rows as 64 at a time."""
    import paper_0902_4463_amd as g6
    jm = workloads.random_cluster(1300, seed=4400)
    slots = workloads.active_set(jm.n, ni, seed=ni)
    with g6.Session(4, precision=prec) as s:
        s.load(jm)
        xi, vi = jm.x[slots], jm.v[slots]
        a = evaluate(g6, s, jm, slots, xi, vi, 1e-6, 0.02, (256, 2))
        parts = [evaluate(g6, s, jm, slots[k:k + 64], xi[k:k + 64], vi[k:k + 64], 1e-6, 0.02, (256, 2))
                 for k in range(0, ni, 64)]
    keys = ("acc", "jerk", "pot", "nn_index", "nn_r2", "nb_count", "nb_list")
    assert_same_sums(a, {k: np.concatenate([p[k] for p in parts]) for k in keys})


@pytest.mark.parametrize("ni,changed", [(1, 1), (17, 0), (341, 341), (1024, 700), (1025, 3), (1500, 2500)])
def test_host_calls_with_and_without_copies(ni, changed):
    """Host calls whose inputs and results travel through pinned memory
    without copies (small blocks, few stored records) and those that use
    copies, against the device-resident path on the same particles; a second
    call stores `changed` records first.  Negative and large particle indices
    look their slots up outside the index array."""
    import torch

    import paper_0902_4463_amd as g6
    n = 3000
    jm = workloads.random_cluster(n, seed=4300)
    jm.index[:] = np.arange(n) * 3 - 100
    jm.index[7::11] = np.arange(len(jm.index[7::11])) + 10 ** 8
    slots = workloads.active_set(n, ni, seed=ni)
    new = np.arange(n)[::-1][:changed]
    xi, vi = jm.x[slots], jm.v[slots]
    dev = [torch.from_numpy(np.ascontiguousarray(q)).cuda() for q in (slots.astype(np.int32), xi, vi, np.full(ni, 4e-4))]
    with g6.Session(4) as s:
        s.load(jm)
        for call in range(2):
            host = s.calc(n, jm.meta["ti"], jm.index[slots], xi, vi, 1e-6, 4e-4)
            acc, jerk = (torch.zeros(ni, 3, device="cuda", dtype=torch.float64) for _ in range(2))
            pot = torch.zeros(ni, device="cuda", dtype=torch.float64)
            nnb = torch.zeros(ni, device="cuda", dtype=torch.int32)
            torch.cuda.synchronize()
            g6.check(s.id, g6.g6mi_calc_device(s.id, n, ni, dev[0], dev[1], dev[2], 1e-6, dev[3], acc, jerk, pot, nnb))
            assert g6.g6mi_last_status(s.id) == 0
            torch.cuda.synchronize()
            assert np.array_equal(host["acc"], acc.cpu().numpy()) and np.array_equal(host["jerk"], jerk.cpu().numpy())
            assert np.array_equal(host["pot"], pot.cpu().numpy()) and np.array_equal(host["nn_index"], nnb.cpu().numpy())
            assert not np.any(host["nn_index"] == jm.index[slots])
            if call == 0 and changed:
                jm.x[new] += 0.01
                jm.index[new] += 5 * 10 ** 8
                g6.check(s.id, g6.g6mi_set_j_particles(s.id, changed, new, jm.index[new], jm.t[new], None, jm.m[new],
                                                       jm.j6[new], jm.a2[new], jm.v[new], jm.x[new]))


def test_partials_of_large_float32_calls():
    """One i-particle per lane for a large float32 block takes no more memory
    for its split partials (68 bytes per i-particle and split, kept by the
    handle) than two per lane on 64 workgroups of 512 per compute unit."""
    import torch

    import paper_0902_4463_amd as g6
    n, ni, hid = 1 << 20, 1 << 18, 4
    x = torch.rand(n, 3, dtype=torch.float64, device="cuda", generator=torch.Generator("cuda").manual_seed(5))
    z, t = torch.zeros_like(x), torch.zeros(n, dtype=torch.float64, device="cuda")
    index = torch.arange(n, dtype=torch.int32, device="cuda")
    out = [torch.zeros(ni, k, dtype=torch.float64, device="cuda") for k in (3, 3, 1)]
    torch.cuda.synchronize()
    with g6.Session(hid, precision="fp32", neighbour_lists=False):
        g6.check(hid, g6.g6mi_set_j_particles_device(hid, n, t, t + 1.0 / n, index, x, z, z, z))
        g6.check(hid, g6.g6mi_calc_device(hid, n, ni, index, x, z, 1e-6, t, *out))
        shape, ncu = g6.g6mi_get_shape(hid), g6.g6mi_device_info(hid)["compute_units"]
        assert g6.g6mi_last_status(hid) == 0
    assert shape["i_per_group"] == 256
    assert 68 * ni * shape["j_splits"] <= 68 * 512 * 64 * max(ncu, 256)


@pytest.mark.parametrize("n,ni,ipw", [(1 << 18, 4096, 512), ((1 << 18) - 256, 4096, 256), (1 << 14, 1 << 16, 512)])
def test_float64_blocks_of_many_tiles_take_two_per_lane(n, ni, ipw):
    """From 2^14 tiles times i-blocks of 256 on."""
    import torch

    import paper_0902_4463_amd as g6
    x = torch.rand(max(n, ni), 3, dtype=torch.float64, device="cuda", generator=torch.Generator("cuda").manual_seed(6))
    z, t = torch.zeros_like(x), torch.zeros(len(x), dtype=torch.float64, device="cuda")
    index = torch.arange(len(x), dtype=torch.int32, device="cuda")
    out = [torch.zeros(ni, k, dtype=torch.float64, device="cuda") for k in (3, 3, 1)]
    torch.cuda.synchronize()
    with g6.Session(4, precision="fp64", neighbour_lists=False):
        g6.check(4, g6.g6mi_set_j_particles_device(4, n, t, t + 1.0 / n, index, x, z, z, z))
        slot = torch.where(index < n, index, torch.full_like(index, -1))
        torch.cuda.synchronize()
        g6.check(4, g6.g6mi_calc_device(4, n, ni, slot, x, z, 1e-6, t, *out))
        assert g6.g6mi_last_status(4) == 0
        assert g6.g6mi_get_shape(4)["i_per_group"] == ipw
