"""Workloads of the force library for timing and comparing builds.

Each case is one call (or one short run of calls) through the package's
public entry points, as a program that uses the library makes it:

  grape    the GRAPE-6 calling sequence on host arrays: store the block just
           corrected, set the time, first half, last half, nearest neighbour
           and, where asked for, the neighbour lists;
  device   one device-resident force calculation on a stream;
  batch    one batched calculation of many independent clusters;
  hermite  block steps of the integrator inside the library up to the next
           output time, and the state read back.

Positions and velocities are Plummer spheres in Henon units.  ``system``:
"salpeter" has power-law masses, softening 1e-4, neighbour radius 0.01 and
particles that were corrected at their own block times; "equal" has equal
masses, softening 1/64 and neighbour radius 0.1 (a small run's start);
"binaries" has equal masses, 5% of the particles in hard binaries, no
softening, and is shifted by 1e4 in each coordinate.
"""

from __future__ import annotations

import math

import numpy as np
import torch

import paper_0902_4463_amd as g6

TI = 2.0 ** -4          # time of the force calculations
HERMITE_SPAN = 2.0 ** -7  # time between two outputs of an integration
ETA, ETA_S, DT_MAX, DT_MIN = 0.01, 0.01, 2.0 ** -4, 2.0 ** -40
EXACT_PAIRS = 7.5e10    # pairs that the 64-bit sums manage in some 15 seconds


def listed():
    def case(name, kind, **kw):
        return dict(name=name, kind=kind, **kw)

    return [
        # one block step of a small run driven from the host by a client that
        # also wants the neighbour lists: all latency
        case("grape_1k_block24_lists", "grape", n=1024, ni=24, prec="ds", system="equal", lists=True),
        # one block step of a 32k run (its mean block is 341)
        case("grape_32k_block341", "grape", n=32768, ni=341, prec="ds", system="salpeter", lists=False),
        # the smallest block of a large run: the j-memory streamed once
        case("device_1m_block1", "device", n=1 << 20, ni=1, prec="ds", system="salpeter", lists=True),
        # a small block of a large run, not a power of two
        case("device_1m_block100", "device", n=1 << 20, ni=100, prec="ds", system="salpeter", lists=True),
        # the mean block of a 128k run, in plain float32 without lists
        case("device_128k_block785_fp32", "device", n=131072, ni=785, prec="fp32", system="salpeter", lists=False),
        # an ordinary block of a large run
        case("device_1m_block3000", "device", n=1 << 20, ni=3000, prec="ds", system="salpeter", lists=True),
        # every particle of a mid-size system of no round size (a start, an
        # energy check)
        case("device_100003_all", "device", n=100003, ni=100003, prec="ds", system="salpeter", lists=True),
        # the throughput workload: every particle of 2^20
        case("device_1m_all", "device", n=1 << 20, ni=1 << 20, prec="ds", system="salpeter", lists=True),
        # the precision workload: hard binaries far from the origin, float64
        case("device_256k_binaries_fp64", "device", n=1 << 18, ni=1 << 18, prec="fp64", system="binaries",
             lists=True),
        # 256 clusters with their own block sizes, replayed as a graph
        case("batch_256", "batch", ncl=256, nlo=256, nhi=8192, prec="ds", graph=True, lists=True),
        # a few small clusters in float64, launched directly
        case("batch_24_fp64", "batch", ncl=24, nlo=256, nhi=1024, prec="fp64", graph=False, lists=True),
        # a 32k run between two outputs
        case("hermite_32k", "hermite", n=32768, prec="ds"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["grape", "grape", "device", "device", "device", "device", "batch", "hermite"])
    prec = rng.choice(["ds", "ds", "ds", "fp64", "fp32"])
    lists = rng.random() < 0.75
    if kind == "grape":
        n = _log_int(rng, 256, 131072)
        system = "equal" if n <= 8192 and rng.random() < 0.5 else "salpeter"
        return dict(kind=kind, n=n, ni=_log_int(rng, 1, min(n, 2048)), prec=prec, system=system,
                    lists=rng.random() < 0.3)
    if kind == "device":
        n = _log_int(rng, 256, 1 << 20)
        most = min(n, int((2.0 ** 37 if prec == "fp64" else 2.0 ** 38) / n))
        ni = most if rng.random() < 0.2 else _log_int(rng, 1, most)
        system = "binaries" if prec != "fp32" and rng.random() < 0.2 else "salpeter"
        return dict(kind=kind, n=n, ni=ni, prec=prec, system=system, lists=lists)
    if kind == "batch":
        nlo = _log_int(rng, 64, 1024)
        return dict(kind=kind, ncl=_log_int(rng, 2, 512), nlo=nlo, nhi=_log_int(rng, 2 * nlo, 8192), prec=prec,
                    graph=rng.random() < 0.5, lists=lists)
    return dict(kind=kind, n=_log_int(rng, 512, 65536), prec=rng.choice(["ds", "fp64"]))


# ----------------------------------------------------------------- inputs

def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _rand(g, *shape):
    return torch.rand(*shape, generator=g, device="cuda", dtype=torch.float64)


def _isotropic(g, r):
    z = 2.0 * _rand(g, r.shape[0]) - 1.0
    phi = 2.0 * math.pi * _rand(g, r.shape[0])
    s = torch.sqrt(1.0 - z * z)
    return torch.stack([r * s * torch.cos(phi), r * s * torch.sin(phi), r * z], 1)


def _plummer(g, n):
    """Plummer sphere (mass fractions above 0.999 cut off) in Henon units."""
    length = 3.0 * math.pi / 16.0
    r = (((_rand(g, n) * 0.999).clamp_min(1e-12)) ** (-2.0 / 3.0) - 1.0) ** -0.5
    x = _isotropic(g, r)
    # speed in units of the escape speed: the inverse of the tabulated
    # cumulative distribution of q^2 (1 - q^2)^(7/2)
    q = torch.linspace(0.0, 1.0, 4097, device="cuda", dtype=torch.float64)
    f = q * q * (1.0 - q * q) ** 3.5
    cdf = torch.cat([torch.zeros(1, device="cuda", dtype=torch.float64), torch.cumsum(0.5 * (f[1:] + f[:-1]), 0)])
    cdf = cdf / cdf[-1].clone()
    u = _rand(g, n)
    k = torch.searchsorted(cdf, u).clamp(1, 4096)
    speed = q[k - 1] + (q[k] - q[k - 1]) * ((u - cdf[k - 1]) / (cdf[k] - cdf[k - 1]).clamp_min(1e-300)).clamp(0, 1)
    v = _isotropic(g, speed * math.sqrt(2.0) * (1.0 + r * r) ** -0.25)
    return x * length, v / math.sqrt(length)


def _masses(g, n):
    p = -1.35
    m = (0.1 ** p + _rand(g, n) * (100.0 ** p - 0.1 ** p)) ** (1.0 / p)
    return m / m.sum()


def _system(g, n, system, ti):
    """j-memory of n particles as float64 tensors, with eps2 and h2."""
    x, v = _plummer(g, n)
    a2 = torch.zeros(n, 3, device="cuda", dtype=torch.float64)
    j6 = torch.zeros_like(a2)
    t = torch.full((n,), ti, device="cuda", dtype=torch.float64)
    m = torch.full((n,), 1.0 / n, device="cuda", dtype=torch.float64)
    eps2, h2 = 1e-8, 1e-4
    if system == "binaries":
        nb = max(1, int(0.025 * n)) if n > 1 else 0
        a = 10.0 ** (-5.0 + 2.0 * _rand(g, nb))
        d = _isotropic(g, a)
        w = _isotropic(g, torch.ones(nb, device="cuda", dtype=torch.float64))
        w = torch.cross(d, w, dim=1)
        w = w / w.norm(dim=1, keepdim=True) * torch.sqrt(2.0 / (n * a))[:, None]  # circular orbits
        x[nb:2 * nb], v[nb:2 * nb] = x[:nb] + 0.5 * d, v[:nb] + 0.5 * w
        x[:nb], v[:nb] = x[:nb] - 0.5 * d, v[:nb] - 0.5 * w
        x = x + 1e4
        eps2 = 0.0
    else:
        a2 = torch.randn(n, 3, generator=g, device="cuda", dtype=torch.float64) / math.sqrt(12.0)
        j6 = torch.randn(n, 3, generator=g, device="cuda", dtype=torch.float64) / math.sqrt(12.0)
        step = 2.0 ** -torch.randint(6, 12, (n,), generator=g, device="cuda").double()
        t = ti - step * torch.randint(0, 2, (n,), generator=g, device="cuda").double()
        if system == "equal":
            eps2, h2 = 2.0 ** -12, 1e-2
        else:
            m = _masses(g, n)
    return dict(x=x, v=v, m=m, t=t, a2=a2, j6=j6, eps2=eps2, h2=h2)


def _predict(s, ti, rows=None):
    pick = (lambda q: q) if rows is None else (lambda q: q[rows])
    x, v, a2, j6 = (pick(s[k]) for k in ("x", "v", "a2", "j6"))
    tau = (ti - pick(s["t"]))[:, None]
    return x + tau * (v + tau * (a2 + tau * j6)), v + tau * (2.0 * a2 + tau * 3.0 * j6)


def _block(g, s, ni, ti):
    """ni active particles and their predicted state."""
    n = s["m"].shape[0]
    act = torch.randperm(n, generator=g, device="cuda")[:ni].sort().values
    xi, vi = _predict(s, ti, act)
    return act, xi.contiguous(), vi.contiguous()


def _inputs(case, seed):
    """The arrays of a grape or device case."""
    g = _gen(seed)
    s = _system(g, case["n"], case["system"], TI)
    out = dict(sys=s)
    if case["kind"] == "grape":
        # the block corrected in the step before, at its new state and time
        up = torch.randperm(case["n"], generator=g, device="cuda")[: case["ni"]].sort().values
        new = {k: q.clone() for k, q in s.items() if torch.is_tensor(q)}
        new["x"][up] += 1e-3 * s["v"][up]
        new["t"][up] = TI - 2.0 ** -9
        out.update(up=up, before=s)
        out["sys"] = s = dict(s, **new)
    out["act"], out["xi"], out["vi"] = _block(g, s, case["ni"], TI)
    return out


def _clusters(case, seed):
    """The arrays of a batch case: clusters of log-uniform sizes one after
    the other in one j-memory, blocks of 2^k of their particles, each cluster
    at its own time and place.  Sizes and blocks belong to the case, the rest
    to the seed."""
    ncl = case["ncl"]
    g = _gen(1000003 * ncl + 1009 * case["nlo"] + case["nhi"])
    size = torch.exp(math.log(case["nlo"]) + _rand(g, ncl) * math.log(case["nhi"] / case["nlo"])).long()
    k = (_rand(g, ncl) * (torch.floor(torch.log2(size.double())) + 1.0)).long()
    ni = 2 ** k
    g = _gen(seed)
    n, rows = int(size.sum()), int(ni.sum())
    joff, ioff = torch.cumsum(size, 0) - size, torch.cumsum(ni, 0) - ni
    cl = torch.repeat_interleave(torch.arange(ncl, device="cuda"), size)
    ti = torch.randint(1, 64, (ncl,), generator=g, device="cuda").double() * 2.0 ** -8
    s = _system(g, n, "salpeter", 0.0)
    s["t"] = s["t"] + ti[cl]
    run = torch.cat([torch.zeros(1, device="cuda", dtype=torch.float64), torch.cumsum(s["m"], 0)])
    s["m"] = s["m"] / (run[joff + size] - run[joff])[cl]
    s["x"] = s["x"] + (200.0 * _rand(g, ncl, 3) - 100.0)[cl]
    # the first ni of a random order of each cluster's particles, by slot
    order = torch.argsort(cl.double() + _rand(g, n))
    rank = torch.arange(n, device="cuda") - joff[cl]
    act = order[rank < ni[cl]].sort().values
    xi, vi = _predict(dict(s, t=s["t"] - ti[cl]), 0.0, act)
    host = [q.cpu().numpy() for q in (joff, size, ioff, ni, ti)]
    desc = g6.clusters(*host, np.full(ncl, s["eps2"]))
    return dict(sys=s, act=act, xi=xi.contiguous(), vi=vi.contiguous(), desc=desc, n=n, rows=rows)


def _hermite_inputs(case, seed):
    x, v = _plummer(_gen(seed), case["n"])
    return x, v, torch.full((case["n"],), 1.0 / case["n"], device="cuda", dtype=torch.float64)


# ------------------------------------------------------- prepare and run

_free_ids = list(range(g6.MAX_HANDLES - 1, -1, -1))
_shared = {}


def _stream():
    """The program's compute stream."""
    if "stream" not in _shared:
        _shared["stream"] = torch.cuda.Stream()
    return _shared["stream"]


class _Handle:
    """An open handle, closed with the state that holds it."""

    def __init__(self, prec, lists):
        self.id = _free_ids.pop()
        g6.check(self.id, g6.g6_open(self.id))
        g6.check(self.id, g6.g6mi_set_precision(self.id, prec))
        g6.check(self.id, g6.g6mi_set_neighbour_lists(self.id, lists))

    def __del__(self):
        g6.g6_close(self.id)
        _free_ids.append(self.id)


def _load(handle, s):
    n = s["m"].shape[0]
    index = torch.arange(n, device="cuda", dtype=torch.int32)
    torch.cuda.synchronize()
    g6.check(handle.id, g6.g6mi_set_j_particles_device(handle.id, n, s["t"], s["m"], index, s["x"], s["v"], s["a2"],
                                                       s["j6"], stream=_stream()))
    _stream().synchronize()


def _outputs(n):
    f = dict(device="cuda", dtype=torch.float64)
    return dict(acc=torch.zeros(n, 3, **f), jerk=torch.zeros(n, 3, **f), pot=torch.zeros(n, **f),
                nnb=torch.zeros(n, device="cuda", dtype=torch.int32), r2nn=torch.zeros(n, **f))


def prepare(case, seed):
    kind = case["kind"]
    handle = _Handle(case["prec"], case.get("lists", False))
    st = dict(kind=kind, case=case, handle=handle)
    if kind == "hermite":
        n = case["n"]
        x, v, m = (q.cpu().numpy() for q in _hermite_inputs(case, seed))
        zero = np.zeros((n, 3))
        g6.check(handle.id, g6.g6mi_set_j_particles(handle.id, n, np.arange(n), np.arange(n), np.zeros(n), None, m,
                                                    zero, zero, v, x))
        g6.check(handle.id, g6.g6mi_hermite_init(handle.id, n, 1e-8, 0.0, ETA, ETA_S, DT_MAX, DT_MIN))
        st["t"] = 0.0
        return st
    if kind == "batch":
        d = _clusters(case, seed)
        _load(handle, d["sys"])
        g6.check(handle.id, g6.g6mi_batch_use_graph(handle.id, case["graph"]))
        st.update(ncl=case["ncl"], rows=d["rows"], xi=d["xi"], vi=d["vi"], islot=d["act"].int(),
                  desc=torch.from_numpy(d["desc"].view(np.uint8).copy()).cuda(),
                  h2=torch.full((d["rows"],), d["sys"]["h2"], device="cuda", dtype=torch.float64),
                  out=_outputs(d["rows"]))
        torch.cuda.synchronize()
        return st
    d = _inputs(case, seed)
    s, ni = d["sys"], case["ni"]
    if kind == "device":
        _load(handle, s)
        st.update(xi=d["xi"], vi=d["vi"], islot=d["act"].int(), eps2=s["eps2"],
                  h2=torch.full((ni,), s["h2"], device="cuda", dtype=torch.float64), out=_outputs(ni))
        g6.g6_set_ti(handle.id, TI)
        torch.cuda.synchronize()
        return st
    n = case["n"]
    b = {k: q.cpu().numpy() for k, q in d["before"].items() if torch.is_tensor(q)}
    g6.check(handle.id, g6.g6mi_set_j_particles(handle.id, n, np.arange(n), np.arange(n), b["t"], None, b["m"],
                                                b["j6"], b["a2"], b["v"], b["x"]))
    up = d["up"]
    st.update(n=n, ni=ni, up={k: s[k][up].cpu().numpy() for k in ("t", "m", "j6", "a2", "v", "x")},
              slots=up.cpu().numpy().astype(np.int32), index=d["act"].cpu().numpy().astype(np.int32),
              xi=d["xi"].cpu().numpy(), vi=d["vi"].cpu().numpy(), eps2=s["eps2"], h2=np.full(ni, s["h2"]),
              out=dict(acc=np.zeros((ni, 3)), jerk=np.zeros((ni, 3)), pot=np.zeros(ni),
                       nnb=np.zeros(ni, dtype=np.int32), r2nn=np.zeros(ni)))
    if case["lists"]:
        st["out"].update(nb_count=np.zeros((ni, 1), dtype=np.int32),
                         nb_list=np.zeros((ni, g6.NB_MAX), dtype=np.int32))
    return st


def run(st):
    kind, id, o = st["kind"], st["handle"].id, st.get("out")
    if kind == "device":
        g6.check(id, g6.g6mi_calc_device(id, st["case"]["n"], st["case"]["ni"], st["islot"], st["xi"], st["vi"],
                                         st["eps2"], st["h2"], o["acc"], o["jerk"], o["pot"], o["nnb"], o["r2nn"],
                                         stream=_stream()))
        return o
    if kind == "batch":
        g6.check(id, g6.g6mi_batch_calc_device(id, st["ncl"], st["desc"], st["rows"], st["islot"], st["xi"],
                                               st["vi"], st["h2"], o["acc"], o["jerk"], o["pot"], o["nnb"],
                                               o["r2nn"], stream=_stream()))
        return o
    if kind == "hermite":
        st["t"] += HERMITE_SPAN
        rc, _, _, _ = g6.g6mi_hermite_advance(id, st["t"], 1 << 40)
        g6.check(id, rc)
        return g6.g6mi_hermite_state(id, st["case"]["n"])
    up, ni = st["up"], st["ni"]
    g6.check(id, g6.g6mi_set_j_particles(id, ni, st["slots"], st["slots"], up["t"], None, up["m"], up["j6"],
                                         up["a2"], up["v"], up["x"]))
    g6.g6_set_ti(id, TI)
    g6.check(id, g6.g6calc_firsthalf(id, st["n"], ni, st["index"], st["xi"], st["vi"], None, None, None,
                                     st["eps2"], st["h2"]))
    g6.check(id, g6.g6calc_lasthalf2(id, st["n"], ni, st["index"], st["xi"], st["vi"], st["eps2"], st["h2"],
                                     o["acc"], o["jerk"], o["pot"], o["nnb"]))
    g6.check(id, g6.g6_nearest_neighbour(id, ni, o["nnb"], o["r2nn"]))
    if st["case"]["lists"]:
        g6.check(id, g6.g6_read_neighbour_list(id))
        for i in range(ni):
            g6.check(id, g6.g6_get_neighbour_list(id, i, g6.NB_MAX, o["nb_count"][i], o["nb_list"][i]))
    return o


# ------------------------------------------------------------------ work

def _hermite_steps(n):
    """About how many block steps, of what mean size, one output interval
    takes (measured: 370 blocks of 341 at n = 32768; the block grows about
    as n^0.6)."""
    return 370.0 * (n / 32768.0) ** 0.4, max(1.0, 341.0 * (n / 32768.0) ** 0.6)


def work(case):
    """j-records read once (116 B), i-particles read (60 B) and results
    written (68 B) once; 60 operations per pair."""
    if case["kind"] == "hermite":
        steps, block = _hermite_steps(case["n"])
        return dict(bytes=steps * (116.0 * case["n"] + 128.0 * block), flops=60.0 * steps * block * case["n"])
    if case["kind"] == "batch":
        # means of the log-uniform size n and of the block 2^k, k uniform in
        # 0 .. log2 n: about 2 n / log2(2 n)
        lo, hi, ncl = case["nlo"], case["nhi"], case["ncl"]
        n = (hi - lo) / math.log(hi / lo)
        ni = 1.5 * n / math.log2(2.0 * n)
        pairs = 1.5 * (hi * hi - lo * lo) / (2.0 * math.log(hi / lo)) / math.log2(2.0 * n)
        return dict(bytes=ncl * (116.0 * n + 128.0 * ni), flops=60.0 * ncl * pairs)
    n, ni = case["n"], case["ni"]
    extra = 128.0 * ni if case["kind"] == "grape" else 0.0  # the stored block
    return dict(bytes=116.0 * n + 128.0 * ni + extra, flops=60.0 * n * ni)


# ----------------------------------------------------------------- exact

def _forces(xp, vp, m, xi, vi, act, eps2):
    """Direct sums in float64; act: each i-particle's own row."""
    n, ni = xp.shape[0], xi.shape[0]
    acc, jerk = torch.empty_like(xi), torch.empty_like(xi)
    pot, r2nn = torch.empty(ni, device="cuda", dtype=torch.float64), torch.empty(ni, device="cuda", dtype=torch.float64)
    xj, vj = xp.t().contiguous(), vp.t().contiguous()
    step = max(1, (1 << 25) // n)
    for a in range(0, ni, step):
        b = min(ni, a + step)
        own = (torch.arange(b - a, device="cuda"), act[a:b])
        d = [xj[k][None, :] - xi[a:b, k, None] for k in range(3)]
        w = [vj[k][None, :] - vi[a:b, k, None] for k in range(3)]
        r2 = d[0] * d[0]
        r2.addcmul_(d[1], d[1]).addcmul_(d[2], d[2])
        r2[own] = math.inf
        r2nn[a:b] = r2.min(dim=1).values
        rinv = (r2 + eps2).rsqrt_()
        rv = d[0] * w[0]
        rv.addcmul_(d[1], w[1]).addcmul_(d[2], w[2])
        mr = rinv * m
        pot[a:b] = -mr.sum(dim=1)
        rinv.mul_(rinv)
        mr.mul_(rinv)
        rv.mul_(rinv).mul_(-3.0)
        for k in range(3):
            acc[a:b, k] = (mr * d[k]).sum(dim=1)
            jerk[a:b, k] = w[k].addcmul_(rv, d[k]).mul_(mr).sum(dim=1)
    return acc, jerk, pot, r2nn


def _exact_hermite(case, seed):
    """Fourth-order Hermite with block time steps up to the first output."""
    x, v, m = _hermite_inputs(case, seed)
    n, eps2 = case["n"], 1e-8
    rows = torch.arange(n, device="cuda")
    acc, jerk, pot, _ = _forces(x, v, m, x, v, rows, eps2)
    t = torch.zeros(n, device="cuda", dtype=torch.float64)

    def power2(dt):
        return torch.ldexp(torch.ones_like(dt), torch.frexp(dt).exponent - 1)

    dt = power2((ETA_S * acc.norm(dim=1) / jerk.norm(dim=1)).clamp(DT_MIN, DT_MAX))
    while True:
        tn = t + dt
        tb = float(tn.min())
        if tb > HERMITE_SPAN:
            break
        act = (tn == tb).nonzero()[:, 0]
        s = dict(x=x, v=v, a2=acc / 2.0, j6=jerk / 6.0, t=t)
        xp, vp = _predict(s, tb)
        a1, j1, p1, _ = _forces(xp, vp, m, xp[act], vp[act], act, eps2)
        h = dt[act][:, None]
        a0, j0 = acc[act], jerk[act]
        a2 = (-6.0 * (a0 - a1) - h * (4.0 * j0 + 2.0 * j1)) / h ** 2
        a3 = (12.0 * (a0 - a1) + 6.0 * h * (j0 + j1)) / h ** 3
        x[act] = xp[act] + a2 * h ** 4 / 24.0 + a3 * h ** 5 / 120.0
        v[act] = vp[act] + a2 * h ** 3 / 6.0 + a3 * h ** 4 / 24.0
        na, nj, n2, n3 = (q.norm(dim=1) for q in (a1, j1, a2 + h * a3, a3))
        want = torch.sqrt(ETA * (na * n2 + nj * nj) / (nj * n3 + n2 * n2).clamp_min(1e-300))
        old = dt[act]
        new = torch.where(want < old, torch.minimum(old, power2(want.clamp_min(DT_MIN))), old)
        twice = 2.0 * old
        grow = (want >= twice) & (torch.remainder(torch.full_like(old, tb), twice) == 0.0) & (twice <= DT_MAX)
        dt[act] = torch.where(grow, twice, new)
        acc[act], jerk[act], pot[act], t[act] = a1, j1, p1, tb
    return dict(x=x, v=v, acc=acc, jerk=jerk, pot=pot, t=t, dt=dt)


def exact(case, seed):
    kind = case["kind"]
    if kind == "hermite":
        return _exact_hermite(case, seed)
    if kind == "batch":
        d = _clusters(case, seed)
        s, parts = d["sys"], []
        for c in d["desc"]:
            j = slice(int(c["joff"]), int(c["joff"] + c["nj"]))
            i = slice(int(c["ioff"]), int(c["ioff"] + c["ni"]))
            sub = {k: s[k][j] for k in ("x", "v", "a2", "j6", "t")}
            xp, vp = _predict(sub, float(c["ti"]))
            parts.append(_forces(xp, vp, s["m"][j], d["xi"][i], d["vi"][i], d["act"][i] - int(c["joff"]), s["eps2"]))
        acc, jerk, pot, r2nn = (torch.cat(q) for q in zip(*parts))
        return dict(acc=acc, jerk=jerk, pot=pot, nnb=None, r2nn=r2nn)
    if float(case["n"]) * case["ni"] > EXACT_PAIRS:
        return None
    d = _inputs(case, seed)
    s = d["sys"]
    xp, vp = _predict(s, TI)
    acc, jerk, pot, r2nn = _forces(xp, vp, s["m"], d["xi"], d["vi"], d["act"], s["eps2"])
    if kind == "device":
        return dict(acc=acc, jerk=jerk, pot=pot, nnb=None, r2nn=r2nn)
    out = dict(acc=acc.cpu().numpy(), jerk=jerk.cpu().numpy(), pot=pot.cpu().numpy(), nnb=None,
               r2nn=r2nn.cpu().numpy())
    if case["lists"]:
        out.update(nb_count=None, nb_list=None)
    return out
