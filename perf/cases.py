"""Performance cases of the lattice heat bath, through the package's Python entry points.

Each case is one call, or the two or three calls, that a Monte Carlo program makes over and
over: sweeps of one lattice (smallest, ordinary, largest; FP32, FP64, SU(3)), sweeps of a batch
of replicas, training steps of the learned proposal, measurements on a configuration, and the
exchange of a configuration with the host.  `exact` gives the same results in 64 bits from
plain torch: the chains are driven by Philox4x32-10 counters, so a heat-bath sweep has one.
"""
import math

import numpy as np
import torch

import paper_1010_1486_amd as su2

BOTH = su2.SU2_MEAS_PLAQ | su2.SU2_MEAS_POLY


# ------------------------------------------------------------------ cases
def listed():
    return [
        # The smallest lattice (parity and teaching runs): latency of whole sweeps.
        {"name": "lattice_4x4x4x4", "kind": "lattice", "nx": 4, "ny": 4, "nz": 4, "nt": 4,
         "beta": 2.3, "sweeps": 100, "reunit": 10, "hot": True},
        # One ordinary chain with unequal extents: heat bath with microcanonical
        # over-relaxation, every pass a launch of its own.
        {"name": "overrelax_18x12x10x14", "kind": "overrelax", "nx": 18, "ny": 12, "nz": 10,
         "nt": 14, "beta": 2.4, "sweeps": 4, "reunit": 4, "n_or": 3, "hot": True},
        # The benchmark lattice: a captured reunitarisation period, replayed.
        {"name": "replay_48x48x48x48", "kind": "replay", "nx": 48, "ny": 48, "nz": 48, "nt": 48,
         "beta": 6.0, "sweeps": 10, "hot": True},
        # The scan over couplings: 16 values, each from a cold and a hot start.
        {"name": "scan_32_of_16x16x16x16", "kind": "scan", "n": 32, "nx": 16, "ny": 16, "nz": 16,
         "nt": 16, "beta": 1.5, "beta_hi": 3.0, "sweeps": 10, "reunit": 10, "poly": False},
        # The Polyakov loop against temperature: 13 couplings at each of three Nt.
        {"name": "polyakov_39_of_32x32x32xNt", "kind": "scan", "n": 39, "nx": 32, "ny": 32,
         "nz": 32, "nt": 0, "beta": 2.0, "beta_hi": 2.6, "sweeps": 5, "reunit": 0, "poly": True},
        # The learned proposal on uneven replicas (L = 8..20).
        {"name": "learned_64_of_8..20", "kind": "learned", "n": 64, "lo": 8, "hi": 20,
         "beta": 1.8, "beta_hi": 3.0, "sweeps": 10, "width": -1.0},
        # FP64 links.
        {"name": "f64_24x24x24x24", "kind": "f64", "nx": 24, "ny": 24, "nz": 24, "nt": 24,
         "beta": 2.0, "sweeps": 4, "reunit": 4, "hot": True},
        # SU(3) at the benchmark size.
        {"name": "su3_48x48x48x48", "kind": "su3", "nx": 48, "ny": 48, "nz": 48, "nt": 48,
         "beta": 6.0, "sweeps": 2, "reunit": 10, "hot": True},
        # A batch of small SU(3) lattices near the transition, with the Polyakov loop.
        {"name": "su3_64_of_16x16x16x4", "kind": "su3_scan", "n": 64, "nx": 16, "ny": 16,
         "nz": 16, "nt": 4, "beta": 5.4, "beta_hi": 6.0, "sweeps": 4, "reunit": 10, "hot": True},
        # Training steps of the learned proposal (forward, backward, Adam).
        {"name": "train_16384", "kind": "train", "samples": 262144, "batch": 16384, "steps": 20,
         "lr": 3e-3},
        # All measurements on one configuration: Wilson loops for the scale, plaquette,
        # Polyakov loop.
        {"name": "measure_32x32x32x32", "kind": "measure", "nx": 32, "ny": 32, "nz": 32, "nt": 32,
         "size": 4},
        # A configuration saved to the host layout and loaded into another lattice.
        {"name": "exchange_32x32x32x32", "kind": "exchange", "nx": 32, "ny": 32, "nz": 32,
         "nt": 32},
    ]


def _even(rng, lo, hi):
    return 2 * rng.randint(lo // 2, hi // 2)


def _spread(rng, lo, hi):
    """An even number, log-uniform in [lo, hi]."""
    v = math.exp(rng.uniform(math.log(lo), math.log(hi + 1.99)))
    return max(lo, min(hi, 2 * int(v / 2)))


def _extents(rng, lo, hi):
    """Four even extents around one size that is log-uniform in [lo, hi]."""
    m = _spread(rng, lo, hi)
    e = [max(lo, min(hi, m + 2 * rng.randint(-m // 8, m // 8))) for _ in range(4)]
    return {"nx": e[0], "ny": e[1], "nz": e[2], "nt": e[3]}


def draw(rng):
    """One more case of the kinds and ranges that the listed ones stand for."""
    kind = rng.choice([c["kind"] for c in listed()])
    beta = round(rng.uniform(1.8, 3.0), 3)
    if kind == "lattice":
        # whole-sweep lattices and the first sizes beyond them
        return {"kind": kind, **_extents(rng, 4, 10), "beta": beta,
                "sweeps": rng.randint(10, 100), "reunit": rng.choice([0, 5, 10]),
                "hot": rng.random() < 0.5}
    if kind == "overrelax":
        return {"kind": kind, **_extents(rng, 8, 32), "beta": beta, "sweeps": rng.randint(1, 5),
                "reunit": rng.choice([0, 2]), "n_or": rng.randint(1, 4), "hot": True}
    if kind == "replay":
        return {"kind": kind, **_extents(rng, 12, 48), "beta": round(rng.uniform(2.0, 6.0), 3),
                "sweeps": rng.choice([5, 10]), "hot": True}
    if kind == "scan":
        e = _extents(rng, 8, 24)
        return {"kind": kind, "n": rng.randint(5, 32), **e, "beta": 1.5,
                "beta_hi": round(rng.uniform(2.5, 3.0), 3), "sweeps": rng.randint(2, 10),
                "reunit": rng.choice([0, 5]), "poly": rng.random() < 0.5}
    if kind == "learned":
        lo = _even(rng, 6, 10)
        return {"kind": kind, "n": rng.randint(9, 64), "lo": lo, "hi": lo + _even(rng, 2, 10),
                "beta": 1.8, "beta_hi": 3.0, "sweeps": rng.randint(2, 10),
                "width": rng.choice([-1.0, 0.02])}
    if kind == "f64":
        return {"kind": kind, **_extents(rng, 8, 40), "beta": beta, "sweeps": rng.randint(2, 4),
                "reunit": rng.choice([0, 2]), "hot": rng.random() < 0.5}
    if kind == "su3":
        return {"kind": kind, **_extents(rng, 8, 46), "beta": round(rng.uniform(5.4, 6.4), 3),
                "sweeps": rng.randint(1, 3), "reunit": rng.choice([0, 2]), "hot": True}
    if kind == "su3_scan":
        return {"kind": kind, "n": rng.randint(5, 64), **_extents(rng, 6, 14), "beta": 5.4,
                "beta_hi": 6.0, "sweeps": rng.randint(1, 4), "reunit": 2, "hot": False}
    if kind == "train":
        return {"kind": kind, "samples": rng.randint(20000, 300000),
                "batch": int(math.exp(rng.uniform(math.log(256), math.log(20000)))),
                "steps": rng.randint(5, 30), "lr": 3e-3}
    if kind == "measure":
        return {"kind": kind, **_extents(rng, 6, 32), "size": rng.randint(2, 4)}
    return {"kind": kind, **_extents(rng, 6, 36)}


# ---------------------------------------------------------------- helpers
def _dims(c, nt=None):
    return [c["nx"], c["ny"], c["nz"], c["nt"] if nt is None else nt]


def _couplings(c):
    n = c["n"]
    return [c["beta"] + (c["beta_hi"] - c["beta"]) * r / max(n - 1, 1) for r in range(n)]


def _replicas(c):
    """Extents, couplings and starts of the replicas of a scan."""
    n = c["n"]
    if c["nt"] == 0:  # the temperature grid: Nt = 4, 6, 8, the couplings repeated for each
        m = n // 3
        b = [c["beta"] + (c["beta_hi"] - c["beta"]) * k / max(m - 1, 1) for k in range(m)]
        return ([_dims(c, 4 + 2 * (r // m)) for r in range(3 * m)], [b[r % m] for r in range(3 * m)],
                [su2.SU2_COLD] * (3 * m))
    m = (n + 1) // 2
    b = [c["beta"] + (c["beta_hi"] - c["beta"]) * k / max(m - 1, 1) for k in range(m)]
    return ([_dims(c)] * n, [b[r // 2] for r in range(n)],
            [su2.SU2_HOT if r % 2 else su2.SU2_COLD for r in range(n)])


class _DeviceArray:
    """Device memory of the library as a torch tensor (no copy); keeps its owner alive."""

    def __init__(self, owner, ptr, shape, typestr):
        self.owner = owner
        self.__cuda_array_interface__ = {"shape": shape, "typestr": typestr, "data": (ptr, False),
                                         "strides": None, "version": 2}


def _view(owner, ptr, shape, typestr):
    return torch.as_tensor(_DeviceArray(owner, ptr, shape, typestr), device="cuda:0")


_streams = []


def _stream():
    """The one stream other than the default that captured sweeps run on."""
    if not _streams:
        _streams.append(torch.cuda.Stream())
    return _streams[0]


def _parity(dims):
    """Parity of every site, canonical order (x fastest)."""
    g = [torch.arange(n, device="cuda:0") for n in dims]
    return ((g[3][:, None, None, None] + g[2][:, None, None] + g[1][:, None] + g[0]) & 1).reshape(-1)


def _to_classes(U, dims):
    """[mu][t, z, y, x, ...] -> [mu * 2 + parity][half-site, ...]."""
    V = math.prod(dims)
    p = _parity(dims).reshape(V // 2, 2)
    i = torch.arange(V // 2, device=p.device)
    out = []
    for mu in range(4):
        u = U[mu].reshape(V // 2, 2, *U[mu].shape[4:])
        out += [u[i, (p[:, 0] != par).long()] for par in (0, 1)]
    return torch.stack(out)


def _near_unit(dims, seed, spread):
    """Seeded SU(2) links near the identity, like a configuration at weak coupling, as FP32
    (4, Nt, Nz, Ny, Nx, 4)."""
    g = torch.Generator(device="cuda:0").manual_seed(seed)
    u = spread * torch.randn((4, *dims[::-1], 4), generator=g, device="cuda:0")
    u[..., 0] += 1.0
    return u / u.double().norm(dim=-1, keepdim=True).float()


def _samples(c, seed):
    """Training pairs: alpha log-uniform in [0.5, 30], a0 from sqrt(1 - a0^2) exp(alpha a0)
    (Kennedy-Pendleton)."""
    g = np.random.default_rng(seed)
    n = c["samples"]
    alpha = (0.5 * 60.0 ** g.random(n)).astype(np.float32)
    a0 = np.empty(n, np.float32)
    left = np.arange(n)
    while left.size:
        r = 1.0 - g.random((4, left.size))
        d = -(np.log(r[0]) + np.cos(2 * np.pi * r[1]) ** 2 * np.log(r[2])) / alpha[left]
        ok = r[3] ** 2 <= 1.0 - 0.5 * d
        a0[left[ok]] = 1.0 - d[ok]
        left = left[~ok]
    return alpha, a0


def _start_params(seed):
    """Network parameters a program starts from: hidden layers uniform in 1/sqrt(fan in), output
    weights small, output biases of the identity spline."""
    g = np.random.default_rng(seed)
    p = np.zeros(2671, np.float32)
    p[0:32] = g.uniform(-1, 1, 32)
    p[64:1088] = g.uniform(-1, 1, 1024) / np.sqrt(32)
    p[1120:2624] = g.uniform(-0.05, 0.05, 1504)
    p[2656:2671] = np.log(np.expm1(1.0 - 1e-3))
    return p


def _fitted_params(seed):
    """Network parameters of a proposal that fits the heat bath: random hidden layers and output
    weights by least squares on the spline whose knots are quantiles of the exact density."""
    g = np.random.default_rng(seed)
    p = np.zeros(2671, np.float64)
    p[0:32], p[32:64] = g.uniform(-2, 2, 32), g.uniform(-1, 1, 32)
    p[64:1088], p[1088:1120] = g.uniform(-1, 1, 1024) / 4, g.uniform(-1, 1, 32)
    f = np.linspace(-1, 1, 64)
    x = np.linspace(-1, 1, 4001)
    want = np.empty((f.size, 47))
    for i, fi in enumerate(f):
        al = 0.5 * 60.0 ** ((fi + 1) / 2)
        w = np.sqrt(1 - x * x) * np.exp(al * (x - 1)) + 1e-7
        cdf = np.concatenate([[0.0], np.cumsum(0.5 * (w[1:] + w[:-1]))])
        cdf /= cdf[-1]
        # knots at mixed quantiles of the density and of the interval
        q = np.interp(np.linspace(0, 1, 17), 0.8 * cdf + 0.1 * (x + 1), x)
        q[0], q[-1] = -1.0, 1.0
        W, H = np.diff(q) / 2, np.diff(np.interp(q, x, cdf))
        pw, ph = (W - 1e-3) / (1 - 16e-3), (H - 1e-3) / (1 - 16e-3)
        dens = np.interp(q[1:-1], x, w) / (np.sum(0.5 * (w[1:] + w[:-1])) * (x[1] - x[0])) * 2
        want[i, :16], want[i, 16:32] = np.log(np.maximum(pw, 1e-5)), np.log(np.maximum(ph, 1e-5))
        want[i, 32:] = np.log(np.expm1(np.clip(dens, 5e-3, 50) - 1e-3))
    want[:, :16] -= want[:, :16].mean(1, keepdims=True)
    want[:, 16:32] -= want[:, 16:32].mean(1, keepdims=True)
    h1 = np.tanh(f[:, None] * p[0:32] + p[32:64])
    h2 = np.tanh(h1 @ p[64:1088].reshape(32, 32).T + p[1088:1120])
    A = np.vstack([np.hstack([h2, np.ones((f.size, 1))]), 1e-3 * np.eye(33)])
    sol = np.linalg.lstsq(A, np.vstack([want, np.zeros((33, 47))]), rcond=None)[0]
    p[1120:2624], p[2624:] = sol[:32].T.reshape(-1), sol[32]
    return p.astype(np.float32)


# ---------------------------------------------------------------- prepare
def prepare(case, seed):
    c, k = case, case["kind"]
    s = {"c": c}
    start = su2.SU2_HOT if c.get("hot") else su2.SU2_COLD
    if k in ("lattice", "overrelax", "replay"):
        # capture needs a stream that is not the default one
        stream = _stream() if k == "replay" else torch.cuda.current_stream()
        with torch.cuda.stream(stream):
            s["lat"] = lat = su2.Lattice(_dims(c), c["beta"], seed, start)
        s["links"] = lat.links_t.view(torch.float32).view(8, -1, 4)
        rows = c["sweeps"] * (1024 if k == "replay" else 1)
        s["hist"] = torch.zeros((rows, 3), dtype=torch.float64, device="cuda:0")
        if k == "overrelax":
            lat.set_hb_overrelax(c["n_or"])
        if k == "replay":
            torch.cuda.synchronize()  # the history is cleared on the default stream
            lat.set_reunit_fused(True)
            s["pass"] = 1024
            _capture(s)
    elif k == "scan":
        d, b, st = _replicas(c)
        s["batch"] = su2.Batch(d, b, st, seed)
        s["hist"] = torch.zeros((c["sweeps"], len(d), 3), dtype=torch.float64, device="cuda:0")
    elif k == "learned":
        sizes = list(range(c["lo"], c["hi"] + 1, 2))
        d = [[sizes[r % len(sizes)]] * 4 for r in range(c["n"])]
        s["batch"] = b = su2.Batch(d, _couplings(c), su2.SU2_HOT, seed)
        s["nn"] = nn = su2.NN(_fitted_params(seed))
        nn.build_table()
        b.set_proposal(nn)
        b.set_overrelax(c["width"])
        s["hist"] = torch.zeros((c["sweeps"], c["n"], 3), dtype=torch.float64, device="cuda:0")
    elif k == "f64":
        d = _dims(c)
        s["lat"] = lat = su2.Lattice64(d, c["beta"], seed, start)
        ptr, _ = su2.su2_links_device(lat.h)
        s["links"] = _view(lat, ptr, (8, 2, math.prod(d) // 2, 2), "<f8")
        s["hist"] = torch.zeros((c["sweeps"], 3), dtype=torch.float64, device="cuda:0")
    elif k == "su3":
        d = _dims(c)
        s["lat"] = su2.Lattice3(d, c["beta"], seed, start)
    elif k == "su3_scan":
        s["batch"] = su2.Batch3(_dims(c), _couplings(c), seed, start)
    elif k == "train":
        s["nn"] = nn = su2.NN(_start_params(seed))
        nn.set_data(*_samples(c, seed))
    elif k in ("measure", "exchange"):
        d = _dims(c)
        s["lat"] = lat = su2.Lattice(d, 2.4, seed)
        links = lat.links_t.view(torch.float32).view(8, -1, 4)
        links.copy_(_to_classes(_near_unit(d, seed, 0.3), d))
        if k == "exchange":
            s["to"] = su2.Lattice(d, 2.4, seed)
            s["links"] = s["to"].links_t.view(torch.float32).view(8, -1, 4)
    return s


def _capture(s):
    """Record one period of sweeps; its rows start again at the front of the history."""
    n = s["c"]["sweeps"]
    if (s["pass"] + 1) * n > s["hist"].shape[0]:
        s["lat"].capture(n, su2.SU2_KP, n, su2.SU2_MEAS_PLAQ, s["hist"])
        s["pass"] = 0


# -------------------------------------------------------------------- run
def run(state):
    s, c = state, state["c"]
    k = c["kind"]
    if k == "lattice":
        s["lat"].sweep_measure(c["sweeps"], su2.SU2_KP, c["reunit"], BOTH, s["hist"])
        return {"links": s["links"], "history": s["hist"]}
    if k == "overrelax":
        s["lat"].sweep_measure(c["sweeps"], su2.SU2_KP_OR, c["reunit"], BOTH, s["hist"])
        return {"links": s["links"], "history": s["hist"]}
    if k == "replay":
        _capture(s)
        s["lat"].replay(1)
        n, s["pass"] = c["sweeps"], s["pass"] + 1
        return {"links": s["links"], "history": s["hist"][(s["pass"] - 1) * n:s["pass"] * n]}
    if k == "scan":
        s["batch"].sweep_measure(c["sweeps"], su2.SU2_KP, c["reunit"],
                                 BOTH if c["poly"] else su2.SU2_MEAS_PLAQ, s["hist"])
        return {"history": s["hist"]}
    if k == "learned":
        s["batch"].sweep_measure(c["sweeps"], su2.SU2_LEARNED, 0, su2.SU2_MEAS_PLAQ, s["hist"])
        return {"history": s["hist"]}
    if k == "f64":
        s["lat"].sweep_measure(c["sweeps"], su2.SU2_KP, c["reunit"], BOTH, s["hist"])
        return {"links": s["links"], "history": s["hist"]}
    if k == "su3":
        h = s["lat"].heatbath_sweep(c["sweeps"], c["reunit"], history=True)
        return {"plaquettes": h, "polyakov": s["lat"].polyakov()}
    if k == "su3_scan":
        h = s["batch"].heatbath_sweep(c["sweeps"], c["reunit"], history=True)
        return {"plaquettes": h, "polyakov": s["batch"].polyakov()}
    if k == "train":
        h = s["nn"].train(c["steps"], c["batch"], c["lr"], 1e-5)
        return {"loss": h, "params": s["nn"].params}
    if k == "measure":
        lat = s["lat"]
        return {"wilson": lat.wilson_loops(c["size"], c["size"]), "plaquette": lat.plaquette(),
                "polyakov": lat.polyakov()}
    links = s["lat"].get_links()
    s["to"].set_links(links)
    return {"saved": links, "loaded": s["links"]}


# ------------------------------------------------------------------- work
def _sweeps_work(V, sweeps, per_link, site_bytes):
    """Sweeps of V sites: the links read and written once a sweep (a sweep's last pass needs what
    its first wrote), `per_link` operations for each of the 4 V links."""
    return {"bytes": 2.0 * site_bytes * V * sweeps, "flops": 4.0 * V * sweeps * per_link}


def work(case):
    # operations of one update: twelve products of the six staples, the sum, the sampler (about
    # 60) and the product with the sampled element; SU(2) products are 28 operations, SU(3) 198
    c, k = case, case["kind"]
    su2_link, su3_link = 12 * 28 + 20 + 60 + 28, 12 * 198 + 90 + 198 + 3 * 150
    if k in ("lattice", "replay"):
        return _sweeps_work(math.prod(_dims(c)), c["sweeps"], su2_link, 64)
    if k == "f64":
        return _sweeps_work(math.prod(_dims(c)), c["sweeps"], su2_link, 128)
    if k == "overrelax":
        return _sweeps_work(math.prod(_dims(c)), c["sweeps"] * (1 + c["n_or"]), su2_link, 64)
    if k == "scan":
        V = sum(math.prod(d) for d in _replicas(c)[0])
        return _sweeps_work(V, c["sweeps"], su2_link, 64)
    if k == "learned":
        sizes = list(range(c["lo"], c["hi"] + 1, 2))
        V = sum(sizes[r % len(sizes)] ** 4 for r in range(c["n"]))
        return _sweeps_work(V, c["sweeps"], su2_link + 100, 64)
    if k == "su3":
        return _sweeps_work(math.prod(_dims(c)), c["sweeps"], su3_link, 192)
    if k == "su3_scan":
        return _sweeps_work(c["n"] * math.prod(_dims(c)), c["sweeps"], su3_link, 192)
    if k == "train":
        n = c["steps"] * c["batch"]
        # 32 + 1024 + 1504 multiply-adds forward, twice that backward, about 600 for the spline
        return {"bytes": 8.0 * n + c["steps"] * 2671 * 24.0, "flops": n * (6.0 * 2560 + 600)}
    V = math.prod(_dims(c))
    if k == "measure":
        m = c["size"]
        return {"bytes": 64.0 * V, "flops": V * (6.0 * 28 * (2 * m + 4 * m * m) + 6 * 60 + 28)}
    return {"bytes": 4 * 64.0 * V, "flops": 0.0}


# ------------------------------------------------------------------ exact
M32 = 0xFFFFFFFF


def _philox(c0, c1, c2, c3, seed):
    """Philox4x32-10 on int64 tensors of 32-bit words."""
    k0, k1 = seed & M32, (seed >> 32) & M32
    c1, c2, c3 = (torch.full_like(c0, v) if isinstance(v, int) else v for v in (c1, c2, c3))
    for _ in range(10):
        p0, p1 = c0 * 0xD2511F53, c2 * 0xCD9E8D57  # low 64 bits: the product is exact modulo 2^64
        c0, c1, c2, c3 = (((p1 >> 32) & M32) ^ c1 ^ k0, p1 & M32, ((p0 >> 32) & M32) ^ c3 ^ k1,
                          p0 & M32)
        k0, k1 = (k0 + 0x9E3779B9) & M32, (k1 + 0xBB67AE85) & M32
    return c0, c1, c2, c3


def _u01(w):
    return (2 * (w >> 9) + 1).double() * 2.0 ** -24


def _mul(a, b):
    w, v, x, y = a[..., :1], a[..., 1:], b[..., :1], b[..., 1:]
    return torch.cat([w * x - (v * y).sum(-1, keepdim=True),
                      w * y + x * v - torch.linalg.cross(v, y)], -1)


def _dag(a):
    return a * torch.tensor([1.0, -1.0, -1.0, -1.0], dtype=a.dtype, device=a.device)


def _up(U, mu, n=1):
    return torch.roll(U, -n, 3 - mu)


def _heatbath(V, beta, site, sweep, word, seed):
    """New SU(2) elements for staple sums V (n, 4): X (V/|V|)^+, X from its exact density."""
    k = V.norm(dim=-1)
    alpha = beta * k
    kp = alpha >= 1.0
    delta = torch.zeros_like(k)
    left = torch.arange(k.numel(), device=k.device)
    first, t = None, 0
    while left.numel():
        w = _philox(site[left], sweep, word, t, seed)
        if first is None:
            first = w
        r1, r2, r3, r4 = (_u01(x) for x in w)
        a, isk = alpha[left], kp[left]
        d = -(r1.log() + torch.cos(2 * math.pi * r2) ** 2 * r3.log()) / a
        h = 1.0 - r1.sqrt() * torch.cos(2 * math.pi * r2)
        ok = torch.where(isk, r4 * r4 <= 1 - 0.5 * d, r3 <= torch.exp(-a * h))
        delta[left[ok]] = torch.where(isk, d, h)[ok]
        left, t = left[~ok], t + 1
    a, b, c, d = (x & 511 for x in first)
    r5, r6 = ((2 * (x | (y << 9)) + 1).double() * 2.0 ** -19 for x, y in ((a, b), (c, d)))
    mag, sth = (delta * (2 - delta)).sqrt(), 2 * (r5 * (1 - r5)).sqrt()
    X = torch.stack([1 - delta, mag * sth * torch.cos(2 * math.pi * r6),
                     mag * sth * torch.sin(2 * math.pi * r6), mag * (1 - 2 * r5)], -1)
    return _mul(X, _dag(V / k[:, None]))


def _start2(dims, hot, seed, replica):
    V = math.prod(dims)
    site = torch.arange(V, device="cuda:0")
    U = []
    for mu in range(4):
        u = torch.zeros(V, 4, dtype=torch.float64, device="cuda:0")
        u[:, 0] = 1.0
        if hot:
            r = [_u01(x) for x in _philox(site, 0, mu | (2 << 2) | (replica << 6), 0, seed)]
            a, b = (-2 * r[0].log()).sqrt(), (-2 * r[2].log()).sqrt()
            u = torch.stack([a * torch.cos(2 * math.pi * r[1]), a * torch.sin(2 * math.pi * r[1]),
                             b * torch.cos(2 * math.pi * r[3]), b * torch.sin(2 * math.pi * r[3])], -1)
            u = u / u.norm(dim=-1, keepdim=True)
        U.append(u.view(*dims[::-1], 4))
    return U


def _staples(U, mu, mul, dag):
    out = 0
    for nu in range(4):
        if nu != mu:
            n = U[nu]
            f = mul(mul(_up(n, mu), dag(_up(U[mu], nu))), dag(n))
            b = mul(dag(mul(U[mu], _up(n, mu))), n)
            out = out + f + _up(b, nu, -1)
    return out


def _plaquette2(U):
    s = sum((_mul(U[m], _up(U[n], m)) * _mul(U[n], _up(U[m], n))).sum()
            for m in range(4) for n in range(m + 1, 4))
    return s / (6 * U[0][..., 0].numel())


def _polyakov2(U):
    P = U[3][0]
    for t in range(1, U[3].shape[0]):
        P = _mul(P, U[3][t])
    return P[..., 0].mean()


def _chain2(dims, beta, seed, hot, sweeps, reunit, n_or=0, replica=0, poly=True):
    """(links, history) after `sweeps` sweeps in 64 bits."""
    U = _start2(dims, hot, seed, replica)
    par = _parity(dims).view(dims[::-1])
    sites = torch.arange(par.numel(), device=par.device).view(par.shape)
    rows = []
    for j in range(sweeps):
        for step in range(1 + n_or):
            for mu in range(4):
                for p in (0, 1):
                    at = par == p
                    V = _staples(U, mu, _mul, _dag)[at]
                    new = U[mu].clone()
                    if step == 0:
                        new[at] = _heatbath(V, beta, sites[at], j, mu | (replica << 6), seed)
                    else:
                        v = _dag(V / V.norm(dim=-1, keepdim=True))
                        new[at] = _mul(_mul(v, _dag(U[mu][at])), v)
                    U[mu] = new
        if reunit and (j + 1) % reunit == 0:
            U = [u / u.norm(dim=-1, keepdim=True) for u in U]
        L = _polyakov2(U) if poly else torch.zeros((), dtype=torch.float64, device="cuda:0")
        rows.append(torch.stack([_plaquette2(U), L, L.abs()]))
    return U, torch.stack(rows)


def _mul3(a, b):
    return sum(a[..., :, k, None] * b[..., k, None, :] for k in range(3))


def _dag3(a):
    return a.conj().transpose(-1, -2)


def _chain3(dims, beta, seed, hot, sweeps, replica=0):
    """(plaquettes, Polyakov loop) of an SU(3) chain in 64 bits (links there stay unitary)."""
    V = math.prod(dims)
    par = _parity(dims).view(dims[::-1])
    sites = torch.arange(V, device="cuda:0")
    U = []
    for mu in range(4):
        if hot:
            g = []
            for dr in range(3):
                r = [_u01(x) for x in _philox(sites, 0, mu | (10 << 2) | (replica << 6), dr, seed)]
                for i in (0, 2):
                    m = (-2 * r[i].log()).sqrt()
                    g.append(torch.polar(m, 2 * math.pi * r[i + 1]))
            a, b = torch.stack(g[:3], -1), torch.stack(g[3:], -1)
            a = a / a.norm(dim=-1, keepdim=True)
            b = b - (a.conj() * b).sum(-1, keepdim=True) * a
            b = b / b.norm(dim=-1, keepdim=True)
            u = torch.stack([a, b, torch.linalg.cross(a, b).conj()], -2)
        else:
            u = torch.eye(3, dtype=torch.complex128, device="cuda:0").expand(V, 3, 3).clone()
        U.append(u.view(*dims[::-1], 3, 3))
    sites, rows = sites.view(par.shape), []
    for j in range(sweeps):
        for mu in range(4):
            for p in (0, 1):
                at = par == p
                A, u, site = _staples(U, mu, _mul3, _dag3)[at], U[mu][at], sites[at]
                for g, (a, b) in enumerate(((0, 1), (1, 2), (0, 2))):
                    W = _mul3(u, A)
                    x = 0.5 * torch.stack([(W[:, a, a] + W[:, b, b]).real,
                                           (W[:, a, b] + W[:, b, a]).imag,
                                           (W[:, a, b] - W[:, b, a]).real,
                                           (W[:, a, a] - W[:, b, b]).imag], -1)
                    r = _heatbath(x, 2 * beta / 3, site, j, mu | ((7 + g) << 2) | (replica << 6), seed)
                    c00, c01 = torch.complex(r[:, 0], r[:, 3]), torch.complex(r[:, 2], r[:, 1])
                    ua = c00[:, None] * u[:, a] + c01[:, None] * u[:, b]
                    ub = -c01.conj()[:, None] * u[:, a] + c00.conj()[:, None] * u[:, b]
                    u = u.clone()
                    u[:, a], u[:, b] = ua, ub
                new = U[mu].clone()
                new[at] = u
                U[mu] = new
        s = sum((_mul3(U[m], _up(U[n], m)) * _mul3(U[n], _up(U[m], n)).conj()).sum().real
                for m in range(4) for n in range(m + 1, 4))
        rows.append(float(s) / (18 * V))
    P = U[3][0]
    for t in range(1, dims[3]):
        P = _mul3(P, U[3][t])
    L = torch.diagonal(P, dim1=-2, dim2=-1).sum(-1) / 3
    return rows, (float(L.real.mean()), float(L.imag.mean()), float(L.abs().mean()))


def _nll(p, f, a0):
    """Mean negative log-likelihood of a0 under the spline of the network, 64 bits."""
    h = torch.tanh(f[:, None] * p[0:32] + p[32:64])
    h = torch.tanh(h @ p[64:1088].view(32, 32).T + p[1088:1120])
    o = h @ p[1120:2624].view(47, 32).T + p[2624:]
    W, H = (2 * (1e-3 + (1 - 16e-3) * torch.softmax(x, -1)) for x in (o[:, :16], o[:, 16:32]))
    one = torch.ones_like(f)[:, None]
    d = torch.cat([one, 1e-3 + torch.nn.functional.softplus(o[:, 32:]), one], -1)
    X = torch.cat([-one, -1 + torch.cumsum(W, -1)], -1)
    k = (a0[:, None] >= X[:, 1:16].detach()).sum(-1, keepdim=True)
    w, hh, x, dl, dh = (v.gather(1, i)[:, 0] for v, i in ((W, k), (H, k), (X, k), (d, k), (d, k + 1)))
    s, xi = hh / w, (a0 - x) / w
    om = xi * (1 - xi)
    num = dh * xi * xi + 2 * s * om + dl * (1 - xi) ** 2
    return -(math.log(0.5) + 2 * s.log() + num.log() - 2 * (s + (dh + dl - 2 * s) * om).log()).mean()


def _train_exact(c, seed):
    alpha, a0 = (torch.from_numpy(v).double().cuda() for v in _samples(c, seed))
    f = 2 * torch.log2(alpha / 0.5) / math.log2(60.0) - 1
    p = torch.from_numpy(_start_params(seed)).double().cuda().requires_grad_()
    m, v, at, loss = torch.zeros_like(p), torch.zeros_like(p), 0, []
    for t in range(c["steps"]):
        i = (at + torch.arange(c["batch"], device="cuda:0")) % c["samples"]
        at = (at + c["batch"]) % c["samples"]
        L = _nll(p, f[i], a0[i])
        g, = torch.autograd.grad(L, p)
        loss.append(float(L))
        lr = 1e-5 + 0.5 * (c["lr"] - 1e-5) * (1 + math.cos(math.pi * t / c["steps"]))
        with torch.no_grad():
            m, v = 0.9 * m + 0.1 * g, 0.999 * v + 0.001 * g * g
            p -= lr * (m / (1 - 0.9 ** (t + 1))) / ((v / (1 - 0.999 ** (t + 1))).sqrt() + 1e-8)
    return {"loss": np.array(loss), "params": p.detach().cpu().numpy()}


def _wilson_exact(U, size):
    def line(mu, n):
        P = U[mu]
        for k in range(1, n):
            P = _mul(P, _up(U[mu], mu, k))
        return P
    lines = [[line(mu, n + 1) for n in range(size)] for mu in range(4)]
    out = torch.zeros(size, size, dtype=torch.float64, device="cuda:0")
    for mu in range(4):
        for nu in range(4):
            if mu != nu:
                for r in range(size):
                    for t in range(size):
                        a = _mul(lines[mu][r], _up(lines[nu][t], mu, r + 1))
                        b = _mul(lines[nu][t], _up(lines[mu][r], nu, t + 1))
                        out[r, t] += (a * b).sum()
    return (out / (12 * U[0][..., 0].numel())).cpu().numpy()


def exact(case, seed):
    c, k = case, case["kind"]
    # A decision taken within FP32 rounding of its threshold sends a chain another way, and the
    # difference spreads: beyond a few sweeps a long chain in 64 bits is another chain, and a
    # lattice of FP32 links says nothing about it; an over-relaxation step keeps the old link's
    # rounding and adds twice the staples', so there it takes one sweep.  (The trained proposal's Metropolis chain is
    # left out for its accept test, which has a wide band of such decisions.)
    if k == "f64":
        U, h = _chain2(_dims(c), c["beta"], seed, c["hot"], c["sweeps"], c["reunit"])
        return {"links": _to_classes(U, _dims(c)).view(8, -1, 2, 2).transpose(1, 2).contiguous(),
                "history": h}
    if k in ("lattice", "overrelax") and c["sweeps"] * (1 + 4 * c.get("n_or", 0)) <= 5:
        U, h = _chain2(_dims(c), c["beta"], seed, c["hot"], c["sweeps"], c["reunit"],
                       c.get("n_or", 0))
        return {"links": _to_classes(U, _dims(c)), "history": h}
    if k == "scan" and c["sweeps"] <= 5 and sum(math.prod(d) for d in _replicas(c)[0]) < 1 << 23:
        h = [_chain2(d, b, seed, st == su2.SU2_HOT, c["sweeps"], c["reunit"], 0, r, c["poly"])[1]
             for r, (d, b, st) in enumerate(zip(*_replicas(c)))]
        return {"history": torch.stack(h, 1)}
    if k == "su3" and math.prod(_dims(c)) < 1 << 20:
        h, L = _chain3(_dims(c), c["beta"], seed, c["hot"], c["sweeps"])
        return {"plaquettes": np.array(h), "polyakov": L}
    if k == "su3_scan" and c["n"] * math.prod(_dims(c)) < 1 << 21:
        got = [_chain3(_dims(c), b, seed, c["hot"], c["sweeps"], r)
               for r, b in enumerate(_couplings(c))]
        return {"plaquettes": np.array([g[0] for g in got]).T.copy(),
                "polyakov": np.array([g[1] for g in got])}
    if k == "train":
        return _train_exact(c, seed)
    if k in ("measure", "exchange"):
        f = _near_unit(_dims(c), seed, 0.3)
        if k == "exchange":
            V = math.prod(_dims(c))
            return {"saved": f.permute(1, 2, 3, 4, 0, 5).reshape(V, 4, 4).double().cpu().numpy(),
                    "loaded": _to_classes(f, _dims(c)).double()}
        U = list(f.double())
        L = float(_polyakov2(U))
        return {"wilson": _wilson_exact(U, c["size"]), "plaquette": float(_plaquette2(U)),
                "polyakov": (L, abs(L))}
    return None
