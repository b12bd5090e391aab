"""Measured cases of the drag framework: what a program that uses it has it do.

A case is one pass through the public entry points of paper_1312_3691_amd:
the no-allocation call, the plain path (seed -> trace -> forces), the batched
path (one-shot, or a resident batch replayed from its graph), the
continuous-batching server, and the build of a new body followed by its first
drag query.  `prepare` makes what such a program holds before the call (a mesh
on the device, queries, a batch or server handle), `run` is the call, `work`
what it cannot do without, and `exact` the same particles followed in 64 bits
with plain torch (small cases only).

Every result field of the library is returned except `preculled`, which counts
work done (how many particles the seeding estimate removed), differs between
paths by design and is not an answer.
"""
import asyncio
import math

import numpy as np
import torch

from paper_1312_3691_amd import inputs as I
from paper_1312_3691_amd import serve, tpmc

T_INF, T_W = 1000.0, 300.0
FIELDS = ("F_over_q", "M_over_q", "Fhat", "CD", "CD_sigma", "Gamma_hat", "rays", "hits", "segments", "missed",
          "escaped", "capped", "Qhat", "CH", "CH_sigma", "Mhat", "tr_capped", "guard_trips")
X_REF = (0.3, -0.2, 0.1)  # the point moments are taken about (a centre of mass off the body's centre), m
EXACT_PAIRS = 3e10  # ray-triangle pairs that `exact` tests at most (a few seconds on the GPU)


def _case(name, path, body, tris, n, nq=1, S=0.0, alpha=1.0, totals=False, box=False, alpha_E=1.0, energy=False,
          builder="sah"):
    """S = 0 draws each query's speed ratio from U[2, 10]."""
    return dict(name=name, path=path, body=body, tris=tris, n=n, nq=nq, S=float(S), alpha=float(alpha),
                totals=totals, box=box, energy=energy, alpha_E=float(alpha_E), builder=builder)


def listed():
    return [
        # The smallest call: one interactive question about a plate, answered
        # without allocation; latency and launches are all there is.
        _case("plate_noalloc_1k", "noalloc", "plate", 2, 1_000, S=5.0),
        # The sphere of the paper's verification at 1e5 particles, from a tight
        # loop (an optimiser, a trajectory code) that must not allocate.
        _case("sphere_noalloc_100k", "noalloc", "sphere", 1280, 100_000, S=5.0),
        # The same question through the plain path, with what it alone gives:
        # seeded states, first-hit triangles and per-triangle loads.
        _case("sphere_plain_100k", "plain", "sphere", 1280, 100_003, S=5.0),
        # A verification run of the paper's kind and size class on the plain path.
        _case("cylinder_plain_3M", "plain", "cylinder", 256, 3_000_001, S=3.0),
        # The plate's verification sweep (angles x S x accommodation): a resident
        # batch replayed from its graph.
        _case("plate_sweep_60x1M", "graph", "plate", 2, 1_000_000, nq=60),
        # The capped cylinder's sweep, one shot: new queries, so the batch is
        # made, launched and read.
        _case("cylinder_sweep_60x1M", "batch", "cylinder", 256, 1_000_000, nq=60),
        # Multiple reflections in a cup with a rectangular control volume and
        # incomplete energy accommodation.
        _case("cup_box_energy_3x300k", "batch", "cup", 3008, 300_001, nq=3, S=6.0, alpha=0.9, box=True, energy=True,
              alpha_E=0.6),
        # One drag query on the concave 50k-triangle satellite, per-triangle loads.
        _case("satellite_10M", "graph", "satellite", 50_000, 10_000_000, S=7.0, alpha=0.9),
        # A quick attitude scan: many small queries, totals only, one shot.
        _case("attitudes_200x50k", "batch", "satellite", 20_000, 50_001, nq=200, alpha=0.9, totals=True),
        # The attitude database: 1024 attitudes at 1e6 particles each (the largest).
        _case("attitudes_1024x1M", "graph", "satellite", 50_000, 1_000_000, nq=1024, alpha=0.9, totals=True),
        # A burst of mixed requests (four bodies, 1e5 to 1e6 particles) at the server.
        _case("served_24", "serve", "satellite", 100_000, 1_000_000, nq=24, alpha=0.9),
        # A new body: its hierarchy is built and its first query answered.
        _case("new_body_50k", "build", "satellite", 50_000, 100_000, S=7.0, alpha=0.9),
    ]


def _log_uniform(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def draw(rng):
    path = rng.choice(["noalloc", "plain", "batch", "graph", "serve", "build"])
    body = rng.choice(["plate", "cylinder", "sphere", "cup", "satellite", "satellite"])
    tris = {"plate": 2, "cylinder": 4 * rng.randint(8, 128), "sphere": 20 * 4 ** rng.randint(1, 4),
            "cup": int(_log_uniform(rng, 300, 6000)), "satellite": int(_log_uniform(rng, 1_000, 100_000))}[body]
    nq, totals = 1, False
    if path == "noalloc":
        tris = min(tris, 50_000)
        n, nq = int(_log_uniform(rng, 1_000, 1_000_000)), rng.choice([1, 1, 1, 3])
    elif path == "plain":
        n, nq = int(_log_uniform(rng, 1_000, 3_000_000)), rng.choice([1, 1, 2, 5])
    elif path in ("batch", "graph"):
        nq = int(_log_uniform(rng, 1, 300))
        n = int(_log_uniform(rng, 10_000, min(1e7, 2e8 / nq)))
        totals = rng.random() < 0.5 or nq * tris > 2_000_000
    elif path == "serve":
        body, tris = "satellite", int(_log_uniform(rng, 20_000, 100_000))
        n, nq = int(_log_uniform(rng, 200_000, 3_000_000)), rng.randint(4, 31)
    else:
        body, tris = "satellite", int(_log_uniform(rng, 1_000, 500_000))
        n = int(_log_uniform(rng, 10_000, 300_000))
    c = _case("", path, body, tris, n, nq, S=_log_uniform(rng, 0.3, 12.0), alpha=rng.choice([0.0, 1.0, 0.9, 0.9]),
              totals=totals, box=rng.random() < 0.2, energy=rng.random() < 0.25,
              alpha_E=round(rng.uniform(0.1, 1.0), 3), builder=rng.choice(["sah", "sah", "lbvh"]))
    del c["name"]
    return c


# --------------------------------------------------------------------------- inputs
def _body(kind, tris, seed):
    if kind == "plate":
        return I.plate(1.0)
    if kind == "cylinder":
        return I.capped_cylinder(segments=max(3, tris // 4))
    if kind == "sphere":
        return I.icosphere(int(round(math.log(tris / 20.0, 4))))
    if kind == "cup":
        k = max(4, int(round(math.sqrt(tris / 5.3))))
        return I.hemisphere_cup(n_theta=k, n_phi=int(2.67 * k))
    return I.satellite(tris, seed=seed)


def _queries(case, seed, n=None):
    nq = case["nq"]
    rng = np.random.default_rng([seed, 77])
    quats = I.random_quats(nq, seed=int(rng.integers(1 << 30)))
    out = []
    for i in range(nq):
        S = case["S"] if case["S"] > 0 else float(rng.uniform(2.0, 10.0))
        out.append(I.query(q=quats[i], S=S, T_inf=T_INF, T_w=T_W, alpha=case["alpha"],
                           n=case["n"] if n is None else n[i], seed=int(rng.integers(1 << 40)), max_reflections=16,
                           flags=tpmc.Q_NO_TRIANGLE_TALLY if case["totals"] else 0, cv_box=case["box"],
                           alpha_E=case["alpha_E"] if case["energy"] else None))
    return out


SERVE_SLOTS = 32
SERVE_TILES = 1024  # tiles per step (16384 particles each)


def _serve_bodies(case, seed):
    top = case["tris"]
    return {"b%d" % i: I.satellite(t, seed=seed + i) for i, t in enumerate((1_000, 20_000, max(1_000, top // 3), top))}


def _serve_requests(case, seed):
    """(mesh name, query) of each request: sizes log-uniform over a decade."""
    rng = np.random.default_rng([seed, 78])
    n = [int(v) for v in np.exp(rng.uniform(math.log(case["n"] / 10), math.log(case["n"]), case["nq"]))]
    return list(zip(["b%d" % k for k in rng.integers(0, 4, case["nq"])], _queries(case, seed, n)))


def prepare(case, seed):
    ctx = tpmc.Context(0)
    s = {"case": case, "ctx": ctx}
    if case["path"] == "serve":
        s["meshes"] = {k: ctx.build_mesh(*b, builder=case["builder"]) for k, b in _serve_bodies(case, seed).items()}
        s["requests"] = _serve_requests(case, seed)
        words = 7 * sum(m.nt for m in s["meshes"].values()) * SERVE_SLOTS
        s["executor"] = serve.GpuExecutor(ctx, s["meshes"], SERVE_SLOTS, words, x_ref=X_REF)
        s["loop"] = asyncio.new_event_loop()
        return s
    V, T = _body(case["body"], case["tris"], seed)
    s["queries"] = _queries(case, seed)
    if case["path"] == "build":
        s["V"], s["T"] = V, T
        return s
    s["mesh"] = ctx.build_mesh(V, T, builder=case["builder"])
    if case["path"] == "graph":
        s["batch"] = tpmc.Batch(s["mesh"], s["queries"])
    return s


# --------------------------------------------------------------------------- the call
def _stack(results):
    return {f: np.array([r[f] for r in results]) for f in FIELDS}


async def _serve(s):
    words = s["executor"].server.max_slots * 7 * sum(m.nt for m in s["meshes"].values())
    sched = serve.Scheduler(s["executor"], SERVE_SLOTS, words, SERVE_TILES)
    futures = [sched.submit(mesh, q) for mesh, q in s["requests"]]
    while sched.step_once():
        await asyncio.sleep(0)
    return [f.result() for f in futures]


def run(s):
    case = s["case"]
    path = case["path"]
    if path == "noalloc":
        return _stack(tpmc.batch_run_noalloc(s["mesh"], s["queries"], x_ref=X_REF))
    if path == "batch":
        b = tpmc.Batch(s["mesh"], s["queries"])
        out = b.launch().results(x_ref=X_REF)
        b.close()
        return _stack(out)
    if path == "graph":
        return _stack(s["batch"].launch(use_graph=True).results(x_ref=X_REF))
    if path == "serve":
        return _stack(s["loop"].run_until_complete(_serve(s)))
    if path == "build":
        mesh = s["ctx"].build_mesh(s["V"], s["T"], builder=case["builder"])
        out = _stack(tpmc.batch_run_noalloc(mesh, s["queries"], x_ref=X_REF))
        info = mesh.info
        mesh.close()
        out["body"] = np.array(info["box_lo"] + info["box_hi"] + info["sphere_center"] + [info["sphere_radius"]])
        out["hierarchy"] = np.array([info["nv"], info["nt"], info["depth"], info["stack_slots"],
                                     info["device_bytes"]])
        return out
    pr = tpmc.PlainRun(s["mesh"], s["queries"], first_tri=True).seed().trace()
    out = _stack(pr.forces(x_ref=X_REF))
    out["tally"] = np.stack([pr.tally(i) for i in range(case["nq"])])
    out["state"] = pr.planes()
    out["first_tri"] = pr.first_tri
    pr.close()
    return out


# --------------------------------------------------------------------------- what it cannot do without
# Operations per particle seeded: two Philox blocks (20 rounds of two products
# and a few additions), the two inverse distributions, the frame.  A particle
# that meets the body walks about log2(triangles) nodes of two boxes, tests a
# triangle and re-emits; about one in five does.
OPS_SEED, OPS_NODE, OPS_HIT, HIT_SHARE = 400.0, 24.0, 250.0, 0.2


def _triangles(case):
    if case["path"] != "serve":
        return case["tris"]
    return (21_000 + case["tris"] // 3 + case["tris"]) / 4.0


def work(case):
    nt, nq = _triangles(case), case["nq"]
    n = case["n"] * nq * (0.39 if case["path"] == "serve" else 1.0)  # mean of a log-uniform decade
    depth = max(1.0, math.log2(nt))
    flops = n * (OPS_SEED + HIT_SHARE * (depth * OPS_NODE + OPS_HIT))
    bodies = 4 if case["path"] == "serve" else 1
    nbytes = bodies * nt * (64 + 48 + 4) + nq * 272
    if not case["totals"]:
        nbytes += nq * nt * 56
    if case["path"] == "plain":
        nbytes += n * (24 + 4)
    if case["path"] == "build":
        nbytes += nt * (12 + 6) + nt * (64 + 48 + 4)
        flops += nt * depth * 30
    return {"bytes": float(nbytes), "flops": float(flops)}


# --------------------------------------------------------------------------- the same in 64 bits
SQRT_PI = math.sqrt(math.pi)


def _philox(c, k):
    """Philox4x32-10 on int64 tensors holding 32-bit words: counter c (4), key k (2)."""
    M = 0xFFFFFFFF
    c = list(c)
    for _ in range(10):
        hi, lo = [], []
        for mul, x in ((0xD2511F53, c[0]), (0xCD9E8D57, c[2])):  # 32 x 32 -> 64 bits in halves
            a, b = (x >> 16) * mul, (x & 0xFFFF) * mul
            s = a + (b >> 16)
            hi.append(s >> 16)
            lo.append(((s & 0xFFFF) << 16) | (b & 0xFFFF))
        c = [hi[1] ^ c[1] ^ k[0], lo[1], hi[0] ^ c[3] ^ k[1], lo[0]]
        k = ((k[0] + 0x9E3779B9) & M, (k[1] + 0xBB67AE85) & M)
    return c


def _stream(q, pid, step):
    zero = torch.zeros_like(pid)
    return _philox((pid & 0xFFFFFFFF, pid >> 32, zero + step, zero), (q["seed"] & 0xFFFFFFFF, q["seed"] >> 32))


def _u64(k):
    return (k.double() + 0.5) * 2.0 ** -32


def _u23(k):
    return ((k >> 9).double() + 0.5) * 2.0 ** -23


def _solve(f, lo, hi):
    for _ in range(64):
        m = 0.5 * (lo + hi)
        below = f(m) < 0
        lo, hi = torch.where(below, m, lo), torch.where(below, hi, m)
    return 0.5 * (lo + hi)


def _chi(s):
    return torch.exp(-s * s) + SQRT_PI * s * torch.special.erfc(-s)


def _normal_speed(s, u):
    """Inward normal speed x >= 0 of density 2 x exp(-(x - s)^2) / chi(s)."""
    es, es2 = torch.special.erfc(-s), torch.exp(-s * s)
    target = u * _chi(s)

    def f(x):  # the CDF's numerator minus the target, written so that nothing cancels for s < 0
        return es2 - torch.exp(-(x - s) ** 2) + SQRT_PI * s * (es - torch.special.erfc(x - s)) - target

    return _solve(f, torch.zeros_like(s), s.clamp(min=0.0) + 7.5)


def _seed64(q, V, pid, dev):
    """Positions and velocities [N, 3] of the particles pid, and Gamma_hat, centre."""
    w, x, y, z = q["q"]
    R = np.array([[1 - 2 * (y * y + z * z), 2 * (x * y - w * z), 2 * (x * z + w * y)],
                  [2 * (x * y + w * z), 1 - 2 * (x * x + z * z), 2 * (y * z - w * x)],
                  [2 * (x * z - w * y), 2 * (y * z + w * x), 1 - 2 * (x * x + y * y)]])
    U, e1, e2 = (torch.tensor(R[k], device=dev) for k in range(3))
    S = q["S"]
    lo, hi = V.min(0), V.max(0)
    c0n = 0.5 * (lo + hi)
    c0 = torch.tensor(c0n, device=dev)
    r0, r1 = _stream(q, pid, 0), _stream(q, pid, 1)
    if q["flags"] & I.BOX_CV:
        h = 0.5 * (hi - lo)
        h = h + 1e-3 * math.sqrt(float((h * h).sum()))
        s_f = np.array([S * R[0][f // 2] * (1.0 if f % 2 == 0 else -1.0) for f in range(6)])
        share = [4.0 * h[(f // 2 + 1) % 3] * h[(f // 2 + 2) % 3]
                 * (math.exp(-s * s) + SQRT_PI * s * math.erfc(-s)) for f, s in enumerate(s_f)]
        cum = torch.tensor(np.cumsum(share), device=dev)
        gamma = float(cum[-1]) / (2.0 * SQRT_PI)
        f = torch.bucketize(_u64(r0[0]) * cum[-1], cum[:5], right=True)
        axis = f // 2
        nsign = 1.0 - 2.0 * (f % 2).double()
        wn = _normal_speed(torch.tensor(s_f, device=dev)[f], _u64(r0[2]))
        j = (axis + 1) % 3
        p1, p2 = 2.0 * _u64(r0[1]) - 1.0, 2.0 * _u64(r1[1]) - 1.0
    else:
        r = float(np.sqrt(((V - c0n) ** 2).sum(1)).max()) * (1.0 + 1e-3)
        Z = math.exp(-S * S) + SQRT_PI * (S + 0.5 / S) * math.erf(S)
        gamma = SQRT_PI * r * r * Z
        u = _u64(r0[0]) * Z

        def G(t):
            st = S * t
            c = torch.special.erfc(-st)
            E = torch.where(st < -1.0, c - math.erfc(S), torch.special.erf(st) + math.erf(S))
            return (SQRT_PI / (4.0 * S) * E + 0.5 * SQRT_PI * S * (t * t * c - math.erfc(S))
                    + 0.5 * (t * torch.exp(-st * st) + math.exp(-S * S)) - u)

        mu = _solve(G, torch.full_like(u, -1.0), torch.full_like(u, 1.0))
        cphi = torch.sqrt((1.0 - mu * mu).clamp(min=0.0))
        th = 2.0 * math.pi * _u64(r0[1])
        wn = _normal_speed(S * mu, _u64(r0[2]))
    rad = torch.sqrt(-2.0 * torch.log(_u64(r0[3]))) / math.sqrt(2.0)
    b = 2.0 * math.pi * _u64(r1[0])
    g1, g2 = rad * torch.cos(b), rad * torch.sin(b)
    if q["flags"] & I.BOX_CV:
        pos, vel = [], []
        for i in range(3):
            on, first = axis == i, j == i
            pos.append(torch.where(on, c0[i] - nsign * h[i], c0[i] + torch.where(first, p1, p2) * h[i]))
            vel.append(torch.where(on, wn * nsign, S * U[i] + torch.where(first, g1, g2)))
        return torch.stack(pos, 1), torch.stack(vel, 1), gamma, c0
    c = torch.cos(th)[:, None] * e1 + torch.sin(th)[:, None] * e2
    d = -torch.sin(th)[:, None] * e1 + torch.cos(th)[:, None] * e2
    mu, cphi = mu[:, None], cphi[:, None]
    n = mu * U - cphi * c
    t1 = cphi * U + mu * c
    return c0 - r * n, wn[:, None] * n + (S * cphi + g1[:, None]) * t1 - g2[:, None] * d, gamma, c0


def _closest(o, d, prev, v0, ea, eb, lo, hi):
    """Nearest two-sided hit of rays (o, d) other than triangle prev: (index or -1, t)."""
    best = torch.full((len(o),), -1, dtype=torch.int64, device=o.device)
    t_best = torch.full((len(o),), math.inf, dtype=torch.float64, device=o.device)
    inv = 1.0 / d
    a, b = (lo - o) * inv, (hi - o) * inv
    may = torch.nonzero(torch.minimum(a, b).amax(1).clamp(min=0.0) <= torch.maximum(a, b).amin(1) + 1e-9).flatten()
    nrm = torch.linalg.cross(ea, eb)
    step = max(1, int(2 ** 25 // len(v0)))
    for i in range(0, len(may), step):
        r = may[i:i + step]
        D, O = d[r], o[r]
        # scalar triple products by matrix products: (O - v0).n, D.n, D x O . e
        dn = D @ nrm.T
        t = ((v0 * nrm).sum(1) - O @ nrm.T) / dn
        m = torch.linalg.cross(D, O)
        u = (m @ eb.T + D @ torch.linalg.cross(eb, v0).T) / dn
        v = -(m @ ea.T + D @ torch.linalg.cross(ea, v0).T) / dn
        hit = (u >= 0) & (v >= 0) & (u + v <= 1) & (t > 0)
        ok = prev[r] >= 0
        hit[torch.nonzero(ok).flatten(), prev[r][ok]] = False
        t = torch.where(hit, t, math.inf)
        tm, k = t.min(1)
        t_best[r] = tm
        best[r] = torch.where(torch.isfinite(tm), k, -1)
    return best, t_best


def _follow64(q, V, T, dev):
    """One query followed in 64 bits: result fields, per-triangle sums, seeds."""
    V = V.astype(np.float64)
    nt = len(T)
    pid = torch.arange(q["n"], device=dev)
    x, w, gamma, c0 = _seed64(q, V, pid, dev)
    seeds = (x, w)
    P = torch.tensor(V[T.astype(np.int64)], device=dev)
    v0, ea, eb = P[:, 0], P[:, 1] - P[:, 0], P[:, 2] - P[:, 0]
    nrm = torch.linalg.cross(ea, eb)
    nrm = nrm / nrm.norm(dim=1, keepdim=True)
    lo, hi = (torch.tensor(f(0), device=dev) for f in (V.min, V.max))
    w_, x_, y_, z_ = q["q"]
    U = torch.tensor([1 - 2 * (y_ * y_ + z_ * z_), 2 * (x_ * y_ - w_ * z_), 2 * (x_ * z_ + w_ * y_)], device=dev,
                     dtype=torch.float64)
    tau = math.sqrt(q["T_w"] / q["T_inf"])
    N = q["n"]
    D, E = torch.zeros(N, dtype=torch.float64, device=dev), torch.zeros(N, dtype=torch.float64, device=dev)
    tal = torch.zeros(nt, 7, dtype=torch.float64, device=dev)
    live, prev = pid, torch.full_like(pid, -1)
    for bounce in range(q["max_reflections"]):
        k, t = _closest(x, w, prev, v0, ea, eb, lo, hi)
        on = k >= 0
        live, x, w, k, t = live[on], x[on], w[on], k[on], t[on]
        if len(live) == 0:
            break
        x = x + t[:, None] * w
        n = nrm[k]
        r = _stream(q, live, 2 + bounce)
        wn = (w * n).sum(1)
        spec = w - 2.0 * wn[:, None] * n
        e_in = (w * w).sum(1)
        tr = torch.full_like(wn, tau)
        if q["flags"] & I.ENERGY_ACC:
            tr = torch.sqrt(q["alpha_E"] * tau * tau + (1.0 - q["alpha_E"]) * 0.5 * e_in)
        s = torch.where(wn[:, None] < 0, n, -n)
        sign = torch.where(s[:, 2] >= 0, 1.0, -1.0).double()  # tangents: Duff et al., JCGT 2017
        a = -1.0 / (sign + s[:, 2])
        b = s[:, 0] * s[:, 1] * a
        b1 = torch.stack([1.0 + sign * s[:, 0] ** 2 * a, sign * b, -sign * s[:, 0]], 1)
        b2 = torch.stack([b, sign + s[:, 1] ** 2 * a, -s[:, 1]], 1)
        vn = tr * torch.sqrt(-torch.log(_u23(r[1])))
        rad = tr * torch.sqrt(-torch.log(_u23(r[2])))
        an = 2.0 * math.pi * _u23(r[3])
        diff = vn[:, None] * s + (rad * torch.cos(an))[:, None] * b1 + (rad * torch.sin(an))[:, None] * b2
        out = torch.where((_u23(r[0]) < float(np.float32(q["alpha"])))[:, None], diff, spec)
        dw = w - out
        D[live] += dw @ U
        E[live] += e_in - (out * out).sum(1)
        tal.index_add_(0, k, torch.cat([dw, torch.linalg.cross(x - c0, dw), torch.ones_like(wn)[:, None]], 1))
        w, prev = out, k
    F, L = tal[:, :3].sum(0), tal[:, 3:6].sum(0)
    M = L + torch.linalg.cross(c0 - torch.tensor(X_REF, dtype=torch.float64, device=dev), F)
    S = q["S"]
    K = 2.0 * gamma / (N * S * S)
    per = tal.clone()
    per[:, 3:6] += torch.linalg.cross(c0.expand(nt, 3), per[:, :3])
    mD, mE = float(D.mean()), float(E.mean())
    sD, sE = math.sqrt(max(0.0, float((D * D).mean()) - mD * mD) / N), math.sqrt(max(0.0, float((E * E).mean()) - mE * mE) / N)
    res = {"F_over_q": (K * F).cpu().numpy(), "M_over_q": (K * M).cpu().numpy(), "Fhat": (gamma / N * F).cpu().numpy(),
           "Mhat": (gamma / N * M).cpu().numpy(), "CD": float(K * (F @ U)), "CD_sigma": 2.0 * gamma / (S * S) * sD,
           "Gamma_hat": gamma, "Qhat": gamma * mE, "CH": gamma * mE / S ** 3, "CH_sigma": gamma / S ** 3 * sE}
    return res, per.cpu().numpy(), seeds


def exact(case, seed):
    """Whole-number outputs have no 64-bit value; None where the brute-force search would take too long."""
    if case["path"] == "serve" or case["n"] * case["nq"] * case["tris"] > EXACT_PAIRS:
        return None
    V, T = _body(case["body"], case["tris"], seed)
    dev = "cuda:0" if torch.cuda.is_available() else "cpu"
    got = [_follow64(q, V, T, dev) for q in _queries(case, seed)]
    out = {f: np.array([g[0][f] for g in got]) if f in got[0][0] else None for f in FIELDS}
    if case["alpha"] == 0.0:  # specular: no energy is exchanged, and what comes back is rounding alone
        out["Qhat"] = out["CH"] = out["CH_sigma"] = None
    if case["path"] == "build":
        X = V.astype(np.float64)
        c0 = 0.5 * (X.min(0) + X.max(0))
        r = float(np.sqrt(((X - c0) ** 2).sum(1)).max()) * (1.0 + 1e-3)
        out["body"], out["hierarchy"] = np.concatenate([X.min(0), X.max(0), c0, [r]]), None
    if case["path"] == "plain":
        out["tally"] = np.stack([g[1] for g in got])
        out["state"] = [torch.cat([g[2][k // 3][:, k % 3] for g in got]) for k in range(6)]
        out["first_tri"] = None
    return out
