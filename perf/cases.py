"""The calls that a program built on this library makes, as timed cases.

A case is one pass of one kind of use, through the package's public entry
points:

  scatter   one body in free space from its geometry: build the operator,
            factor it, and evaluate the scattered field of some incident waves
  evaluate  more incident waves and field points on an operator that the
            program keeps
  sum       the phased 3x3 neighbour sum of given point sources
  batch     many different bodies built and factored in one call, each with
            the field of one wave
  solve     the periodic solve of some incident waves on a kept operator, or
            from the geometry on (build = True)
  serve     a stream of incident waves through the continuous-batching server

Outputs are fields, amplitudes, singular values and ranks.  MFS coefficients
themselves are not among them: the systems' condition numbers reach the
truncation's 1e10, so their digits mean nothing, while the fields they give
are determined to about 1e-13.
"""
import math
import random

import numpy as np
import torch

import paper_1506_05083_amd as mfs

TWO_PI = 2 * math.pi


# ------------------------------------------------------------------- cases

def _body(shape="polar", a=0.3, eps=0.1, j=3, N=40, M=48, P=24, q=160, k=5.0, tau=0.2, colloc="mid", km=0.0):
    return dict(shape=shape, a=a, eps=eps, j=j, N=N, M=M, P=P, q=q, k=k, tau=tau, colloc=colloc, km=km)


def _lat(ex=1.0, ey=1.0, z0=0.6, p=24, N0=10.0, M1=20):
    return dict(ex=ex, ey=ey, z0=z0, p=p, N0=N0, M1=M1)


_SPHERE = _body(a=0.5, eps=0.0, j=0, N=40, M=60, P=32, q=128, k=TWO_PI, tau=math.log(1 / 0.7), colloc="gauss")
_K10 = _body(N=200, M=240, P=64, q=400, k=10.0, tau=0.1)
_K10_LAT = _lat(z0=0.8, p=30, N0=14.0, M1=24)


def listed():
    return [
        # a single small sphere, one wave, from its geometry: launches and latency
        dict(name="scatter_sphere", kind="scatter", waves=1, targets=64, q_field=128, **_SPHERE),
        # the penetrable sphere: the doubled systems, fields outside and inside
        dict(name="scatter_penetrable", kind="scatter", waves=1, targets=32, q_field=128,
             **dict(_SPHERE, km=1.5 * TWO_PI)),
        # a large single obstacle (the upper end of the batched build's sizes), several waves
        dict(name="scatter_large_body", kind="scatter", waves=5, targets=129, q_field=450,
             **_body(a=0.37, eps=0.12, j=4, N=551, M=662, P=128, q=450, k=28.0, tau=0.1)),
        # an incidence sweep on a kept operator
        dict(name="evaluate_sweep", kind="evaluate", waves=16, targets=1000, q_field=256, **_K10),
        # the neighbour sum on the surface nodes, as a program that iterates by itself calls it
        dict(name="sum_surface", kind="sum", set="surface", waves=3, points=0, **_K10, **_K10_LAT),
        # the smallest periodic solve, two waves
        dict(name="solve_small", kind="solve", build=False, waves=2, targets=20, q_field=64, tol=1e-12,
             **_body(), **_lat()),
        # a small penetrable obstacle in the lattice
        dict(name="solve_small_penetrable", kind="solve", build=False, waves=2, targets=20, q_field=64, tol=1e-12,
             **_body(km=7.5), **_lat()),
        # one wave on the k = 10 operator: the latency of a single answer
        dict(name="solve_k10_one", kind="solve", build=False, waves=1, targets=32, q_field=256, tol=1e-10,
             **_K10, **_K10_LAT),
        # the benchmark's step: the k = 10 body from its geometry, eight waves
        dict(name="solve_k10_step", kind="solve", build=True, waves=8, targets=32, q_field=256, tol=1e-10,
             **_K10, **_K10_LAT),
        # cups four wavelengths apart, two waves: the largest solve that is not minutes
        dict(name="solve_cup", kind="solve", build=False, waves=2, targets=17, q_field=480, tol=1e-10,
             **_body(shape="cup", a=0.35, eps=0.2, N=180, M=216, P=72, q=480, k=8 * math.pi, tau=0.07),
             **_lat(z0=0.55, p=46, N0=21.0, M1=32)),
        # a batch of different bodies
        dict(name="batch_16", kind="batch", count=16, sizes=3, targets=16),
        # the server with more requests than slots
        dict(name="serve_k10", kind="serve", waves=12, slots=8, targets=16, q_field=256, tol=1e-10,
             **_K10, **_K10_LAT),
    ]


def _smooth(x):
    """The smallest even 2^a 3^b 5^c that is at least x."""
    n = max(2, math.ceil(x))
    while True:
        r = n
        for f in (2, 3, 5):
            while r % f == 0:
                r //= f
        if n % 2 == 0 and r == 1:
            return n
        n += 1


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["scatter", "evaluate", "sum", "batch", "solve", "solve", "solve", "solve", "serve"])
    if kind == "batch":
        return dict(kind=kind, count=rng.randint(2, 14), sizes=rng.randint(10, 10000), targets=rng.randint(8, 40))
    periodic = kind in ("sum", "solve", "serve")
    N = _log(rng, 30, 200 if periodic else 500)
    P = 2 * rng.randint(8, 32 if periodic else 64)
    tau = rng.uniform(0.1, 0.2)
    km = 0.0
    k = rng.uniform(3.0, 10.0 if periodic else 24.0)
    if rng.random() < 0.2 and N <= 120 and kind != "sum":
        km = 1.5 * k
    b = _body(a=rng.uniform(0.2, 0.4), eps=rng.uniform(0.0, 0.1), j=rng.randint(2, 4), N=N, M=math.ceil(1.2 * N), P=P,
              q=_smooth(max(P, P / 2 + 37 / tau)), k=k, tau=tau, km=km)
    if periodic and rng.random() < 0.2:
        b.update(shape="cup", a=0.35, eps=0.2, tau=0.1, km=0.0, q=_smooth(P / 2 + 320))
    case = dict(kind=kind, waves=rng.randint(1, 8), targets=_log(rng, 10, 40 if periodic else 2000), q_field=b["q"], **b)
    if periodic:
        N0 = rng.randint(8, 13)
        case.update(_lat(ex=rng.choice([1.0, 1.0, 1.15]), ey=rng.choice([1.0, 1.0, 1.1]), z0=rng.uniform(0.6, 0.8),
                         p=rng.randint(16, 28), N0=float(N0), M1=2 * rng.randint(9, 12)), tol=10.0 ** -rng.randint(9, 11))
    if kind == "sum":
        case.pop("tol")
        case.update(set=rng.choice(["surface", "walls", "user"]), points=_log(rng, 50, 5000))
    if kind == "solve":
        case.update(build=rng.random() < 0.3)
    if kind == "serve":
        case.update(slots=rng.randint(2, 8), waves=rng.randint(2, 12), km=0.0)
    return case


# ------------------------------------------------------- inputs from a seed

def _rmax(c):
    return c["a"] if c["shape"] == "cup" else c["a"] * (1 + c["eps"])


def _geometry(c):
    if c["shape"] == "cup":
        return mfs.cup_geometry(c["a"], c["eps"], math.pi / 6, c["M"], c["N"], c["tau"], c["colloc"])
    g = mfs.polar_geometry(c["a"], c["eps"], c["j"], c["M"], c["N"], c["tau"], c["colloc"])
    if c["km"] > 0:
        o = mfs.polar_geometry(c["a"], c["eps"], c["j"], c["M"], c["N"], -c["tau"], c["colloc"])
        g["srho_out"], g["sz_out"] = o["srho"], o["sz"]
    return g


def _spec(c):
    return mfs.BodySpec(c["M"], c["N"], c["P"], c["q"], c["k"], _geometry(c), c["km"])


def _kvec(k, w):
    return k * np.array([math.sin(w[0]) * math.cos(w[1]), math.sin(w[0]) * math.sin(w[1]), -math.cos(w[0])])


def _incidences(c, rng):
    """Directions from above; on a lattice none whose Bragg orders come near grazing (a Wood anomaly)."""
    out = []
    while len(out) < c["waves"]:
        w = (rng.uniform(0.0, 1.4), rng.uniform(0.0, TWO_PI))
        if "ex" in c:
            kv, n = _kvec(c["k"], w), np.arange(-8, 9)
            kx, ky = kv[0] + TWO_PI * n[:, None] / c["ex"], kv[1] + TWO_PI * n[None, :] / c["ey"]
            if np.min(np.abs(c["k"] ** 2 - kx ** 2 - ky ** 2)) < (0.05 * c["k"]) ** 2:
                continue
        out.append(w)
    return out


def _points(c, seed, inside=False):
    """Field points: around the body in free space, or in the unit cell outside it."""
    g = np.random.default_rng(seed)
    r = _rmax(c)
    if inside or "ex" not in c:
        u = g.normal(size=(c["targets"], 3))
        lo, hi = (0.1 * r, 0.45 * r) if inside else (1.5 * r, 4.0)
        return u / np.linalg.norm(u, axis=1, keepdims=True) * g.uniform(lo, hi, (c["targets"], 1))
    pts = []
    while len(pts) < c["targets"]:
        x = g.uniform(-0.5, 0.5, 3) * (c["ex"], c["ey"], 1.8 * c["z0"])
        if np.linalg.norm(x) > r + 0.08 and math.hypot(x[0], x[1]) > 0.02:
            pts.append(x)
    return np.array(pts)


def _batch(case, seed):
    """The bodies of a batch: sizes by the case, shapes and wavenumbers by the seed."""
    sizes, g, out = random.Random(case["sizes"]), random.Random(seed), []
    for _ in range(case["count"]):
        N, P = sizes.randint(100, 600), sizes.choice([32, 64, 96, 128, 160])
        out.append(_body(a=g.uniform(0.2, 0.4), eps=g.uniform(0.0, 0.15), j=g.randint(2, 5), N=N, M=math.ceil(1.2 * N),
                         P=P, q=_smooth(max(P, P / 2 + 370)), k=g.uniform(5.0, 30.0), tau=0.1))
        out[-1].update(waves=1, targets=case["targets"])
    return out


def _sources(c, seed):
    """Point strengths and Bloch phases of a neighbour sum."""
    g = torch.Generator().manual_seed(seed)
    sig = torch.complex(*(torch.randn(c["waves"], c["P"], c["N"], generator=g, dtype=torch.float64) for _ in "ri"))
    kv = np.stack([_kvec(c["k"], w) for w in _incidences(c, random.Random(seed))])
    return sig, np.exp(1j * kv[:, :2] * np.array([c["ex"], c["ey"]]))


def _user_points(c, seed):
    g = np.random.default_rng(seed)
    d = g.normal(size=(c["points"], 3))
    return np.concatenate([_points(dict(c, targets=c["points"]), seed + 1), d / np.linalg.norm(d, axis=1)[:, None]], 1)


def prepare(case, seed):
    s = dict(case=case, ctx=mfs.create(0))
    kind = case["kind"]
    if kind == "batch":
        s["bodies"] = [(_spec(b), np.stack([_kvec(b["k"], w) for w in _incidences(b, random.Random(seed + i))]),
                        _points(b, seed + i)) for i, b in enumerate(_batch(case, seed))]
        return s
    s["spec"] = _spec(case)
    rng = random.Random(seed)
    if kind == "sum":
        sig, s["ab"] = _sources(case, seed)
        s["sigma"] = sig.cuda()
        s["user"] = _user_points(case, seed) if case["set"] == "user" else None
    else:
        s["waves"] = _incidences(case, rng)
        s["kvec"] = np.stack([_kvec(case["k"], w) for w in s["waves"]])
        s["points"] = _points(case, seed)
        s["inner"] = _points(case, seed, inside=True) if case["km"] > 0 else None
    if "ex" in case:
        s["lat"] = mfs.lattice(case["ex"], case["ey"], case["z0"], case["p"], case["N0"], case["M1"])
    if kind == "sum":
        s["op"] = mfs.build_operator(s["ctx"], [s["spec"]])
    elif kind != "scatter" and not case.get("build"):
        s["op"] = mfs.build_operator(s["ctx"], [s["spec"]])
        mfs.factor_modes(s["op"], 1e-10)
    if kind == "serve":
        s["server"] = mfs.Server(s["ctx"], s["op"], s["lat"], slots=case["slots"], admit_batch=case["slots"],
                                 tol=case["tol"], maxit=100, targets=s["points"], q_field=case["q_field"],
                                 hbm_budget=60 << 30)
    return s


# ---------------------------------------------------------------- one pass

def _field(op, body, kvec, points, q_field, inner=None):
    c = mfs.apply_solution_op(op, mfs.rhs_modes(op, kvec, body), body)
    out = mfs.field_free(op, c, q_field, points, body)
    return out if inner is None else (out, mfs.field_interior(op, c, q_field, inner, body))


def _on_orders(case, m, n, v):
    """Values of the Bragg orders (m, n) on a grid of orders that holds those of every direction."""
    reach = [math.ceil((math.pi * case["N0"] + case["k"]) * e / TWO_PI) for e in (case["ex"], case["ey"])]
    out = np.zeros((2 * reach[0] + 1, 2 * reach[1] + 1), complex)
    out[m + reach[0], n + reach[1]] = v
    return out


def _amplitudes(case, res):
    return dict(a=[_on_orders(case, r.m, r.n, r.a) for r in res], b=[_on_orders(case, r.m, r.n, r.b) for r in res],
                kz=np.stack([_on_orders(case, r.m, r.n, r.kz) for r in res]), field=[r.field for r in res])


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "batch":
        op = mfs.build_operator(s["ctx"], [b[0] for b in s["bodies"]])
        ranks = mfs.factor_modes(op, 1e-10)
        q = [b[0].q for b in s["bodies"]]
        return dict(ranks=ranks, sv=[op.singular_values(i) for i in range(len(q))],
                    field=[_field(op, i, b[1], b[2], q[i]) for i, b in enumerate(s["bodies"])])
    if kind == "sum":
        which = {"surface": mfs.TARGETS_SURFACE, "walls": mfs.TARGETS_WALLS, "user": mfs.TARGETS_USER}[case["set"]]
        return mfs.neighbour_sum(s["op"], s["lat"], s["sigma"], s["ab"], which, s["user"], want=1)
    if kind == "serve":
        tickets = [s["server"].submit(*w) for w in s["waves"]]
        return _amplitudes(case, [s["server"].wait(t)[0] for t in tickets])
    op = s.get("op")
    if op is None:
        op = mfs.build_operator(s["ctx"], [s["spec"]])
        ranks = mfs.factor_modes(op, 1e-10)
        if kind == "scatter":
            return dict(ranks=ranks, sv=op.singular_values(),
                        field=_field(op, 0, s["kvec"], s["points"], case["q_field"], s["inner"]))
    if kind == "evaluate":
        return _field(op, 0, s["kvec"], s["points"], case["q_field"], s["inner"])
    return _amplitudes(case, mfs.solve_incident(s["ctx"], op, s["lat"], s["waves"], tol=case["tol"], maxit=200,
                                                targets=s["points"], q_field=case["q_field"]))


# ------------------------------------------------------ what it has to do

def _mode_blocks(c):
    d = 2 if c["km"] > 0 else 1
    return c["P"] // 2 + 1, d * c["M"], d * c["N"]


def _build_work(c):
    """Fill (a kernel value is about 40 operations, a cosine term 4) and a QR of every distinct block; geometry in,
    singular values out."""
    nd, m, n = _mode_blocks(c)
    pairs = m * n * (c["q"] // 2 + 1)
    return 8 * (c["M"] * 4 + c["N"] * 2) + 8 * nd * n, pairs * (40 + 4 * nd) + nd * (8 * m * n * n - 8 * n ** 3 / 3)


def work(case):
    kind = case["kind"]
    if kind == "batch":
        w = [_build_work(b) for b in _batch(case, 0)]
        return {"bytes": sum(x[0] for x in w), "flops": sum(x[1] for x in w)}
    c, W, by, fl = case, case["waves"], 0.0, 0.0
    nd, m, n = _mode_blocks(c)
    if kind == "sum":
        nt, images = {"surface": (c["P"] * c["M"], 8), "walls": (8 * c["M1"] ** 2, 6), "user": (c["points"], 9)}[c["set"]]
        pairs = nt * images * c["P"] * c["N"]
        return {"bytes": 16 * W * (nt + c["P"] * c["N"]) + 48 * nt, "flops": pairs * (40 + 8 * W)}
    if kind == "scatter" or c.get("build"):
        by, fl = _build_work(c)
    else:
        by += 16 * nd * n * (m + n)   # the kept factors
    if kind in ("scatter", "evaluate"):
        by += 16 * W * c["targets"] + 24 * c["targets"]
        return {"bytes": by, "flops": fl + W * (8 * c["P"] * n * (m + n) + c["targets"] * c["q_field"] * c["N"] * 28)}
    # Per wave the periodizer's least squares: Q splits into two parts, even and odd in z.  An iteration cannot do
    # without the products with the solution operator and the periodizer's factors; 10 iterations stand for any number.
    mq = 4 * c["M1"] ** 2
    nq = ((c["p"] + 1) ** 2 + math.pi / 2 * c["N0"] ** 2 * c["ex"] * c["ey"]) / 2
    qr = 2 * (8 * mq * nq * nq - 8 * nq ** 3 / 3)
    it = 8 * c["P"] * n * (m + n) + 2 * 8 * nq * (mq + nq)
    return {"bytes": by + 16 * W * (4 * nq + c["targets"]), "flops": fl + W * (qr + 10 * it)}


# ---------------------------------------------- the same in 64 bits, plainly

def _cerf(x, y):
    """erf(x + i y): along the imaginary direction from the real erf, by Gauss quadrature."""
    x, y = np.broadcast_arrays(np.asarray(x, float), np.asarray(y, float))
    g, w = np.polynomial.legendre.leggauss(40)
    t = y[..., None] * (g + 1) / 2
    f = np.exp(t * t - x[..., None] ** 2 - 2j * x[..., None] * t)
    return np.vectorize(math.erf)(x) + 1j * y / math.sqrt(math.pi) * (f @ w)


def _curve(c, t, tau=0.0):
    """rho + i z and its t derivative at t - i tau."""
    t = np.asarray(t) - 1j * tau
    if c["shape"] == "cup":
        h, b = c["eps"], math.pi / 6
        x = math.pi / 2 - t
        s0 = 2 * (1 - (b - h) / math.pi)
        e, ex = _cerf(x.real / h, x.imag / h), np.exp(-(x / h) ** 2)
        r, th = 1 - h * e, b - h + s0 * (x * e + h / math.sqrt(math.pi) * ex)
        r_t, th_t, f = 2 / math.sqrt(math.pi) * ex, -s0 * e, c["a"] / (1 + h)
        return 1j * f * r * np.exp(-1j * th), 1j * f * (r_t - 1j * r * th_t) * np.exp(-1j * th)
    r, r_t = c["a"] * (1 + c["eps"] * np.cos(c["j"] * t)), -c["a"] * c["eps"] * c["j"] * np.sin(c["j"] * t)
    return 1j * r * np.exp(-1j * t), 1j * (r_t - 1j * r) * np.exp(-1j * t)


class _Exact:
    """One body by plain dense algebra."""

    def __init__(self, c):
        self.c = c
        M, N = c["M"], c["N"]
        t = math.pi * ((np.polynomial.legendre.leggauss(M)[0] + 1) / 2 if c["colloc"] == "gauss" else (np.arange(M) + 0.5) / M)
        z, dz = _curve(c, t)
        sp = np.abs(dz)
        self.surf = np.stack([z.real, z.imag, -dz.imag / sp, dz.real / sp], 1)
        ts = math.pi * (np.arange(N) + 0.5) / N
        self.src = [_curve(c, ts, s * c["tau"])[0] for s in ((1, -1) if c["km"] > 0 else (1,))]
        self.ks = [c["k"], c["km"]]

    def ring(self, rho, z, q):
        ph = TWO_PI * np.arange(q) / q
        return np.stack([np.outer(np.cos(ph), rho), np.outer(np.sin(ph), rho), np.tile(z, (q, 1))], -1)

    def points(self, which, q):
        return self.ring(self.src[which].real, self.src[which].imag, q).reshape(-1, 3)

    @staticmethod
    def kernel(k, x, n, y):
        """G and its derivative along n (or None), targets x [T, 3], sources y [S, 3], on the GPU."""
        d = x[:, None, :] - y[None, :, :]
        r2 = (d * d).sum(-1)
        r = r2.sqrt()
        g = torch.polar(1 / (4 * math.pi * r), k * r)
        if n is None:
            return g, None
        return g, g * torch.complex(-1 / r2, k / r) * (d * n[:, None, :]).sum(-1)

    def blocks(self):
        """The mode blocks n = 0..P/2, [nd][rows][cols]."""
        c = self.c
        x = np.zeros((c["M"], 3))
        nn = np.zeros((c["M"], 3))
        x[:, 0], x[:, 2], nn[:, 0], nn[:, 2] = self.surf.T
        out = []
        for w, s in enumerate(self.src):
            part = []
            for m0 in range(0, c["M"], 64):
                v, d = self.kernel(self.ks[w], _gpu(x[m0:m0 + 64]), _gpu(nn[m0:m0 + 64]), _gpu(self.points(w, c["q"])))
                rows = [v, d] if c["km"] > 0 else [d]
                part.append(torch.stack([torch.fft.fft(a.reshape(len(a), c["q"], -1), dim=1)[:, :c["P"] // 2 + 1] / c["q"]
                                         for a in rows]))
            col = torch.cat(part, 1).permute(2, 0, 1, 3)
            out.append((1 if w == 0 else -1) * col.reshape(col.shape[0], -1, col.shape[3]))
        return torch.cat(out, 2).cpu().numpy()

    def factor(self):
        A = self.blocks()
        u, s, vh = np.linalg.svd(A, full_matrices=False)
        keep = s > 1e-10 * s[:, :1]
        self.sv, self.ranks = s, keep.sum(1).astype(np.int32)
        sinv = np.where(keep, 1 / np.where(keep, s, 1), 0)
        nd, P = A.shape[0], self.c["P"]
        at = [b if b < nd else P - b for b in range(P)]
        self.uh = _gpu(np.conj(np.swapaxes(u, 1, 2)) * sinv[:, :, None])[at]
        self.v = _gpu(np.conj(np.swapaxes(vh, 1, 2)))[at]

    def pinv(self, x):   # [P, rows] -> [P, cols]
        return (self.v @ (self.uh @ x[:, :, None]))[:, :, 0]

    def modes(self, f):   # [.., P, M] angle samples -> [P, rows]
        f = torch.fft.fft(_gpu(f), dim=-2) / self.c["P"]
        return torch.cat(list(f), 1)

    def nodes(self):
        c = self.c
        X = self.ring(self.surf[:, 0], self.surf[:, 1], c["P"])
        return X, self.ring(self.surf[:, 2], self.surf[:, 3], c["P"])

    def rhs(self, kv):
        X, n = self.nodes()
        u = np.exp(1j * (X @ kv))
        d = -1j * (n @ kv) * u
        return self.modes(np.stack([-u, d] if self.c["km"] > 0 else [d]))

    def strengths(self, c, which, qs):   # [P, cols] -> [qs * N]
        P, N = self.c["P"], self.c["N"]
        full = torch.zeros(qs, N, dtype=torch.complex128, device="cuda")
        b = torch.arange(P, device="cuda")
        full[torch.where(b <= P // 2, b, b - P) % qs] = c[:, which * N:(which + 1) * N]
        return torch.fft.ifft(full, dim=0).reshape(-1)

    def field(self, c, x, which=0, shifts=((0.0, 0.0, 0.0, 1.0),), qs=None):
        y, sig = _gpu(self.points(which, qs)), self.strengths(c, which, qs)
        out = torch.zeros(len(x), dtype=torch.complex128, device="cuda")
        for sx, sy, sz, w in shifts:
            for t in range(0, len(x), 256):
                g = self.kernel(self.ks[which], _gpu(x[t:t + 256] - np.array([sx, sy, sz])), None, y)[0]
                out[t:t + 256] += w * (g @ sig)
        return out


def _gpu(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def _harmonics(k, p, x, n):
    """j_l(kr) Y_lm and its derivative along n at points x [T, 3], columns l^2 + l + m."""
    r = np.linalg.norm(x, axis=1)
    ct, rho = x[:, 2] / r, np.hypot(x[:, 0], x[:, 1])
    st, ph = rho / r, np.arctan2(x[:, 1], x[:, 0])
    L = p + 40 + int(k * r.max())
    j = np.zeros((L + 2, len(r)))
    j[L] = 1e-250
    for l in range(L, 0, -1):   # Miller's recurrence, rescaled on the way
        j[l - 1] = (2 * l + 1) / (k * r) * j[l] - j[l + 1]
        big = np.abs(j[l - 1]) > 1e200
        j[l - 1:, big] *= 1e-200
    s, co = np.sin(k * r), np.cos(k * r)
    j0, j1 = s / (k * r), s / (k * r) ** 2 - co / (k * r)
    j *= np.where(np.abs(j0) >= np.abs(j1), j0 / j[0], j1 / j[1])
    er = x / r[:, None]
    ep = np.stack([-np.sin(ph), np.cos(ph), 0 * ph], 1)
    et = np.stack([ct * np.cos(ph), ct * np.sin(ph), -st], 1)
    nr, nt, nph = (np.sum(n * e, 1) for e in (er, et, ep))
    H = np.zeros((len(r), (p + 1) ** 2), complex)
    D = np.zeros_like(H)
    pmm = np.full(len(r), math.sqrt(1 / (4 * math.pi)))
    for m in range(p + 1):
        if m:
            pmm = -math.sqrt((2 * m + 1) / (2 * m)) * st * pmm
        a, b = 0 * pmm, pmm
        e = np.exp(1j * m * ph)
        for l in range(m, p + 1):
            if l > m:
                f = math.sqrt((4 * l * l - 1) / (l * l - m * m))
                g = math.sqrt(((l - 1) ** 2 - m * m) / (4 * (l - 1) ** 2 - 1))
                a, b = b, f * (ct * b - g * a)
            dth = (l * ct * b - (math.sqrt((2 * l + 1) / (2 * l - 1) * (l * l - m * m)) * a if l > m else 0)) / st
            djl = (j[l - 1] if l else -j[1]) - (l + 1) / (k * r) * j[l] if l else -j[1]
            h = j[l] * b * e
            d = (k * djl * b * nr + j[l] * dth / r * nt) * e + 1j * m * h / rho * nph
            H[:, l * l + l + m], D[:, l * l + l + m] = h, d
            if m:
                H[:, l * l + l - m], D[:, l * l + l - m] = (-1) ** m * np.conj(h), (-1) ** m * np.conj(d)
    return H, D


def _exact_solve(c, w, x):
    """Amplitudes a, b and the field at x of one wave: GMRES on the dense operators of the scheme."""
    E = _Exact(c)
    E.factor()
    k, ex, ey, z0, P, M, M1, cut = c["k"], c["ex"], c["ey"], c["z0"], c["P"], c["M"], c["M1"], math.pi * c["N0"]
    kv = _kvec(k, w)
    al, be = np.exp(1j * kv[0] * ex), np.exp(1j * kv[1] * ey)
    near = [(a * ex, b * ey, 0.0, al ** a * be ** b) for a in (-1, 0, 1) for b in (-1, 0, 1)]
    y = _gpu(E.points(0, P))

    def summed(X, n, images, value):
        out = torch.zeros(len(X), len(y), dtype=torch.complex128, device="cuda")
        for sx, sy, _, wt in images:
            for t in range(0, len(X), 512):
                v, d = E.kernel(k, _gpu(X[t:t + 512] - np.array([sx, sy, 0.0])), _gpu(n[t:t + 512]), y)
                out[t:t + 512] += complex(wt) * (v if value else d)
        return out

    X, n = (v.reshape(-1, 3) for v in E.nodes())
    rows = (True, False) if c["km"] > 0 else (False,)
    Kelse = [summed(X, n, [i for i in near if i[:2] != (0.0, 0.0)], v) for v in rows]
    # walls: R, L, F, B, T, D
    g = np.polynomial.legendre.leggauss(M1)[0]
    u, v = (q.ravel() for q in np.meshgrid(g, g, indexing="ij"))
    o = np.ones(M1 * M1)
    walls = [np.stack(q, 1) for q in (((ex / 2) * o, u * ey / 2, v * z0), (-(ex / 2) * o, u * ey / 2, v * z0),
                                      (u * ex / 2, (ey / 2) * o, v * z0), (u * ex / 2, -(ey / 2) * o, v * z0),
                                      (u * ex / 2, v * ey / 2, z0 * o), (u * ex / 2, v * ey / 2, -z0 * o))]
    nrm = [np.tile(np.eye(3)[i // 2], (M1 * M1, 1)) for i in range(6)]

    def far(i):   # the images that the 3x3 cancellation leaves on each wall
        return [q for q in near if i > 3 or round(q[i // 2] / (ex, ey)[i // 2]) == (-1, 1)[i % 2]]

    C = [[summed(walls[i], nrm[i], far(i), val) for val in (True, False)] for i in range(6)]
    S = [_harmonics(k, c["p"], walls[i], nrm[i]) for i in range(6)]
    pair = lambda q: [q[0][0] - al * q[1][0], q[0][1] - al * q[1][1], q[2][0] - be * q[3][0], q[2][1] - be * q[3][1],  # noqa: E731
                      q[4][0], q[4][1], q[5][0], q[5][1]]
    C, S = torch.cat(pair(C), 0), np.concatenate(pair(S), 0)
    reach = [int(cut * e / TWO_PI + abs(kv[i]) * e / TWO_PI) + 2 for i, e in ((0, ex), (1, ey))]
    mn = [(m, q) for m in range(-reach[0], reach[0] + 1) for q in range(-reach[1], reach[1] + 1)
          if (kv[0] + TWO_PI * m / ex) ** 2 + (kv[1] + TWO_PI * q / ey) ** 2 <= cut * cut]
    kx, ky = (np.array([kv[i] + TWO_PI * q[i] / e for q in mn]) for i, e in ((0, ex), (1, ey)))
    kz = np.sqrt((k * k - kx ** 2 - ky ** 2).astype(complex))
    e = np.exp(1j * (np.outer(walls[4][:, 0], kx) + np.outer(walls[4][:, 1], ky)))
    Wa, Wb = np.zeros((2, len(S), len(mn)), complex)
    r0 = 4 * M1 * M1
    Wa[r0:r0 + 2 * M1 * M1] = np.concatenate([e, 1j * kz * e])
    Wb[r0 + 2 * M1 * M1:] = np.concatenate([e, -1j * kz * e])
    Q = np.concatenate([S, -Wa, -Wb], 1)
    D = 1 / np.linalg.norm(Q, axis=0)
    q1, r1 = np.linalg.qr(Q * D)
    uu, ss, vv = np.linalg.svd(r1)
    keep = ss > 1e-10 * ss[0]
    Qu, Qv = _gpu(np.conj((q1 @ uu)[:, keep].T) / ss[keep, None]), _gpu(D[:, None] * np.conj(vv[keep].T))
    B = [_harmonics(k, c["p"], np.stack([E.surf[:, 0], 0 * E.surf[:, 0], E.surf[:, 1]], 1),
                    np.stack([E.surf[:, 2], 0 * E.surf[:, 0], E.surf[:, 3]], 1))[0 if val else 1] for val in rows]
    B, NH = _gpu(np.concatenate(B, 0)), (c["p"] + 1) ** 2
    bins = _gpu(np.concatenate([np.arange(-l, l + 1) for l in range(c["p"] + 1)]) % P)

    def wall_xi(cf):
        return Qv @ (Qu @ (C @ E.strengths(cf, 0, P)))

    def op(xv):
        cf = E.pinv(xv.reshape(P, -1))
        sig = E.strengths(cf, 0, P)
        out = torch.cat([torch.fft.fft((K @ sig).reshape(P, M), dim=0) / P for K in Kelse], 1)
        sub = torch.zeros_like(out)
        sub.index_add_(0, bins, (B * wall_xi(cf)[:NH]).T.contiguous())
        return xv + (out - sub).reshape(-1)

    f = E.rhs(kv).reshape(-1)
    V, H = [f / f.norm()], np.zeros((81, 80), complex)
    for j in range(80):
        z = op(V[j])
        for again in (0, 1):
            for i in range(j + 1):
                h = torch.vdot(V[i], z)
                H[i, j] += h.item()
                z = z - h * V[i]
        H[j + 1, j] = z.norm().item()
        V.append(z / H[j + 1, j].real)
        rhs = np.zeros(j + 2, complex)
        rhs[0] = f.norm().item()
        yv, *_ = np.linalg.lstsq(H[:j + 2, :j + 1], rhs, rcond=None)
        if np.linalg.norm(H[:j + 2, :j + 1] @ yv - rhs) <= 1e-14 * rhs[0].real:
            break
    cf = E.pinv(sum(complex(yv[i]) * V[i] for i in range(j + 1)).reshape(P, -1))
    xi = -wall_xi(cf).cpu().numpy()
    fld = E.field(cf, x, 0, near, c["q_field"]).cpu().numpy() + _harmonics(k, c["p"], x, 0 * x + 1)[0] @ xi[:NH]
    m, n = np.array(mn).T
    return _on_orders(c, m, n, xi[NH:NH + len(mn)]), _on_orders(c, m, n, xi[NH + len(mn):]), fld


def _exact_free(c, kvec, points, inner, seed_q):
    """Ranks, singular values and fields of one body; None where its SVDs would take long."""
    if max(c["M"], 1) * c["N"] ** 2 * (c["P"] // 2 + 1) * (8 if c["km"] > 0 else 1) > 4e8:
        return None
    E = _Exact(c)
    E.factor()
    cs = [E.pinv(E.rhs(kv)) for kv in kvec]
    out = torch.stack([E.field(q, points, 0, qs=seed_q) for q in cs])
    if inner is not None:
        out = (out, torch.stack([E.field(q, inner, 1, qs=seed_q) for q in cs]))
    return E.ranks, E.sv, out


def exact(case, seed):
    """The pass's outputs by plain torch and numpy in 64 bits; None for the largest, and for all but the first wave of
    a periodic solve, whose dense operators take seconds each."""
    c, kind = case, case["kind"]
    if kind == "batch":
        got = [_exact_free(b, [_kvec(b["k"], w) for w in _incidences(b, random.Random(seed + i))], _points(b, seed + i),
                           None, b["q"]) for i, b in enumerate(_batch(case, seed))]
        return dict(ranks=None, sv=[g and g[1] for g in got], field=[g and g[2] for g in got])
    if kind == "sum":
        sig, ab = _sources(c, seed)
        E = _Exact(c)
        y = _gpu(E.points(0, c["P"]))
        if c["set"] == "walls":
            return None   # the rows of the wall conditions are not sums over one image list
        X, n = (v.reshape(-1, 3) for v in E.nodes()) if c["set"] == "surface" else np.split(_user_points(c, seed), 2, 1)
        out = torch.zeros(c["waves"], len(X), dtype=torch.complex128, device="cuda")
        for a in (-1, 0, 1):
            for b in (-1, 0, 1):
                if c["set"] == "surface" and a == b == 0:
                    continue
                wt = _gpu(ab[:, 0] ** a * ab[:, 1] ** b)[:, None]
                for t in range(0, len(X), 512):
                    d = E.kernel(c["k"], _gpu(X[t:t + 512] - np.array([a * c["ex"], b * c["ey"], 0.0])), _gpu(n[t:t + 512]), y)[1]
                    out[:, t:t + 512] += wt * (sig.cuda().reshape(c["waves"], -1) @ d.T.contiguous())
        return out
    waves = _incidences(c, random.Random(seed))
    x = _points(c, seed)
    if kind in ("scatter", "evaluate"):
        got = _exact_free(c, [_kvec(c["k"], w) for w in waves], x, _points(c, seed, inside=True) if c["km"] > 0 else None,
                          c["q_field"])
        if got is None:
            return None
        return got[2] if kind == "evaluate" else dict(ranks=got[0], sv=got[1], field=got[2])
    if c["P"] * c["M"] * c["P"] * c["N"] > 2e8:
        return None
    a, b, f = _exact_solve(c, waves[0], x)
    rest = [None] * (len(waves) - 1)
    return dict(a=[a] + rest, b=[b] + rest, field=[f] + rest, kz=None)
