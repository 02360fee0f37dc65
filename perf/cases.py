"""The calls this library is used for, as cases that can be timed and compared.

A case is a dict of plain values.  ``prepare`` builds what a program holds before the call (a loaded
geometry, a mixer or a synthesis, the input blocks), ``run`` makes one pass through the public entry
points, ``work`` says what the pass cannot do without, and ``exact`` computes the same outputs in
64 bits with plain torch from the ray maps, without the library.

The geometries are the screen-map workloads of this repository's benchmark and tests: a square screen,
one smooth order-0 map and thin rings for the higher orders.  Handles are used as ``geometry_load``
returns them (no tuning run).  Quantities that the library hands back in FP64 although they are
computed from FP32 responses (singular values, probe energies) are returned in FP32, the precision
they carry.
"""
import math
from types import SimpleNamespace

import numpy as np
import torch

import paper_2609_05528_amd as rtt
from paper_2609_05528_amd.autograd import retarded_time_apply

R_IN, R_OUT = 6.0, 20.0
ORDER_DELAY = 16.3
DT_SRC = 4.0
BATCH_S0 = -76.0


# ------------------------------------------------------------------------------------- the cases
def _geo(side, orders, frames, cells, hats, incl, dt_obs=4.0):
    return dict(side=side, orders=orders, frames=frames, cells=cells, hats=hats, incl=incl, dt_obs=dt_obs)


G64 = _geo(64, 1, 40, 32, 40, 20.0)
G128 = _geo(128, 3, 128, 64, 96, 50.0)
G256 = _geo(256, 1, 192, 32, 200, 20.0)
G512 = _geo(512, 3, 512, 128, 256, 75.0, 2.0)


def listed():
    return [
        # one history through A and the hand-written A^T by autograd on the smallest workload: launches and latency
        dict(name="grad_64_1", kind="grad", nvec=1, **G64),
        # A on a block of test vectors (the block of a rank-256 range finder)
        dict(name="apply_128_264", kind="apply", nvec=264, **G128),
        # A^T on the same block
        dict(name="adjoint_128_264", kind="adjoint", nvec=264, **G128),
        # A on one history of the largest geometry (half-step frames)
        dict(name="apply_512_1", kind="apply", nvec=1, **G512),
        # A^T on one data vector of the largest geometry
        dict(name="adjoint_512_1", kind="adjoint", nvec=1, **G512),
        # 60 histories seen by 12 geometries of uneven image sizes and (mostly odd) frame counts: A on the
        # shared histories, then A^T on the data
        dict(name="batch_12_60", kind="batch", members=12, nvec=60),
        # 20 CG iterations of the ridge estimate of one movie (stream-ordered form)
        dict(name="ridge_256_1", kind="ridge", nvec=1, maxit=20, **G256),
        # the rank-256 randomized SVD and the TSVD estimate of four data vectors with its factors
        dict(name="rsvd_128_256", kind="rsvd", rank=256, power=2, nvec=4, **G128),
        # a block Lanczos run (block 32) and the TSVD estimate with its leading Ritz vectors
        dict(name="lanczos_128_8", kind="lanczos", rank=32, steps=8, nvec=4, **G128),
        # the unresolved-image mixer and its transpose on a block of responses
        dict(name="mix_128_264", kind="mix", mixer="unresolved", nvec=264, **G128),
        # age information over the 64-centre age grid, per order, with every geometry's probes
        dict(name="age_128_64", kind="age", mixer="none", ages=64, **G128),
        # the S_224 synthesis map and its transpose on a block of coefficient vectors
        dict(name="synth_128_264", kind="synth", nvec=264, **G128),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _rays(side):
    return max(1, int(0.715 * side * side))


def _draw_geo(rng, lo, hi, half_step=True):
    side = _log_int(rng, lo, hi)
    dt = rng.choice([4.0, 4.0, 2.0]) if half_step else 4.0
    frames = rng.randint(max(20, side // 3), min(512, 40 + 4 * side // 3))
    cells = min(128, max(16, 2 * rng.randint(side // 8, side // 4)))
    orders = rng.choice([1, 3, 3])
    hats = int(math.ceil(frames * dt / DT_SRC * rng.uniform(0.7, 1.1))) + rng.randint(2, 12)
    return _geo(side, orders, frames, cells, min(256, hats), rng.choice([20.0, 50.0, 75.0]), dt)


def _block(rng, c, most=3.0e8, cap=264):
    """A block size for which the data block stays below ``most`` values."""
    rows = _rays(c["side"]) * c["frames"]
    return max(1, min(cap, _log_int(rng, 1, max(1.0, min(cap, most / rows)))))


def draw(rng):
    kind = rng.choice(["grad", "apply", "adjoint", "apply", "adjoint", "batch", "ridge", "rsvd", "lanczos", "mix",
                       "age", "synth"])
    if kind == "batch":
        return dict(kind=kind, members=rng.randint(2, 12), nvec=_log_int(rng, 1, 48))
    if kind == "grad":
        c = _draw_geo(rng, 24, 128)
        return dict(kind=kind, nvec=rng.randint(1, 4), **c)
    if kind in ("apply", "adjoint"):
        c = _draw_geo(rng, 32, 512)
        return dict(kind=kind, nvec=_block(rng, c), **c)
    if kind == "ridge":
        c = _draw_geo(rng, 64, 256)
        return dict(kind=kind, nvec=_block(rng, c, 2.0e7, 16), maxit=rng.randint(8, 20), **c)
    if kind == "rsvd":
        c = _draw_geo(rng, 64, 112, half_step=False)
        return dict(kind=kind, rank=_log_int(rng, 16, 240), power=rng.choice([1, 2]), nvec=rng.randint(1, 6), **c)
    if kind == "lanczos":
        c = _draw_geo(rng, 64, 112, half_step=False)
        return dict(kind=kind, rank=rng.randint(16, 32), steps=rng.randint(4, 8), nvec=rng.randint(1, 6), **c)
    c = _draw_geo(rng, 48, 256, half_step=False)
    if kind == "mix":
        return dict(kind=kind, mixer=rng.choice(["unresolved", "total_flux"]), nvec=_block(rng, c), **c)
    if kind == "age":
        return dict(kind=kind, mixer=rng.choice(["none", "none", "unresolved", "total_flux"]),
                    ages=rng.randint(16, 64), **_draw_geo(rng, 48, 128, half_step=False))
    return dict(kind=kind, nvec=max(1, min(264, int(1.0e8 / (c["cells"] ** 2 * c["hats"])) // rng.randint(1, 16))), **c)


# ------------------------------------------------------------------------------- geometries (inputs)
def _maps(side, incl, orders):
    c = (np.arange(side, dtype=np.float64) + 0.5) * (2.0 * R_OUT / side) - R_OUT
    alpha, beta = (v.ravel() for v in np.meshgrid(c, c, indexing="xy"))
    b, theta = np.hypot(alpha, beta), np.mod(np.arctan2(beta, alpha), 2.0 * math.pi)
    maps = []
    for n in range(orders):
        if n == 0:
            sel = (b >= R_IN) & (b <= R_OUT)
            r = b[sel]
        else:
            rho = 5.2 * (1.0 + 0.02 * (2 - n))
            sel = np.abs(b - rho) <= 0.25
            r = np.clip(R_IN + (b[sel] - rho + 0.25) / 0.5 * (R_OUT - R_IN), R_IN, R_OUT)
        phi = np.mod(theta[sel] + n * math.pi, 2.0 * math.pi)
        delay = r * (1.0 - math.sin(math.radians(incl)) * np.cos(phi)) + ORDER_DELAY * n
        maps.append(SimpleNamespace(r=r, phi=phi, delay=delay, weight=np.full(r.shape, math.exp(-math.pi * n)),
                                    pixel=np.nonzero(sel)[0]))
    return maps


def _geometry(c, incl=None, s0=None):
    incl = c["incl"] if incl is None else incl
    if s0 is None:
        tau = R_OUT * (1.0 + math.sin(math.radians(incl))) + ORDER_DELAY * (c["orders"] - 1)
        s0 = DT_SRC * math.floor(-tau / DT_SRC) - DT_SRC
    grid = SimpleNamespace(n_orders=c["orders"], n_frames=c["frames"], t0=0.0, dt_obs=c["dt_obs"], n_r=c["cells"],
                           n_phi=c["cells"], r_in=R_IN, r_out=R_OUT, n_hat=c["hats"], s0=float(s0), dt_src=DT_SRC)
    return SimpleNamespace(grid=grid, maps=_maps(c["side"], incl, c["orders"]))


def _batch_members(n):
    """The uneven spin x inclination geometries over one shared 64 x 64 x 96 source grid."""
    out = []
    for g in range(12 - n, 12):
        side = 96 + int(round(160.0 * g / 11.0))
        frames = 64 + int(round(96.0 * ((7 * g) % 12) / 11.0))
        out.append(_geo(side, 3, frames, 64, 96, (20.0, 50.0, 75.0)[g % 3]))
    return out


def _geometries(case, seed):
    if case["kind"] == "batch":
        return [_geometry(m, s0=BATCH_S0) for m in _batch_members(case["members"])]
    if case["kind"] == "age":   # the geometry is this call's input: another seed sees it from another inclination
        return [_geometry(case, incl=case["incl"] + np.random.default_rng(seed).uniform(-1.0, 1.0))]
    return [_geometry(case)]


# -------------------------------------------------------------------------------------- the inputs
def _gen(seed):
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    return torch.Generator(device=dev).manual_seed(int(seed)), dev


def _histories(geo, nvec, seed):
    """Positive emissivity histories: blobs with a Gaussian envelope in space and time on a faint floor."""
    g = geo.grid
    gen, dev = _gen(seed)
    u = lambda *s: torch.rand(*s, generator=gen, device=dev)  # noqa: E731
    rc = torch.as_tensor(g.r_in + (np.arange(g.n_r) + 0.5) * (g.r_out - g.r_in) / g.n_r, dtype=torch.float32, device=dev)
    pc = torch.as_tensor((np.arange(g.n_phi) + 0.5) * 2 * math.pi / g.n_phi, dtype=torch.float32, device=dev)
    tk = torch.as_tensor(g.s0 + g.dt_src * np.arange(g.n_hat), dtype=torch.float32, device=dev)
    X, Y = (rc[:, None] * torch.cos(pc)).reshape(-1), (rc[:, None] * torch.sin(pc)).reshape(-1)
    x = 0.05 * u(nvec, g.n_r * g.n_phi, g.n_hat)
    for _ in range(3):
        rb = torch.sqrt(g.r_in ** 2 + (g.r_out ** 2 - g.r_in ** 2) * u(nvec, 1))
        pb, width, life = 2 * math.pi * u(nvec, 1), 1.0 + 2.0 * u(nvec, 1), 8.0 + 32.0 * u(nvec, 1)
        tb = tk[0] + (tk[-1] - tk[0]) * u(nvec, 1)
        sp = torch.exp(-((X - rb * torch.cos(pb)) ** 2 + (Y - rb * torch.sin(pb)) ** 2) / (2 * width ** 2))
        tp = torch.exp(-((tk - tb) ** 2) / (2 * life ** 2))
        x += (0.5 + u(nvec, 1))[:, :, None] * sp[:, :, None] * tp[:, None, :]
    return x.reshape(nvec, -1)


def _normal(shape, seed):
    gen, dev = _gen(seed)
    return torch.randn(shape, generator=gen, device=dev)


def _inputs(case, seed, geos):
    """The tensors of a case, from the seed alone."""
    kind = case["kind"]
    n_cols = sum(q.grid.n_r * q.grid.n_phi * q.grid.n_hat for q in geos)
    n_rows = sum(m.r.size for q in geos for m in q.maps) * geos[0].grid.n_frames if len(geos) == 1 else 0
    t = SimpleNamespace()
    if kind in ("grad", "apply", "batch"):
        t.x = _histories(geos[0], case["nvec"], seed)
    if kind == "grad":
        t.gy = _normal((case["nvec"], n_rows), seed + 1)
    if kind in ("adjoint", "mix", "ridge", "rsvd", "lanczos"):
        # a movie: brightness that varies from ray to ray and slowly in time, and white noise
        F = geos[0].grid.n_frames
        base = _normal((case["nvec"], n_rows // F, 1), seed + 2).abs()
        wave = 1.0 + 0.5 * torch.sin(torch.arange(F, device=base.device) * 0.2 + 3.0 * base)
        t.y = (base * wave + 0.1 * _normal((case["nvec"], n_rows // F, F), seed + 3)).reshape(case["nvec"], n_rows)
    if kind == "rsvd":
        t.omega = _normal((case["rank"] + 8, n_cols), seed + 4)
    if kind == "lanczos":
        t.omega = _normal((32, n_cols), seed + 4)
    if kind == "mix":
        d = _pixel_rows(geos[0], case["mixer"])[1]
        t.d = _normal((case["nvec"], d * geos[0].grid.n_frames), seed + 5)
    if kind == "age":
        t.ages = 4.0 * np.arange(case["ages"]) + np.random.default_rng(seed).uniform(0.0, 1.0)
        t.var = None
        if case["mixer"] != "none":
            t.var = 0.5 + _normal((n_rows,), seed + 6).abs()
    if kind == "synth":
        t.c = _normal((case["nvec"], 224), seed + 7)
        t.x = _histories(geos[0], case["nvec"], seed)
    return t


def prepare(case, seed):
    geos = _geometries(case, seed)
    s = _inputs(case, seed, geos)
    s.case = case
    s.geom = rtt.geometry_load(geos)
    if case.get("mixer", "none") != "none":
        pixels = [m.pixel for m in geos[0].maps] if case["mixer"] == "unresolved" else None
        s.mixer = rtt.mixer_create(s.geom, case["mixer"], pixels)
    else:
        s.mixer = None
    if case["kind"] == "synth":
        s.synth = rtt.Synthesis(s.geom)
    return s


# ----------------------------------------------------------------------------------------- one pass
def run(s):
    case, kind = s.case, s.case["kind"]
    if kind == "apply":
        return rtt.op_apply(s.geom, s.x)
    if kind == "adjoint":
        return rtt.op_apply_adjoint(s.geom, s.y)
    if kind == "grad":
        x = s.x.detach().requires_grad_(True)
        y = retarded_time_apply(x, s.geom)
        (gx,) = torch.autograd.grad(y, x, s.gy)
        return {"y": y, "gx": gx}
    if kind == "batch":
        y = rtt.op_apply_shared(s.geom, s.x)
        return {"y": y, "x": rtt.op_apply_adjoint(s.geom, y)}
    if kind == "ridge":
        x, _ = rtt.ridge_solve(s.geom, s.y, 1e-3, tol=1e-12, maxit=case["maxit"], async_mode=True)
        return x
    if kind in ("rsvd", "lanczos"):
        if kind == "rsvd":
            svd = rtt.rsvd(s.geom, k=case["rank"], p=8, q=case["power"], omega=s.omega)
        else:
            svd = rtt.rsvd(s.geom, k=case["rank"], method="lanczos", block=32, steps=case["steps"], omega=s.omega)
        return {"sigma": torch.from_numpy(svd.sigma).float(), "estimate": rtt.tsvd_solve(s.geom, svd, s.y)}
    if kind == "mix":
        return {"d": rtt.mix_apply(s.mixer, s.y), "y": rtt.mix_adjoint(s.mixer, s.d)}
    if kind == "age":
        e = rtt.age_information(s.geom, s.ages, mixer=s.mixer, var=s.var)
        return torch.from_numpy(e).float()
    return {"x": s.synth.expand(s.c), "c": s.synth.project(s.x)}


# ------------------------------------------------------------------- what a pass cannot do without
def work(case):
    kind = case["kind"]
    members = _batch_members(case["members"]) if kind == "batch" else [case]
    geos = [_geometry(m, s0=BATCH_S0 if kind == "batch" else None) for m in members]
    rows = [sum(m.r.size for m in q.maps) * q.grid.n_frames for q in geos]
    rays = sum(sum(m.r.size for m in q.maps) for q in geos)
    m, n = sum(rows), sum(q.grid.n_r * q.grid.n_phi * q.grid.n_hat for q in geos)
    v = case.get("nvec", 1)
    op = 4.0 * v * (m + n) + 32.0 * rays      # one application: rows, columns and the ray table once
    opf = 12.0 * v * m
    if kind in ("apply", "adjoint"):
        return {"bytes": op, "flops": opf}
    if kind == "grad":
        return {"bytes": 2 * op, "flops": 2 * opf}
    if kind == "batch":                       # one shared coefficient block in, one block per geometry out
        return {"bytes": 4.0 * v * (2 * m + n + n / len(geos)) + 64.0 * rays, "flops": 2 * opf}
    if kind == "ridge":                       # A and A^T per iteration (the data vector between them included)
        it = case["maxit"]
        return {"bytes": (2 * it + 1) * op, "flops": (2 * it + 1) * opf}
    if kind == "rsvd":
        l = case["rank"] + 8
        q = case["power"]
        one = 4.0 * l * (m + n) + 32.0 * rays
        gemm = 2.0 * l * l * ((q + 1) * m + (q + 2) * n) * 1.5 + 2.0 * l * case["rank"] * n
        return {"bytes": (2 * q + 2) * one + op, "flops": gemm + (2 * q + 2) * 12.0 * l * m}
    if kind == "lanczos":
        b, st = 32, case["steps"]
        one = 4.0 * b * (m + n) + 32.0 * rays
        gemm = sum(2.0 * b * b * 1.5 * (m + n) + 2.0 * b * b * (m + n) + 8.0 * (j + 1) * b * b * n for j in range(st))
        return {"bytes": 2 * st * one + op, "flops": gemm + 2 * st * 12.0 * b * m}
    if kind == "mix":
        d = _pixel_rows(geos[0], case["mixer"])[1] * geos[0].grid.n_frames
        return {"bytes": 8.0 * v * (m + d), "flops": 2.0 * v * m}
    if kind == "age":                         # ray table (and variances) in, energies out; a response is summed as it forms
        return {"bytes": 32.0 * rays + (4.0 * m if case["mixer"] != "none" else 0.0) + 64.0 * case["ages"],
                "flops": 6.0 * case["ages"] * m}
    return {"bytes": 8.0 * v * n, "flops": 4.0 * v * n * 7}


# --------------------------------------------------------------------------- the outputs in 64 bits
class _Op:
    """A and A^T of one geometry in 64 bits, straight from the ray maps."""

    def __init__(self, geo, dev):
        g = self.g = geo.grid
        cat = lambda a: np.concatenate([np.asarray(getattr(m, a), dtype=np.float64) for m in geo.maps])  # noqa: E731
        r, phi, delay, w = cat("r"), cat("phi"), cat("delay"), cat("weight")
        ur = np.clip((r - g.r_in) / ((g.r_out - g.r_in) / g.n_r) - 0.5, 0.0, g.n_r - 1.0)
        i = np.minimum(np.floor(ur), g.n_r - 2).astype(np.int64)
        up = np.mod(phi, 2 * math.pi) / (2 * math.pi / g.n_phi) - 0.5
        j = np.floor(up).astype(np.int64)
        fr, fp = ur - i, up - j
        j0, j1 = j % g.n_phi, (j + 1) % g.n_phi
        cells = np.stack([i * g.n_phi + j0, (i + 1) * g.n_phi + j0, i * g.n_phi + j1, (i + 1) * g.n_phi + j1])
        wts = w * np.stack([(1 - fr) * (1 - fp), fr * (1 - fp), (1 - fr) * fp, fr * fp])
        u = (g.t0 + g.dt_obs * np.arange(g.n_frames) - delay[:, None] - g.s0) / g.dt_src
        k = np.floor(u)
        self.theta = torch.as_tensor(u - k, device=dev)
        self.k = torch.as_tensor(np.clip(k, -1, g.n_hat).astype(np.int64) + 1, device=dev)   # 0 .. K + 1, padded hats
        self.theta[torch.as_tensor((k < -1) | (k > g.n_hat), device=dev)] = 0.0
        self.cells, self.w = torch.as_tensor(cells, device=dev), torch.as_tensor(wts, device=dev)
        self.n_rays, self.K, self.F, self.n_cells = r.size, g.n_hat, g.n_frames, g.n_r * g.n_phi

    def _parts(self, nvec):
        step = max(1, int(3e7 // (max(self.K, self.F) * nvec)))
        return [(a, min(a + step, self.n_rays)) for a in range(0, self.n_rays, step)]

    def apply(self, x):
        nv = x.shape[0]
        x = x.double().reshape(nv, self.n_cells, self.K)
        y = torch.empty((nv, self.n_rays, self.F), dtype=torch.float64, device=x.device)
        for a, b in self._parts(nv):
            z = x.new_zeros((nv, b - a, self.K + 3))
            for c in range(4):
                z[:, :, 1:self.K + 1] += self.w[c, a:b, None] * x[:, self.cells[c, a:b]]
            k, th = self.k[a:b].expand(nv, -1, -1), self.theta[a:b]
            y[:, a:b] = (1 - th) * torch.gather(z, 2, k) + th * torch.gather(z, 2, k + 1)
        return y.reshape(nv, -1)

    def adjoint(self, y):
        nv = y.shape[0]
        y = y.reshape(nv, self.n_rays, self.F)
        x = torch.zeros((nv, self.n_cells, self.K), dtype=torch.float64, device=y.device)
        for a, b in self._parts(nv):
            yb, th = y[:, a:b].double(), self.theta[a:b]
            z = x.new_zeros((nv, b - a, self.K + 3))
            k = self.k[a:b].expand(nv, -1, -1)
            z.scatter_add_(2, k, (1 - th) * yb)
            z.scatter_add_(2, k + 1, th * yb)
            for c in range(4):
                x.index_add_(1, self.cells[c, a:b], self.w[c, a:b, None] * z[:, :, 1:self.K + 1])
        return x.reshape(nv, -1)


def _pixel_rows(geo, kind):
    """The mixed row of every ray, and the number of mixed rows per frame."""
    if kind == "total_flux":
        return np.zeros(sum(m.r.size for m in geo.maps), dtype=np.int64), 1
    pix = np.concatenate([m.pixel for m in geo.maps])
    u, inv = np.unique(pix, return_inverse=True)
    return inv.reshape(-1), u.size


def _mix(y, rows, n, F):
    nv = y.shape[0]
    d = torch.zeros((nv, n, F), dtype=torch.float64, device=y.device)
    return d.index_add_(1, rows, y.double().reshape(nv, -1, F)).reshape(nv, -1)


def _qr(Y):
    """Orthonormal rows of a block [l][n] and the upper factor R with Y^T = Q^T R (twice Cholesky, 64 bits)."""
    R = torch.eye(Y.shape[0], dtype=torch.float64, device=Y.device)
    for _ in range(2):
        L = torch.linalg.cholesky(Y @ Y.T)
        Y = torch.linalg.inv(L) @ Y
        R = L.T @ R
    return Y, R


def _rsvd(op, omega, q, k):
    Q = _qr(op.apply(omega))[0]
    for _ in range(q):
        Q = _qr(op.apply(_qr(op.adjoint(Q))[0]))[0]
    Qb, R = _qr(op.adjoint(Q))
    _, s, Wh = torch.linalg.svd(R.T)
    return s[:k], Wh[:k] @ Qb


def _lanczos(op, start, steps, k):
    V, _ = _qr(start.double())
    Vs, b = [V], V.shape[0]
    T = torch.zeros((b * steps, b * steps), dtype=torch.float64, device=V.device)
    U = R = None
    for j in range(steps):
        W = op.apply(Vs[j])
        if U is not None:
            W -= R @ U
        U, L = _qr(W)
        T[j * b:(j + 1) * b, j * b:(j + 1) * b] = L
        Z = op.adjoint(U) - L @ Vs[j]
        for _ in range(2):
            for Vo in Vs:
                Z -= (Z @ Vo.T) @ Vo
        if j + 1 < steps:
            Vn, R = _qr(Z)
            T[j * b:(j + 1) * b, (j + 1) * b:(j + 2) * b] = R.T
            Vs.append(Vn)
    _, s, Ph = torch.linalg.svd(T)
    return s[:k], Ph[:k] @ torch.cat(Vs)


def exact(case, seed):
    kind = case["kind"]
    geos = _geometries(case, seed)
    t = _inputs(case, seed, geos)
    dev = _gen(0)[1]
    if kind == "batch":
        ops = [_Op(q, dev) for q in geos]
        y = torch.empty((case["nvec"], sum(o.n_rays * o.F for o in ops)), dtype=torch.float64, device=dev)
        xs, at = [], 0
        for o in ops:
            m = o.n_rays * o.F
            y[:, at:at + m] = o.apply(t.x)
            xs.append(o.adjoint(y[:, at:at + m]))
            at += m
        return {"y": y, "x": torch.cat(xs, dim=1)}
    if kind == "synth":
        g = geos[0].grid
        rc = g.r_in + (np.arange(g.n_r) + 0.5) * (g.r_out - g.r_in) / g.n_r
        u = np.log(rc / g.r_in) / math.log(g.r_out / g.r_in)
        R = np.stack([(1 - u) ** 3, 3 * u * (1 - u) ** 2, 3 * u ** 2 * (1 - u), u ** 3])
        pc = (np.arange(g.n_phi) + 0.5) * 2 * math.pi / g.n_phi
        P = np.stack([np.ones_like(pc)] + [f(m * pc) for m in (1, 2, 3) for f in (np.cos, np.sin)])
        T = np.stack([np.cos(math.pi * c * (np.arange(g.n_hat) + 0.5) / g.n_hat) for c in range(8)])
        Q = torch.as_tensor(np.einsum("ai,bj,ck->abcijk", R, P, T).reshape(224, -1), device=dev)
        return {"x": t.c.double() @ Q, "c": t.x.double() @ Q.T}
    if kind == "mix":
        rows, n = _pixel_rows(geos[0], case["mixer"])
        rows, F = torch.as_tensor(rows, device=dev), geos[0].grid.n_frames
        d = t.d.double().reshape(case["nvec"], n, F)
        return {"d": _mix(t.y, rows, n, F), "y": d[:, rows].reshape(case["nvec"], -1)}
    op = _Op(geos[0], dev)
    if kind == "apply":
        return op.apply(t.x)
    if kind == "adjoint":
        return op.adjoint(t.y)
    if kind == "grad":
        return {"y": op.apply(t.x), "gx": op.adjoint(t.gy)}
    if kind == "ridge":
        r = op.adjoint(t.y)
        x, p, rr = torch.zeros_like(r), r.clone(), (r * r).sum(1, keepdim=True)
        for _ in range(case["maxit"]):
            Ap = op.adjoint(op.apply(p)) + float(np.float32(1e-3)) * p
            a = rr / (p * Ap).sum(1, keepdim=True)
            x, r = x + a * p, r - a * Ap
            new = (r * r).sum(1, keepdim=True)
            p, rr = r + new / rr * p, new
        return x
    if kind in ("rsvd", "lanczos"):
        if kind == "rsvd":
            s, V = _rsvd(op, t.omega, case["power"], case["rank"])
        else:
            s, V = _lanczos(op, t.omega, case["steps"], case["rank"])
        return {"sigma": s, "estimate": ((op.adjoint(t.y) @ V.T) / s ** 2) @ V}
    g = geos[0].grid
    norm = math.sqrt(math.pi * (g.r_out ** 2 - g.r_in ** 2) * 3.0 * math.sqrt(math.pi))
    sk = g.s0 + g.dt_src * np.arange(g.n_hat)
    x = np.exp(-((sk + t.ages[:, None]) ** 2) / 18.0) / norm
    if case["mixer"] != "none":
        rows, n = _pixel_rows(geos[0], case["mixer"])
        rows = torch.as_tensor(rows, device=dev)
        var = _mix(t.var[None], rows, n, op.F)
    out = torch.zeros((len(t.ages), 1, 8) if case["mixer"] == "none" else (len(t.ages), 1), dtype=torch.float64)
    for i in range(len(t.ages)):
        y = op.apply(torch.as_tensor(x[i], device=dev).repeat(op.n_cells)[None])
        if case["mixer"] != "none":
            out[i, 0] = float((_mix(y, rows, n, op.F) ** 2 / var).sum())
            continue
        at = 0
        for k, m in enumerate(geos[0].maps):
            out[i, 0, k] = float((y[0, at:at + m.r.size * op.F] ** 2).sum())
            at += m.r.size * op.F
    return out
