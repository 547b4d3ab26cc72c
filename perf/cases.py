"""Performance cases of the hierarchical Jacobi library: what a program has it do, through the entry points of
paper_2006_16465_amd.hj, from one 256-point solve to 4096 x 4096 grids, batches and the differentiable solve.

A case is a dict: "kind" says which entry point runs, the rest are its arguments.  Right-hand sides are sums of
random sine modes (as the workloads draw them), constants (the paper's own experiments) or modes plus noise; x0 is 0
or 1.  "cap" bounds the cycles of a solve to a tolerance (a right-hand side with a very smooth mode would take Jacobi
far longer than any other), and "cycles" is the count that the work of a pass is reckoned with: the typical one.
"""
import math

import numpy as np
import torch

from paper_2006_16465_amd import hj

DEV = "cuda"
F64 = torch.float64


def listed():
    return [
        # the paper's 1D size: one small solve to tolerance, latency of a cycle and of the call
        dict(name="1d_256", kind="1d", n=256, tile=64, s=8, overlap=14, tol=1e-6, cap=2000, cycles=270),
        # a large 1D grid, odd size, at the shape the tuner picks: a launch per cycle
        dict(name="1d_1m", kind="1d", n=1_000_003, tile=256, s=32, overlap=62, tol=1e-8, cap=300, cycles=60),
        # the paper's 1D experiment as a batch of copies (constant right-hand side, x0 = 1, to 1e-4), one workgroup each
        dict(name="1d_batch_1024", kind="1d_batch", n=1024, copies=1024, tile=256, s=32, overlap=62, tol=1e-4, cap=4500,
             cycles=4024),
        # the smallest 2D solves: ragged sides, hx != hy, small tiles
        dict(name="2d_150x101_aniso", kind="2d", nx=150, ny=101, pad=3, aniso=1.5, dtype="f64", tx=32, ty=32, s=8, ox=14,
             oy=14, modes=8, noise=0.0, tol=1e-6, cap=1000, cycles=200, method="hierarchical"),
        # the paper's 2D setting (32 x 32 tiles, 16 sub-iterations, no overlap) on its ordinary grid
        dict(name="2d_512_paper", kind="2d", nx=512, ny=512, pad=0, aniso=1.0, dtype="f64", tx=32, ty=32, s=16, ox=0, oy=0,
             modes=16, noise=0.1, tol=1e-6, cap=500, cycles=500, method="hierarchical"),
        # the benchmark's problem and shape: time to 1e-6 on 4096 x 4096
        dict(name="2d_4096", kind="2d", nx=4096, ny=4096, pad=0, aniso=1.0, dtype="f64", tx=64, ty=128, s=16, ox=22, oy=22,
             modes=8, noise=0.0, tol=1e-6, cap=64, cycles=13, method="hierarchical"),
        # classical Jacobi on the same problem, the method every other one is compared with
        dict(name="2d_4096_global", kind="2d", nx=4096, ny=4096, pad=0, aniso=1.0, dtype="f64", tx=32, ty=32, s=1, ox=0,
             oy=0, modes=8, noise=0.0, tol=1e-6, cap=400, cycles=190, method="global"),
        # single precision on a ragged, pitched grid, a fixed number of cycles (a smoother's use)
        dict(name="2d_f32_ragged", kind="2d", nx=2049, ny=1531, pad=7, aniso=1.0, dtype="f32", tx=64, ty=64, s=12, ox=22,
             oy=22, modes=8, noise=0.1, tol=0.0, cap=40, cycles=40, method="hierarchical"),
        # FP32 cycles inside FP64 refinement, to 1e-10 on the benchmark's grid
        dict(name="2d_4096_refined", kind="refined", n=4096, tx=64, ty=128, s=12, o=22, modes=8, tol=1e-10, cap=2000,
             cycles=30),
        # many problems of uneven sizes at once, in the batched workload's ranges
        dict(name="batch_mixed", kind="batch", n2=40, n1=12, size_seed=0, dtype="f64", tx=64, ty=64, s=10, o=18, t1=256,
             s1=32, o1=62, refine=False, tol=1e-8, cap=200, cycles=60),
        # a training step through the differentiable solve: forward, adjoint, gradients of f and a
        dict(name="vc_train_64x16", kind="vc_train", n=64, batch=16, tx=64, ty=32, s=8, o=14, tol=1e-10, cap=100_000,
             cycles=9000),
        # the variable-coefficient forward solve at its configured size
        dict(name="vc_1024x16", kind="vc", nx=1024, ny=1024, batch=16, tx=64, ty=32, s=8, o=14, tol=1e-10, cap=100,
             cycles=100),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["1d", "1d_batch", "2d", "2d", "2d", "2d", "refined", "batch", "vc_train", "vc"])
    if kind == "1d":
        n = _log(rng, 200, 1_000_003)
        tile = rng.choice([64, 128, 256, 512])
        s = rng.choice([4, 8, 16, 32])
        o = rng.choice([0, min(2 * s - 2, tile // 2), s // 2])
        return dict(kind="1d", n=n, tile=tile, s=s, overlap=o, tol=1e-6, cap=300, cycles=100)
    if kind == "1d_batch":
        n = _log(rng, 100, 1500)
        tile, s = rng.choice([(128, 16), (256, 32), (256, 16)])
        return dict(kind="1d_batch", n=n, copies=_log(rng, 16, 1024), tile=tile, s=s, overlap=2 * s - 2, tol=1e-4, cap=1000,
                    cycles=1000)
    if kind == "2d":
        nx, ny = _log(rng, 64, 4096), _log(rng, 128, 4096)
        method = "global" if rng.random() < 0.2 else "hierarchical"
        tx, ty = rng.choice([(32, 32), (32, 64), (64, 32), (64, 64), (64, 128)])
        s = rng.choice([4, 8, 12, 16])
        o = min(rng.choice([0, 2 * s - 2, 2 * s - 6, s // 2]), min(tx, ty) // 2)
        dtype = rng.choice(["f64", "f64", "f32"])
        cap = max(6, min(300, int(60 * 2 ** 20 / (nx * ny))))
        return dict(kind="2d", nx=nx, ny=ny, pad=rng.choice([0, 0, 1, 6]), aniso=rng.choice([1.0, 1.0, 1.0, 0.7]),
                    dtype=dtype, tx=tx, ty=ty, s=s, ox=max(0, o), oy=max(0, o), modes=8, noise=rng.choice([0.0, 0.1]),
                    tol=0.0 if dtype == "f32" else rng.choice([0.0, 1e-6]), cap=cap, cycles=cap, method=method)
    if kind == "refined":
        n = _log(rng, 512, 4096)
        return dict(kind="refined", n=n, tx=64, ty=rng.choice([64, 128]), s=12, o=22, modes=8, tol=1e-10, cap=2000, cycles=30)
    if kind == "batch":
        return dict(kind="batch", n2=rng.randint(8, 40), n1=rng.randint(2, 12), size_seed=rng.randint(1, 10 ** 6),
                    dtype=rng.choice(["f64", "f64", "f32"]), tx=rng.choice([32, 64]), ty=64, s=10, o=18, t1=256, s1=32, o1=62,
                    refine=False, tol=0.0, cap=rng.choice([20, 60]), cycles=40)
    if kind == "vc_train":
        return dict(kind="vc_train", n=rng.randint(20, 64), batch=rng.randint(1, 16), tx=rng.choice([32, 64]), ty=32, s=8,
                    o=14, tol=1e-10, cap=100_000, cycles=4000)
    return dict(kind="vc", nx=_log(rng, 48, 1024), ny=_log(rng, 48, 1024), batch=rng.randint(1, 16), tx=rng.choice([32, 64]),
                ty=rng.choice([16, 32]), s=rng.choice([4, 8]), o=rng.choice([0, 14]), tol=1e-10, cap=100, cycles=100)


# ---------------------------------------------------------------- inputs
def _modes_1d(n, modes, rng):
    k = torch.from_numpy(rng.integers(1, n + 1, modes).astype(np.float64)).to(DEV)
    a = torch.from_numpy(rng.standard_normal(modes)).to(DEV)
    x = torch.arange(1, n + 1, dtype=F64, device=DEV) / (n + 1)
    return (a[:, None] * torch.sin(math.pi * k[:, None] * x[None, :])).sum(0)


def _mode_tables(nx, ny, modes, rng):
    k = rng.integers(1, nx + 1, modes).astype(np.float64)
    l = rng.integers(1, ny + 1, modes).astype(np.float64)
    a = rng.standard_normal(modes)
    k, l, a = (torch.from_numpy(v).to(DEV) for v in (k, l, a))
    sx = torch.sin(math.pi * k[:, None] * (torch.arange(1, nx + 1, dtype=F64, device=DEV) / (nx + 1))[None, :])
    sy = torch.sin(math.pi * l[:, None] * (torch.arange(1, ny + 1, dtype=F64, device=DEV) / (ny + 1))[None, :])
    return k, l, a, sx, sy


def _modes_2d(nx, ny, modes, rng, noise=0.0):
    _, _, a, sx, sy = _mode_tables(nx, ny, modes, rng)
    f = (sy.T * a[None, :]) @ sx
    if noise > 0.0:
        g = torch.Generator(device=DEV).manual_seed(int(rng.integers(0, 2 ** 31)))
        f = f + noise * torch.randn(ny, nx, dtype=F64, device=DEV, generator=g)
    return f


def _coefficient(nx, ny, rng, length=0.05):
    """exp of a Gaussian random field on the (ny + 2) x (nx + 2) nodes: white noise filtered by FFT."""
    w = torch.from_numpy(rng.standard_normal((ny + 2, nx + 2))).to(DEV)
    ky = torch.fft.fftfreq(ny + 2, d=1.0 / (ny + 1), dtype=F64, device=DEV)
    kx = torch.fft.fftfreq(nx + 2, d=1.0 / (nx + 1), dtype=F64, device=DEV)
    filt = torch.exp(-math.pi ** 2 * length ** 2 * (ky[:, None] ** 2 + kx[None, :] ** 2))
    g = torch.fft.ifft2(torch.fft.fft2(w) * filt).real
    return torch.exp(g / torch.sqrt((filt ** 2).mean())).contiguous()


def _spacings(c):
    hx = 1.0 / (c["nx"] + 1)
    return hx, hx * c["aniso"]


def _pitched(f, pad, dtype):
    """f in rows of nx + pad elements."""
    buf = torch.zeros(f.shape[0], f.shape[1] + pad, dtype=dtype, device=DEV)
    v = buf[:, : f.shape[1]]
    v.copy_(f)
    return v


def _batch_sizes(c):
    r = np.random.default_rng(c["size_seed"])
    sides = np.exp(r.uniform(np.log(64), np.log(1024), c["n2"])).astype(np.int64)
    ns = np.exp(r.uniform(np.log(1_000), np.log(1_000_000), c["n1"])).astype(np.int64)
    return [int(v) for v in sides], [int(v) for v in ns]


def _type(c):
    return F64 if c.get("dtype", "f64") == "f64" else torch.float32


def _inputs(c, seed):
    """The right-hand side(s) and whatever else the problem holds, in the case's type."""
    rng = np.random.default_rng(seed)
    kind = c["kind"]
    if kind == "1d":
        return _modes_1d(c["n"], 8, rng)
    if kind == "1d_batch":
        amp = torch.from_numpy(rng.uniform(0.5, 2.0, c["copies"])).to(DEV)
        return amp[:, None].expand(-1, c["n"]).contiguous()
    if kind == "2d":
        return _pitched(_modes_2d(c["nx"], c["ny"], c["modes"], rng, c["noise"]), c["pad"], _type(c))
    if kind == "refined":
        return _modes_2d(c["n"], c["n"], c["modes"], rng)
    if kind == "batch":
        sides, ns = _batch_sizes(c)
        fs = [_modes_2d(n, n, 8, rng).to(_type(c)) for n in sides]
        return fs + [_modes_1d(n, 8, rng).to(_type(c)) for n in ns]
    nx, ny = (c["n"], c["n"]) if kind == "vc_train" else (c["nx"], c["ny"])
    a = _coefficient(nx, ny, rng)
    f = torch.stack([_modes_2d(nx, ny, 8, rng) for _ in range(c["batch"])])
    if kind == "vc":
        return f, a
    t = torch.stack([_smooth(nx, rng) for _ in range(c["batch"])]) * 1e-3
    return f, a, t


def _smooth(n, rng):
    """A smooth target: three products of the lowest modes."""
    xs = torch.arange(1, n + 1, dtype=F64, device=DEV) / (n + 1)
    u = torch.zeros(n, n, dtype=F64, device=DEV)
    for _ in range(3):
        k, l = rng.integers(1, 4, 2)
        u += float(rng.standard_normal()) * torch.outer(torch.sin(math.pi * int(l) * xs), torch.sin(math.pi * int(k) * xs))
    return u


# ---------------------------------------------------------------- the framework's pass
def prepare(case, seed):
    hj.load()
    c, kind = case, case["kind"]
    v = _inputs(c, seed)
    st = {"c": c}
    if kind in ("1d", "refined"):
        st |= {"f": v, "x": torch.zeros_like(v)}
    elif kind == "1d_batch":
        st |= {"f": v, "x": torch.ones_like(v)}
        st["table"] = [(st["f"][i], st["x"][i], 1.0 / (c["n"] + 1)) for i in range(c["copies"])]
    elif kind == "2d":
        x = torch.zeros(c["ny"], c["nx"] + c["pad"], dtype=_type(c), device=DEV)
        st |= {"f": v, "x": x[:, : c["nx"]]}
    elif kind == "batch":
        st["x"] = [torch.zeros_like(f) for f in v]
        st["table"] = [(f, x, 1.0 / (f.shape[-1] + 1)) for f, x in zip(v, st["x"])]
    elif kind == "vc":
        st |= {"f": v[0], "a": v[1], "x": torch.zeros_like(v[0])}
    else:
        st |= {"f": v[0].requires_grad_(True), "a": v[1].requires_grad_(True), "t": v[2]}
    return st


def _report(info):
    return {"cycles": info.cycles, "rel_residual": info.rel_residual, "r0_norm": info.r0_norm}


def _reports(infos):
    return {"cycles": np.array([i.cycles for i in infos]), "rel_residual": np.array([i.rel_residual for i in infos]),
            "r0_norm": np.array([i.r0_norm for i in infos])}


def run(state):
    c = state["c"]
    kind = c["kind"]
    if kind == "1d":
        x = state["x"].zero_()
        info = hj.solve_1d(state["f"], x, 1.0 / (c["n"] + 1), tile=c["tile"], s=c["s"], overlap=c["overlap"],
                           rel_tol=c["tol"], max_cycles=c["cap"], allow_not_converged=True)
        return {"x": x, **_report(info)}
    if kind == "1d_batch":
        state["x"].fill_(1.0)
        infos = hj.solve_batched(state["table"], rel_tol=c["tol"], tile_1d=c["tile"], s_1d=c["s"], overlap_1d=c["overlap"],
                                 max_cycles=c["cap"], one_workgroup_1d=True, allow_not_converged=True)
        return {"x": state["x"], **_reports(infos)}
    if kind == "2d":
        x = state["x"].zero_()
        hx, hy = _spacings(c)
        info = hj.solve_2d(state["f"], x, hx=hx, hy=hy, tile=(c["tx"], c["ty"]), s=c["s"], overlap=(c["ox"], c["oy"]),
                           method=c["method"], rel_tol=c["tol"], max_cycles=c["cap"], allow_not_converged=True)
        return {"x": x, **_report(info)}
    if kind == "refined":
        x = state["x"].zero_()
        info = hj.solve_2d_refined(state["f"], x, 1.0 / (c["n"] + 1), tile=(c["tx"], c["ty"]), s=c["s"],
                                   overlap=(c["o"], c["o"]), rel_tol=c["tol"], inner_max_cycles=c["cap"], max_outer=3,
                                   allow_not_converged=True)
        return {"x": x, "outer": info.outer, "inner_cycles": info.inner_cycles, "fp64_cycles": info.fp64_cycles}
    if kind == "batch":
        for x in state["x"]:
            x.zero_()
        infos = hj.solve_batched(state["table"], rel_tol=c["tol"], tile=(c["tx"], c["ty"]), s=c["s"], overlap=(c["o"], c["o"]),
                                 tile_1d=c["t1"], s_1d=c["s1"], overlap_1d=c["o1"], max_cycles=c["cap"], refine=c["refine"],
                                 allow_not_converged=True)
        return {"x": list(state["x"]), **_reports(infos)}
    if kind == "vc":
        x = state["x"].zero_()
        infos = hj.solve_vc_2d(state["a"], state["f"], x, hx=1.0 / (c["nx"] + 1), hy=1.0 / (c["ny"] + 1),
                               tile=(c["tx"], c["ty"]), s=c["s"], overlap=(c["o"], c["o"]), rel_tol=c["tol"],
                               max_cycles=c["cap"], allow_not_converged=True)
        return {"x": x, **_reports(infos)}
    u = hj.diffusion_solve(state["f"], state["a"], 1.0 / (c["n"] + 1), tile=(c["tx"], c["ty"]), s=c["s"],
                           overlap=(c["o"], c["o"]), rel_tol=c["tol"], max_cycles=c["cap"])
    loss = torch.mean((u - state["t"]) ** 2)
    gf, ga = torch.autograd.grad(loss, (state["f"], state["a"]))
    return {"u": u, "grad_f": gf, "grad_a": ga}


def work(case):
    """Bytes: the inputs once, the results once.  Flops: 6 a point and sweep (10 with coefficients of its own)."""
    c, kind = case, case["kind"]
    es = 4 if c.get("dtype") == "f32" else 8
    sweeps = c["cycles"] * c.get("s", 1)
    if kind == "1d":
        return {"bytes": 24 * c["n"], "flops": 4 * c["n"] * sweeps}
    if kind == "1d_batch":
        pts = c["n"] * c["copies"]
        return {"bytes": 24 * pts, "flops": 4 * pts * sweeps}
    if kind == "2d":
        pts = c["nx"] * c["ny"]
        return {"bytes": 3 * es * pts, "flops": 6 * pts * (c["cycles"] if c["method"] == "global" else sweeps)}
    if kind == "refined":
        return {"bytes": 24 * c["n"] ** 2, "flops": 6 * c["n"] ** 2 * sweeps}
    if kind == "batch":
        sides, ns = _batch_sizes(c)
        p2, p1 = sum(n * n for n in sides), sum(ns)
        return {"bytes": 3 * es * (p2 + p1), "flops": c["cycles"] * (6 * p2 * c["s"] + 4 * p1 * c["s1"])}
    nx, ny = (c["n"], c["n"]) if kind == "vc_train" else (c["nx"], c["ny"])
    pts = nx * ny * c["batch"]
    if kind == "vc":
        return {"bytes": 24 * pts + 8 * nx * ny, "flops": 10 * pts * sweeps}
    return {"bytes": 2 * 24 * pts + 16 * nx * ny, "flops": 2 * 10 * pts * sweeps}


# ---------------------------------------------------------------- the same in plain torch, 64 bits
def _axis(n, t, o):
    """Tiles of an axis (first points), their extent, and for each point its tile and its place in it."""
    ext = min(n, t)
    first = [0]
    while first[-1] + ext < n:
        first.append(min(first[-1] + ext - o, n - ext))
    begin = [0] + [b + (a + ext - b + 1) // 2 for a, b in zip(first, first[1:])] + [n]
    tile = np.repeat(np.arange(len(first)), np.diff(begin))
    return first, ext, tile, np.arange(n) - np.array(first)[tile]


class _Cycle:
    """One cycle on a 2D grid (1D: one row, wy = 0): every tile with its frozen halo, s sweeps, the owned points back."""

    def __init__(self, f, wx, wy, tile, s, overlap):
        ny, nx = f.shape
        self.f, self.wx, self.wy, self.s = f, wx, wy, s
        self.exact = all(n <= t or o >= 2 * s - 2 for n, t, o in zip((nx, ny), tile, overlap))
        if self.exact:
            return
        idx = lambda v: torch.as_tensor(np.asarray(v), device=f.device)  # noqa: E731
        fx, ex, tx, px = _axis(nx, tile[0], overlap[0])
        fy, ey, ty, py = _axis(ny, tile[1], overlap[1])
        self.rows = idx(np.array(fy)[:, None] + np.arange(ey + 2))[:, None, :, None]
        self.cols = idx(np.array(fx)[:, None] + np.arange(ex + 2))[None, :, None, :]
        self.back = (idx(ty)[:, None], idx(tx)[None, :], idx(py)[:, None], idx(px)[None, :])
        pad = torch.nn.functional.pad(f, (1, 1, 1, 1))
        self.ft = pad[self.rows, self.cols][..., 1:-1, 1:-1].contiguous()

    def _sweep(self, x, f):
        """The new interior of arrays x with a halo of one."""
        wx, wy = self.wx, self.wy
        v = wx * (x[..., 1:-1, :-2] + x[..., 1:-1, 2:])
        v = v + wy * (x[..., :-2, 1:-1] + x[..., 2:, 1:-1])
        return (f + v) / (2 * wx + 2 * wy)

    def __call__(self, x):
        pad = torch.nn.functional.pad(x, (1, 1, 1, 1))
        if self.exact:
            for _ in range(self.s):
                pad[1:-1, 1:-1] = self._sweep(pad, self.f)
            return pad[1:-1, 1:-1].clone()
        t = pad[self.rows, self.cols]
        for _ in range(self.s):
            t[..., 1:-1, 1:-1] = self._sweep(t, self.ft)
        return t[..., 1:-1, 1:-1][self.back]

    def residual(self, x):
        p = torch.nn.functional.pad(x, (1, 1, 1, 1))
        ax = self.wx * ((2 * x - p[1:-1, :-2]) - p[1:-1, 2:]) + self.wy * ((2 * x - p[:-2, 1:-1]) - p[2:, 1:-1])
        return float(torch.linalg.vector_norm(self.f - ax))


def _iterate(cycle, residual, x, tol, cap):
    """x after the first cycle whose residual meets tol (tol <= 0: after cap cycles), and what the library reports."""
    r0 = r = residual(x)
    c = 0
    while c < cap and (tol <= 0.0 or r > tol * r0):
        x = cycle(x)
        c += 1
        if tol > 0.0 or c == cap:
            r = residual(x)
    return x, c, r / r0, r0


def _exact_grid(f, hx, hy, tile, s, overlap, tol, cap):
    """hy = None: f is a vector, solved as one row with no coupling in y."""
    if hy is None:
        x, c, rel, r0 = _exact_grid(f[None], hx, math.inf, (tile, 1), s, (overlap, 0), tol, cap)
        return x[0], c, rel, r0
    cyc = _Cycle(f, 1.0 / hx ** 2, 1.0 / hy ** 2, tile, s, overlap)
    return _iterate(cyc, cyc.residual, torch.zeros_like(f), tol, cap)


def _faces(a, hx, hy):
    w = 0.5 * (a[1:-1, 1:-1] + a[1:-1, :-2]) / hx ** 2
    e = 0.5 * (a[1:-1, 1:-1] + a[1:-1, 2:]) / hx ** 2
    s = 0.5 * (a[1:-1, 1:-1] + a[:-2, 1:-1]) / hy ** 2
    n = 0.5 * (a[1:-1, 1:-1] + a[2:, 1:-1]) / hy ** 2
    return w, e, s, n


def _exact_vc(c, f, a):
    """All right-hand sides of a forward solve together; a cycle that equals s sweeps of the whole grid only."""
    w, e, s, n = _faces(a, 1.0 / (c["nx"] + 1), 1.0 / (c["ny"] + 1))
    d = w + e + s + n

    def around(x):
        p = torch.nn.functional.pad(x, (1, 1, 1, 1))
        return w * p[..., 1:-1, :-2] + e * p[..., 1:-1, 2:] + s * p[..., :-2, 1:-1] + n * p[..., 2:, 1:-1]

    def norms(x):
        return torch.linalg.vector_norm(f - (d * x - around(x)), dim=(1, 2))

    x = torch.zeros_like(f)
    r0 = norms(x)
    out, rel = x.clone(), torch.ones_like(r0)
    cycles = torch.full(r0.shape, c["cap"], device=DEV, dtype=torch.int64)
    live = torch.ones_like(r0, dtype=torch.bool)
    for k in range(1, c["cap"] + 1):
        for _ in range(c["s"]):
            x = (f + around(x)) / d
        r = norms(x) / r0
        out = torch.where(live[:, None, None], x, out)
        rel = torch.where(live, r, rel)
        met = live & (r <= c["tol"])
        cycles[met] = k
        live = live & ~met
        if not bool(live.any()):
            break
    return {"x": out, "cycles": cycles.cpu().numpy(), "rel_residual": rel.cpu().numpy(), "r0_norm": r0.cpu().numpy()}


def _exact_train(c, f, a, t):
    """u, dL/df and dL/da by a dense solve and torch's own gradients, on the host."""
    n, h = c["n"], 1.0 / (c["n"] + 1)
    f, a, t = f.detach().cpu().requires_grad_(True), a.detach().cpu().requires_grad_(True), t.cpu()
    w, e, s, no = _faces(a, h, h)
    at = torch.arange(n * n).reshape(n, n)
    m = torch.zeros(n * n, n * n, dtype=F64)
    m = m.index_put((at.reshape(-1), at.reshape(-1)), (w + e + s + no).reshape(-1))
    m = m.index_put((at[:, 1:].reshape(-1), at[:, :-1].reshape(-1)), -w[:, 1:].reshape(-1))
    m = m.index_put((at[:, :-1].reshape(-1), at[:, 1:].reshape(-1)), -e[:, :-1].reshape(-1))
    m = m.index_put((at[1:].reshape(-1), at[:-1].reshape(-1)), -s[1:].reshape(-1))
    m = m.index_put((at[:-1].reshape(-1), at[1:].reshape(-1)), -no[:-1].reshape(-1))
    u = torch.linalg.solve(m, f.reshape(c["batch"], -1).T).T.reshape(f.shape)
    gf, ga = torch.autograd.grad(torch.mean((u - t) ** 2), (f, a))
    return {"u": u.detach(), "grad_f": gf, "grad_a": ga}


def exact(case, seed):
    c, kind = case, case["kind"]
    v = _inputs(c, seed)
    if kind == "1d":
        x, k, rel, r0 = _exact_grid(v, 1.0 / (c["n"] + 1), None, c["tile"], c["s"], c["overlap"], c["tol"], c["cap"])
        return {"x": x, "cycles": k, "rel_residual": rel, "r0_norm": r0}
    if kind == "1d_batch":
        # every cycle is s classical sweeps; all copies at once, each kept where it stops
        h2 = (1.0 / (c["n"] + 1)) ** 2
        if c["overlap"] < 2 * c["s"] - 2:
            return None
        pad = torch.nn.functional.pad(torch.ones_like(v), (1, 1))
        hf = h2 * v

        def norms():
            return torch.linalg.vector_norm(v - ((2 * pad[:, 1:-1] - pad[:, :-2]) - pad[:, 2:]) / h2, dim=1)

        r0 = norms()
        out, rel = pad[:, 1:-1].clone(), torch.ones_like(r0)
        cycles = torch.full(r0.shape, c["cap"], device=DEV, dtype=torch.int64)
        live = torch.ones_like(r0, dtype=torch.bool)
        for k in range(1, c["cap"] + 1):
            for _ in range(c["s"]):
                pad[:, 1:-1] = (hf + (pad[:, :-2] + pad[:, 2:])) * 0.5
            r = norms() / r0
            met = live & (r <= c["tol"])
            last = live if k == c["cap"] else met
            if bool(last.any()):
                out[last] = pad[:, 1:-1][last]
                rel = torch.where(last, r, rel)
                cycles[last] = k
            live = live & ~met
            if not bool(live.any()):
                break
        return {"x": out, "cycles": cycles.cpu().numpy(), "rel_residual": rel.cpu().numpy(), "r0_norm": r0.cpu().numpy()}
    if kind == "2d":
        hx, hy = _spacings(c)
        tile, s, ov = (c["tx"], c["ty"]), c["s"], (c["ox"], c["oy"])
        if c["method"] == "global":
            tile, s, ov = (c["nx"], c["ny"]), 1, (0, 0)
        x, k, rel, r0 = _exact_grid(v.to(F64), hx, hy, tile, s, ov, c["tol"], c["cap"])
        single = c["dtype"] == "f32"  # single precision has a residual of its own
        return {"x": x, "cycles": k, "rel_residual": None if single else rel, "r0_norm": r0}
    if kind == "refined":
        n = c["n"]
        k, l, a, sx, sy = _mode_tables(n, n, c["modes"], np.random.default_rng(seed))
        lam = (4 * (n + 1) ** 2) * (torch.sin(math.pi * k / (2 * (n + 1))) ** 2 + torch.sin(math.pi * l / (2 * (n + 1))) ** 2)
        return {"x": (sy.T * (a / lam)[None, :]) @ sx, "outer": None, "inner_cycles": None, "fp64_cycles": None}
    if kind == "batch":
        xs, infos = [], []
        for f in v:
            h = 1.0 / (f.shape[-1] + 1)
            shape = ((c["tx"], c["ty"]), c["s"], (c["o"], c["o"])) if f.dim() == 2 else (c["t1"], c["s1"], c["o1"])
            x, *info = _exact_grid(f.to(F64), h, h if f.dim() == 2 else None, *shape, c["tol"], c["cap"])
            xs.append(x)
            infos.append(info)
        single = c["dtype"] == "f32"
        return {"x": xs, "cycles": np.array([i[0] for i in infos]),
                "rel_residual": None if single else np.array([i[1] for i in infos]),
                "r0_norm": np.array([i[2] for i in infos])}
    if kind == "vc":
        if not all(n <= t or c["o"] >= 2 * c["s"] - 2 for n, t in ((c["nx"], c["tx"]), (c["ny"], c["ty"]))):
            return None
        return _exact_vc(c, *v)
    return _exact_train(c, *v)
