"""Performance cases of the solver: what a program that uses it has it do, through the binding's
public entry points, from the smallest calls to the largest grids.

Four kinds of work:
  step      the explicit solve of one problem: (new depth,) start step, leapfrog steps, snapshot;
  family    the same for several regularisations held in one batched context;
  gradient  misfit of receiver traces and its gradient with respect to the nodal depth
            (FdwMisfit: traced forward run with checkpoints, reverse sweep);
  implicit  the factorized implicit scheme (the paper's Section 4, Table 1 workload: 100 steps).

listed() holds the cases; draw() gives more of the same ranges; prepare() / run() set one up and
make one pass; work() counts what a pass cannot do without; exact() is the same result in FP64
from plain torch.
"""
import math

import torch

_REAL = {"f32": torch.float32, "f64": torch.float64}


def listed():
    return [
        # a few steps on a small grid: an interactive or coupled program that looks at every state
        dict(name="short64_f64", kind="step", nx=64, ny=64, steps=10, dtype="f64", energy=False, graph=False,
             face=False, recoeff=False),
        # the 256^2 FP64 line-singularity workload with the energy of every step, replayed from a graph
        dict(name="line256_f64", kind="step", nx=256, ny=256, steps=1000, dtype="f64", energy=True, graph=True,
             face=False, recoeff=False),
        # one solve of an anisotropic problem (separate h2) on a ragged mid-size grid
        dict(name="face1531x1177_f32", kind="step", nx=1531, ny=1177, steps=300, dtype="f32", energy=False,
             graph=False, face=True, recoeff=True),
        # FP64 solve at 2048^2: the forward part of the gradient workload's size
        dict(name="solve2048_f64", kind="step", nx=2048, ny=2048, steps=400, dtype="f64", energy=False, graph=False,
             face=False, recoeff=True),
        # the headline grid: 8192^2 FP32, energies of every step, a depth of its own per solve
        dict(name="solve8192_f32", kind="step", nx=8192, ny=8192, steps=400, dtype="f32", energy=True, graph=False,
             face=False, recoeff=True),
        # a batch of regularisations on grids of several sizes in one context
        dict(name="family2048_f32", kind="family", n=2048, members=8, steps=200, dtype="f32", energy=True),
        # gradient evaluations of an inversion: coarse grid, the 2048^2 FP64 workload, a ragged FP32 one
        dict(name="grad384_f64", kind="gradient", nx=384, ny=384, steps=500, dtype="f64", receivers=64, ckpt=64),
        dict(name="grad2048_f64", kind="gradient", nx=2048, ny=2048, steps=640, dtype="f64", receivers=64, ckpt=64),
        dict(name="grad1801x1403_f32", kind="gradient", nx=1801, ny=1403, steps=500, dtype="f32", receivers=37,
             ckpt=50),
        # Table 1 of the paper: 100 implicit steps at the smallest and the largest of its grids, and
        # between them on a grid that is no power of two
        dict(name="implicit256_f64", kind="implicit", nx=256, ny=256, steps=100, dtype="f64"),
        dict(name="implicit1000x1500_f32", kind="implicit", nx=1000, ny=1500, steps=100, dtype="f32"),
        dict(name="implicit4096_f64", kind="implicit", nx=4096, ny=4096, steps=100, dtype="f64"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: sizes over the logarithm of their range, odd ones among them; a pass costs at
    most about what the largest listed cases cost (nodes x steps is bounded per kind)."""
    kind = rng.choice(["step", "step", "step", "family", "gradient", "gradient", "implicit", "implicit"])
    dtype = rng.choice(["f32", "f64"])
    if kind == "step":
        n = _log_int(rng, 40, 8192 if dtype == "f32" else 5600)
        nx = max(33, min(8192, int(n * rng.uniform(0.7, 1.4))))
        ny = max(33, min(8192, int(n * rng.uniform(0.7, 1.4))))
        cap = (2.2e10 if dtype == "f32" else 1.1e10) / (nx * ny)
        steps = max(5, min(_log_int(rng, 8, 1000), int(cap)))
        graph = n < 1200 and rng.random() < 0.4
        return dict(kind=kind, nx=nx, ny=ny, steps=steps, dtype=dtype, energy=rng.random() < 0.5, graph=graph,
                    face=rng.random() < 0.3, recoeff=not graph and rng.random() < 0.7)
    if kind == "family":
        return dict(kind=kind, n=_log_int(rng, 200, 2048), members=rng.randint(2, 8), steps=_log_int(rng, 30, 200),
                    dtype=dtype, energy=rng.random() < 0.6)
    if kind == "gradient":
        n = _log_int(rng, 64, 2000)
        nx, ny = max(50, int(n * rng.uniform(0.75, 1.3))), max(50, int(n * rng.uniform(0.75, 1.3)))
        steps = max(20, min(_log_int(rng, 60, 640), int(2.6e9 / (nx * ny))))
        return dict(kind=kind, nx=nx, ny=ny, steps=steps, dtype=dtype, receivers=_log_int(rng, 1, 200),
                    ckpt=rng.choice([16, 32, 50, 64, 100]))
    n = _log_int(rng, 100, 3900)
    nx, ny = max(64, min(4096, int(n * rng.uniform(0.7, 1.4)))), max(64, min(4096, int(n * rng.uniform(0.7, 1.4))))
    return dict(kind=kind, nx=nx, ny=ny, steps=max(10, min(100, int(1.6e9 / (nx * ny)))), dtype=dtype)


# --------------------------------------------------------------------------------------
# Inputs (seeded, made on the GPU): [-1, 1]^2 for the explicit kinds, [0, 100]^2 for the implicit one
# --------------------------------------------------------------------------------------
def _gen(seed, salt=0):
    return torch.Generator(device="cuda").manual_seed(1000003 * seed + salt)


def _uniform(g, n, lo, hi):
    return (lo + (hi - lo) * torch.rand(n, generator=g, device="cuda", dtype=torch.float64)).tolist()


def _axes(nx, ny, lo, hi):
    x = torch.linspace(lo, hi, nx, device="cuda", dtype=torch.float64)[None, :]
    y = torch.linspace(lo, hi, ny, device="cuda", dtype=torch.float64)[:, None]
    return x, y


def _smooth_field(nx, ny, g):
    """A smooth random field in [0, 1]: a few seeded plane waves."""
    x, y = _axes(nx, ny, -1.0, 1.0)
    f = torch.zeros((ny, nx), device="cuda", dtype=torch.float64)
    p = _uniform(g, 15, -1.0, 1.0)
    for a, b, c in zip(p[0::3], p[1::3], p[2::3]):
        f += torch.cos(9.0 * a * x + 9.0 * b * y + 3.0 * c)
    f -= f.min()
    return f / f.max().clamp_min(1e-12)


def _depth(nx, ny, g, kind):
    """Regularised singular depth: a smooth bathymetry with a mollified line, jump or point."""
    x, y = _axes(nx, ny, -1.0, 1.0)
    c, w = _uniform(g, 2, 0.0, 1.0)
    eps = max(0.05 * (0.4 + w), 4.0 / nx)
    s = (x - 0.6 * (c - 0.5)).expand(ny, nx)
    if kind == "line":
        sing = 2.0 * torch.exp(-(s * s) / (2 * eps * eps)) / (eps * math.sqrt(2 * math.pi))
    elif kind == "jump":
        sing = 1.5 * (1.0 + torch.erf(s / (eps * math.sqrt(2.0))))
    else:
        sing = 5.0 * torch.exp(-(s * s + y * y) / (2 * eps * eps)) / (2 * math.pi * eps * eps)
    return 0.6 + 0.4 * _smooth_field(nx, ny, g) + sing


def _humps(nx, ny, g, lo, hi, count, width, amp):
    x, y = _axes(nx, ny, lo, hi)
    c = _uniform(g, 2 * count, lo + 0.2 * (hi - lo), lo + 0.8 * (hi - lo))
    u = torch.zeros((ny, nx), device="cuda", dtype=torch.float64)
    for cx, cy in zip(c[0::2], c[1::2]):
        u += amp * torch.exp(-((x - cx) ** 2 + (y - cy) ** 2) / (width * width))
    u[0], u[-1], u[:, 0], u[:, -1] = 0.0, 0.0, 0.0, 0.0
    return u


def _explicit_data(nx, ny, seed, dtype, shape="line", face=False, m=0):
    """(tau, u0, u1, h1, h2 or None) of one explicit problem, in the storage type."""
    g = _gen(seed, 17 * m + 1)
    real = _REAL[dtype]
    h1 = _depth(nx, ny, g, shape)
    h2 = _depth(nx, ny, g, "jump") if face else None
    dx, dy = 2.0 / (nx - 1), 2.0 / (ny - 1)
    hmax = max(float(h1.max()), float(h2.max()) if face else 0.0)
    tau = 0.5 * min(dx, dy) / math.sqrt(hmax)
    u0 = _humps(nx, ny, g, -1.0, 1.0, 4, 0.05 + 2.0 / min(nx, ny), 1.0)
    u1 = 0.1 * _humps(nx, ny, g, -1.0, 1.0, 2, 0.1 + 2.0 / min(nx, ny), 1.0)
    return tau, u0.to(real), u1.to(real), h1.to(real), None if h2 is None else h2.to(real)


def _family_shapes(case):
    """Members of several sizes, as a study over regularisations and resolutions has them."""
    n = case["n"]
    sizes = (n, max(64, n // 2), max(64, (3 * n) // 4 - 1), max(64, n // 4))
    return [(sizes[m % 4], sizes[m % 4], ("line", "jump", "point")[m % 3]) for m in range(case["members"])]


def _implicit_data(case, seed):
    """The Table 1 problem on [0, 100]^2: depth 100 | 10 with a mollified jump, a hump of amplitude
    50, time step 0.05; the jump's place, the bathymetry and the hump come from the seed."""
    nx, ny, real = case["nx"], case["ny"], _REAL[case["dtype"]]
    g = _gen(seed, 2)
    x, y = _axes(nx, ny, 0.0, 100.0)
    c, e = _uniform(g, 2, 0.0, 1.0)
    s = (x - (65.0 + 20.0 * c)) / (0.8 * (0.5 + e))
    h = 10.0 + 90.0 * 0.5 * (1.0 - torch.erf(s)).expand(ny, nx) + 5.0 * _smooth_field(nx, ny, g)
    u0 = _humps(nx, ny, g, 0.0, 100.0, 1, math.sqrt(8.0), 50.0)
    u1 = _humps(nx, ny, g, 0.0, 100.0, 1, 5.0, 1.0)
    return 0.05, u0.to(real), u1.to(real), h.to(real)


def _gradient_data(case, seed):
    """The explicit problem with one more hump on the receivers' row (a regularised line makes the
    time step so small that the others would not reach it), distinct receivers on that row, and
    observed traces: a wavelet of an arrival time of its own at every receiver."""
    nx, ny, N = case["nx"], case["ny"], case["steps"]
    tau, u0, u1, h, _ = _explicit_data(nx, ny, seed, case["dtype"])
    g = _gen(seed, 5)
    x, y = _axes(nx, ny, -1.0, 1.0)
    cx = _uniform(g, 1, -0.6, 0.6)[0]
    hump = torch.exp(-((x - cx) ** 2 + (y - 0.3) ** 2) / (0.1 + 2.0 / min(nx, ny)) ** 2)
    hump[0], hump[-1], hump[:, 0], hump[:, -1] = 0.0, 0.0, 0.0, 0.0
    u0 = (u0.double() + hump).to(u0.dtype)
    R = min(case["receivers"], nx - 4)
    cols = torch.randperm(nx - 4, generator=g, device="cuda")[:R].to(torch.int32) + 2
    rec = torch.stack([cols, torch.full_like(cols, int(0.65 * (ny - 1)))], dim=1).contiguous()
    t0 = torch.rand(R, generator=g, device="cuda", dtype=torch.float64) * N
    k = torch.arange(N + 1, device="cuda", dtype=torch.float64)[:, None]
    d = 0.3 * torch.exp(-(((k - t0[None, :]) / (0.05 * N + 3.0)) ** 2))
    return tau, u0, u1, h, rec, d


# --------------------------------------------------------------------------------------
# One pass through the public entry points
# --------------------------------------------------------------------------------------
def prepare(case, seed):
    from paper_2005_11931_amd import fdw

    code = fdw.FDW_F32 if case["dtype"] == "f32" else fdw.FDW_F64
    kind = case["kind"]
    if kind == "step":
        tau, u0, u1, h1, h2 = _explicit_data(case["nx"], case["ny"], seed, case["dtype"],
                                             "point" if case["nx"] >= 4096 else "line", case["face"])
        s = fdw.Solver([fdw.problem(case["nx"], case["ny"], tau, case["steps"], code)], [u0], [u1])
        s.set_coeff(h1, h2)
        e = None
        if case["graph"]:
            s.configure(fdw.FDW_CFG_USE_GRAPH, 1)
            if case["energy"]:
                e = torch.empty((1, case["steps"]), dtype=torch.float64, device="cuda")
        return dict(case=case, s=s, h1=h1, h2=h2, e=e)
    if kind == "family":
        data = [_explicit_data(nx, ny, seed, case["dtype"], shape, m=m)
                for m, (nx, ny, shape) in enumerate(_family_shapes(case))]
        s = fdw.Solver([fdw.problem(d[1].shape[1], d[1].shape[0], d[0], case["steps"], code) for d in data],
                       [d[1] for d in data], [d[2] for d in data])
        for m, d in enumerate(data):
            s.set_coeff(d[3], member=m)
        return dict(case=case, s=s)
    if kind == "gradient":
        tau, u0, u1, h, rec, d = _gradient_data(case, seed)
        s = fdw.Solver([fdw.problem(case["nx"], case["ny"], tau, case["steps"], code)], [u0], [u1])
        return dict(case=case, s=s, h=h.clone().requires_grad_(True), rec=rec, d=d)
    tau, u0, u1, h = _implicit_data(case, seed)
    p = fdw.problem(case["nx"], case["ny"], tau, case["steps"], code, 0.0, 100.0, 0.0, 100.0)
    return dict(case=case, s=fdw.ImplicitSolver(p, 0.25, u0, u1, h))


def run(state):
    from paper_2005_11931_amd import fdw

    case, s = state["case"], state["s"]
    kind = case["kind"]
    if kind == "step":
        if case["recoeff"]:
            s.set_coeff(state["h1"], state["h2"])
        else:
            s.reset()
        if state["e"] is not None:
            s.step_into(case["steps"], state["e"])
            e = state["e"]
        else:
            e = s.step(case["steps"], energy=case["energy"])
        u, du, _ = s.get_state()
        return dict(u=u, du=du, energy=e)
    if kind == "family":
        for m in range(case["members"]):
            s.reset(m)
        e = s.step(case["steps"], energy=case["energy"])
        return dict(energy=e, states=[s.get_state(m)[:2] for m in range(case["members"])])
    if kind == "gradient":
        loss = fdw.FdwMisfit.apply(state["h"], s, state["rec"], state["d"], case["ckpt"])
        (grad,) = torch.autograd.grad(loss, state["h"])
        return dict(loss=loss.detach(), grad=grad)
    s.reset()
    s.step(case["steps"])
    u, du, _ = s.get_state()
    return dict(u=u, du=du)


def work(case):
    """Bytes: each input field read and each output written once.  Operations: per node and step 10
    for the leapfrog update and 4 for its energy term; per node and step of a gradient two forward
    recurrences, the adjoint one and the face products (44); per node and implicit step the
    right-hand side and two line solves (50)."""
    w = 4 if case["dtype"] == "f32" else 8
    if case["kind"] == "family":
        nodes = sum(nx * ny for nx, ny, _ in _family_shapes(case))
    else:
        nodes = case["nx"] * case["ny"]
    per = {"step": 10, "family": 10, "gradient": 44, "implicit": 50}[case["kind"]]
    fields = {"step": 5, "family": 5, "gradient": 4, "implicit": 5}[case["kind"]]
    extra = 0
    if case.get("energy"):
        per += 4
        extra = 8 * case["steps"] * case.get("members", 1)
    if case.get("face"):
        fields += 1
    if case["kind"] == "gradient":
        extra = 8 * (case["steps"] + 1) * case["receivers"]
    return {"bytes": nodes * w * fields + extra, "flops": nodes * case["steps"] * per}


# --------------------------------------------------------------------------------------
# The same results in FP64 from plain torch
# --------------------------------------------------------------------------------------
class _Operator:
    """tau^2 A with face coefficients and zero Dirichlet data, on [ny][nx] FP64 planes."""

    def __init__(self, h1, h2, tau, dx, dy):
        self.ax, self.ay = 0.5 * tau * tau / (dx * dx), 0.5 * tau * tau / (dy * dy)
        self.fx = self.ax * (h1[:, 1:] + h1[:, :-1])
        self.fy = self.ay * (h2[1:] + h2[:-1])

    def __call__(self, u):
        f = (u[:, 1:] - u[:, :-1]).mul_(self.fx)
        g = (u[1:] - u[:-1]).mul_(self.fy)
        out = torch.zeros_like(u)
        out[1:-1, 1:-1] = (f[1:-1, 1:] - f[1:-1, :-1]) + (g[1:, 1:-1] - g[:-1, 1:-1])
        return out


def _exact_forward(case, steps, data, box=2.0, energy=False, every=None):
    tau, u0, u1, h1, h2 = [None if v is None else v if isinstance(v, float) else v.double() for v in data]
    dx, dy = box / (u0.shape[1] - 1), box / (u0.shape[0] - 1)
    A = _Operator(h1, h1 if h2 is None else h2, tau, dx, dy)
    u, d = u0.clone(), None
    E = []
    for n in range(steps):
        if every is not None:
            every(n, u)
        L = A(u)
        if n == 0:
            d = tau * u1 + 0.5 * L
            d[0], d[-1], d[:, 0], d[:, -1] = 0.0, 0.0, 0.0, 0.0
        else:
            d += L
        u = u + d
        if energy:
            E.append((d * d - u * L).sum() * (dx * dy / (tau * tau)))
    if every is not None:
        every(steps, u)
    return A, u, d, torch.stack(E)[None, :] if energy else None


def _line_solver(F, g, dim):
    """x of (I - g d(F d .)) x = r along dim by parallel cyclic reduction, interior unknowns."""
    F = F.transpose(0, 1) if dim == 0 else F
    lo, up = -g * F[:, :-1], -g * F[:, 1:]
    b = 1.0 - lo - up
    a, c = lo.clone(), up.clone()
    a[:, 0], c[:, -1] = 0.0, 0.0
    n, s, levels = b.shape[1], 1, []

    def shift(v, k, fill):
        out = torch.full_like(v, fill)
        if k > 0:
            out[:, k:] = v[:, :-k]
        else:
            out[:, :k] = v[:, -k:]
        return out

    while s < n:
        al, ga = -a / shift(b, s, 1.0), -c / shift(b, -s, 1.0)
        b = b + al * shift(c, s, 0.0) + ga * shift(a, -s, 0.0)
        a, c = al * shift(a, s, 0.0), ga * shift(c, -s, 0.0)
        levels.append((s, al[:, s:].contiguous(), ga[:, :-s].contiguous()))
        s *= 2

    def solve(r):
        r = (r.transpose(0, 1) if dim == 0 else r).contiguous()
        for k, al, ga in levels:
            q = r.clone()
            q[:, k:] += al * r[:, :-k]
            q[:, :-k] += ga * r[:, k:]
            r = q
        r = r / b
        return r.transpose(0, 1) if dim == 0 else r

    return solve


def _exact_implicit(case, seed):
    tau, u0, u1, h = [v if isinstance(v, float) else v.double() for v in _implicit_data(case, seed)]
    dx, dy = 100.0 / (case["nx"] - 1), 100.0 / (case["ny"] - 1)
    A = _Operator(h, h, tau, dx, dy)
    hx, hy = 0.5 * (h[:, 1:] + h[:, :-1]), 0.5 * (h[1:] + h[:-1])
    sx = _line_solver(hx[1:-1], 0.25 * tau * tau / (dx * dx), 1)
    sy = _line_solver(hy[:, 1:-1], 0.25 * tau * tau / (dy * dy), 0)
    u, d = u0.clone(), None
    for n in range(case["steps"]):
        w = torch.zeros_like(u)
        w[1:-1, 1:-1] = sy(sx(A(u)[1:-1, 1:-1]))
        if n == 0:
            d = tau * u1 + 0.5 * w
            d[0], d[-1], d[:, 0], d[:, -1] = 0.0, 0.0, 0.0, 0.0
        else:
            d = d + w
        u = u + d
    return dict(u=u, du=d)


def _exact_gradient(case, seed):
    tau, u0, u1, h, rec, d = _gradient_data(case, seed)
    N, col, row = case["steps"], rec[:, 0].long(), rec[:, 1].long()
    us = torch.empty((N,) + tuple(u0.shape), dtype=torch.float64, device="cuda")
    tr = torch.empty_like(d)

    def every(n, u):
        tr[n] = u[row, col]
        if n < N:
            us[n] = u

    A, _, _, _ = _exact_forward(case, N, (tau, u0, u1, h, None), every=every)
    e = tr - d
    src = torch.zeros_like(u0, dtype=torch.float64)
    src[row, col] = 2.0 * e[N]
    lam, mu = src.clone(), src.clone()
    sx, sy = torch.zeros_like(A.fx), torch.zeros_like(A.fy)
    for n in range(N - 1, -1, -1):
        w, u = (0.5 if n == 0 else 1.0), us[n]
        sx.addcmul_(u[:, 1:] - u[:, :-1], lam[:, 1:] - lam[:, :-1], value=w)
        sy.addcmul_(u[1:] - u[:-1], lam[1:] - lam[:-1], value=w)
        mu = mu + A(lam)
        mu[row, col] += 2.0 * e[n]
        lam = lam + mu
    grad = torch.zeros_like(u0, dtype=torch.float64)
    grad[:, :-1] -= A.ax * sx
    grad[:, 1:] -= A.ax * sx
    grad[:-1] -= A.ay * sy
    grad[1:] -= A.ay * sy
    return dict(loss=(e * e).sum(), grad=grad)


def exact(case, seed):
    kind = case["kind"]
    if kind == "step":
        data = _explicit_data(case["nx"], case["ny"], seed, case["dtype"],
                              "point" if case["nx"] >= 4096 else "line", case["face"])
        _, u, d, E = _exact_forward(case, case["steps"], data, energy=case["energy"])
        return dict(u=u, du=d, energy=E)
    if kind == "family":
        out = [_exact_forward(case, case["steps"], _explicit_data(nx, ny, seed, case["dtype"], shape, m=m),
                              energy=case["energy"])
               for m, (nx, ny, shape) in enumerate(_family_shapes(case))]
        return dict(energy=torch.cat([o[3] for o in out]) if case["energy"] else None,
                    states=[(o[1], o[2]) for o in out])
    if kind == "gradient":
        return _exact_gradient(case, seed)
    return _exact_implicit(case, seed)
