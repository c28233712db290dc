"""The calls this library's performance is judged on, and what their results
should be.

Each case is one call of the public Python entry points on a seeded problem:
`vjp` (a forward sweep, the loss, the recomputations its budget forces and the
reverse sweep) or `forward` (the program alone). The listed cases are the
workloads of paper_2509_02197_amd/workloads.py and of the committed profiles
(constants' gradients, limiter), with odd and single-precision grids beside
them; `draw` spreads over the same kinds, types, options and sizes.

`exact` evaluates the same program with plain torch operations in 64 bits.
"""
import math

import numpy as np
import torch

import paper_2509_02197_amd as adst

KINDS = {"jacobi": adst.ADST_JACOBI2D5, "allencahn": adst.ADST_ALLENCAHN3D7,
         "vardiff": adst.ADST_VARDIFF2D9, "gs": adst.ADST_GAUSSSEIDEL2D5}
LOSSES = {"half_sq": adst.ADST_LOSS_HALF_SQ, "dot_w": adst.ADST_LOSS_DOT_W,
          "half_sq_diff": adst.ADST_LOSS_HALF_SQ_DIFF, "seed": adst.ADST_LOSS_SEED}
SCHEDS = {"auto": adst.ADST_SCHED_AUTO, "store_all": adst.ADST_SCHED_STORE_ALL,
          "uniform": adst.ADST_SCHED_UNIFORM, "binomial": adst.ADST_SCHED_BINOMIAL}
# The constants the calls leave at their defaults, and the limiter's bounds.
PARAMS = {"jacobi": (0.2, 0.0), "allencahn": (0.1, 0.1), "vardiff": (0.1, 0.0), "gs": (0.2, 0.0)}
BOUNDS = {"jacobi": (0.3, 0.7), "allencahn": (-0.9, 0.9), "vardiff": (0.3, 0.7)}
DEVICE = "cuda"


def _case(name, kind, dtype, shape, steps, loss="half_sq", slots=0, sched="auto", op="vjp",
          dk=False, dparams=False, limit=False):
    c = {"op": op, "kind": kind, "dtype": dtype, "nz": shape[0] if len(shape) == 3 else 1,
         "ny": shape[-2], "nx": shape[-1], "steps": steps, "loss": loss, "slots": slots,
         "sched": sched, "dk": dk, "dparams": dparams, "limit": limit}
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # a grid small enough for interactive work: latency and launches are all there is
        _case("jacobi_f64_64", "jacobi", "f64", (64, 64), 10, slots=9, sched="store_all"),
        # the linear 2-D stencil on a grid that fills the chip; its adjoint reads no state
        _case("jacobi_f64_4096", "jacobi", "f64", (4096, 4096), 100, slots=10),
        # the same stencil in single precision on an odd grid, fitting an observed field and
        # the step's constant together (the gradient of w makes the adjoint read states)
        _case("jacobi_f32_odd_dw", "jacobi", "f32", (2501, 3003), 60, "half_sq_diff", 8,
              dparams=True),
        # a branch in every step (bounded values), under a ten-snapshot budget
        _case("jacobi_f64_4096_limit", "jacobi", "f64", (4096, 4096), 100, slots=10, limit=True),
        # the nonlinear 3-D stencil at the size most 3-D runs have, eight snapshots
        _case("allencahn_f64_512", "allencahn", "f64", (512, 512, 512), 50, "dot_w", 8),
        # the largest grid, where two snapshots are all that fits beside everything else
        _case("allencahn_f64_1024", "allencahn", "f64", (1024, 1024, 1024), 16, "dot_w", 2,
              "binomial"),
        # single precision on an odd box, an explicit cotangent, with dL/dD and dL/dC
        _case("allencahn_f32_odd_dp", "allencahn", "f32", (150, 257, 301), 50, "seed", 6,
              "uniform", dparams=True),
        # the coefficient field's gradient at the size of a large 2-D inversion
        _case("vardiff_f32_8192_dk", "vardiff", "f32", (8192, 8192), 200, "half_sq_diff", 16,
              dk=True),
        # the same inversion in double precision on a modest odd grid, dt's gradient too
        _case("vardiff_f64_odd_dk_dp", "vardiff", "f64", (1023, 1537), 80, "half_sq_diff", 10,
              "binomial", dk=True, dparams=True),
        # the in-place sweep at the size of the paper's Seidel2d case study
        _case("gs_f64_400", "gs", "f64", (400, 400), 100),
        # the in-place sweep on a grid that fills the chip
        _case("gs_f64_4096", "gs", "f64", (4096, 4096), 100),
        # the program without its gradient: a simulation run
        _case("forward_allencahn_f64_256", "allencahn", "f64", (256, 256, 256), 100,
              op="forward"),
    ]


def draw(rng):
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(list(KINDS))
    dtype = rng.choice(["f64", "f32"])
    shape = ((log_int(20, 400), log_int(24, 480), log_int(24, 480)) if kind == "allencahn"
             else (log_int(48, 5000), log_int(48, 5000)))
    if rng.random() < 0.4:  # rows of whole 64-byte lines are as common as odd ones
        shape = shape[:-1] + (max(16, shape[-1] // 16 * 16),)
    steps = log_int(8, 200)
    steps = max(8, min(steps, int(1.5e9 // math.prod(shape))))
    op = "forward" if rng.random() < 0.15 else "vjp"
    vjp = op == "vjp"
    sched = rng.choice(["auto", "uniform", "binomial"])
    return _case(None, kind, dtype, shape, steps, rng.choice(list(LOSSES)), log_int(4, 24), sched,
                 op, dk=vjp and kind == "vardiff" and rng.random() < 0.7,
                 dparams=vjp and kind != "gs" and rng.random() < 0.25,
                 limit=kind != "gs" and rng.random() < 0.2)


def _shape(c):
    return (c["nz"], c["ny"], c["nx"]) if c["kind"] == "allencahn" else (c["ny"], c["nx"])


def _inputs(c, seed):
    """x0, K and the loss's array, as the workloads of the package draw them:
    uniform states, coefficients in [0.5, 1.5), normal weights, uniform targets."""
    dt = torch.float64 if c["dtype"] == "f64" else torch.float32
    gen = torch.Generator(device=DEVICE)
    gen.manual_seed(int(seed) * 4 + 1)
    shape = _shape(c)

    def uniform(lo, hi):
        return torch.empty(shape, dtype=dt, device=DEVICE).uniform_(lo, hi, generator=gen)

    x0 = uniform(-1.0, 1.0) if c["kind"] == "allencahn" else uniform(0.0, 1.0)
    K = uniform(0.5, 1.5) if c["kind"] == "vardiff" else None
    aux = None
    if c["op"] == "vjp" and c["loss"] == "half_sq_diff":
        aux = uniform(0.0, 1.0)
    elif c["op"] == "vjp" and c["loss"] != "half_sq":
        aux = torch.empty(shape, dtype=dt, device=DEVICE).normal_(generator=gen)
    return x0, K, aux


def _budget(c):
    return c["slots"] * math.prod(_shape(c)) * (8 if c["dtype"] == "f64" else 4)


def prepare(case, seed):
    x0, K, aux = _inputs(case, seed)
    state = {"case": case, "x0": x0, "K": K, "aux": aux,
             "lim": BOUNDS[case["kind"]] if case["limit"] else None}
    if case["op"] == "vjp":  # the workspace a program allocates once for its calls
        dims = (case["nx"], case["ny"], case["nz"])
        prob = adst.make_problem(KINDS[case["kind"]],
                                 adst.ADST_F64 if case["dtype"] == "f64" else adst.ADST_F32, dims,
                                 lim=state["lim"])
        grads = ((adst.ADST_GRAD_COEFF if case["dk"] else 0) |
                 (adst.ADST_GRAD_PARAMS if case["dparams"] else 0))
        info = adst.adst_plan(prob, case["steps"], _budget(case), SCHEDS[case["sched"]], grads)
        state["ws"] = torch.empty(info.workspace_bytes, dtype=torch.uint8, device=DEVICE)
    return state


def run(state):
    c = state["case"]
    if c["op"] == "forward":
        return {"xT": adst.forward(KINDS[c["kind"]], state["x0"], state["K"], c["steps"],
                                   lim=state["lim"])}
    out = adst.vjp(KINDS[c["kind"]], state["x0"], state["K"], c["steps"], LOSSES[c["loss"]],
                   state["aux"], _budget(c), SCHEDS[c["sched"]], want_dcoeff=c["dk"],
                   ws=state["ws"], want_dparams=c["dparams"], lim=state["lim"])
    return {k: out[k] for k in ("dx0", "dK", "xT", "loss", "dparams") if out[k] is not None}


def work(case):
    """Inputs once, outputs once; one forward and (for vjp) one adjoint
    evaluation of every point and step, whatever the budget recomputes."""
    n = math.prod(_shape(case))
    size = 8 if case["dtype"] == "f64" else 4
    arrays = 2 + (case["kind"] == "vardiff")  # x0, x_T, K
    flops = {"jacobi": 5, "allencahn": 14, "vardiff": 42, "gs": 5}[case["kind"]]
    if case["op"] == "vjp":
        arrays += 1 + (case["loss"] != "half_sq") + case["dk"]  # dx0, aux, dK
        flops += {"jacobi": 5, "allencahn": 11, "vardiff": 42, "gs": 7}[case["kind"]]
        flops += 42 * case["dk"] + {"jacobi": 6, "allencahn": 13, "vardiff": 42, "gs": 0}[
            case["kind"]] * case["dparams"]
    return {"bytes": n * size * arrays, "flops": n * case["steps"] * flops}


def tolerance(case):
    """About four times what `run` and `exact` differ by over these cases. The
    constants' gradients are sums over every point and step that cancel, which
    magnifies a state's rounding (Jacobi f32: 4e-4 from 64 bits)."""
    if case["limit"] and case["dtype"] == "f32":
        # a value within rounding of a bound may take the other branch
        return {"rel": 1e-2, "max": 0.99}
    if case["dparams"]:
        return {"rel": 4e-12} if case["dtype"] == "f64" else {"rel": 1.6e-3}
    return {"rel": 2e-13} if case["dtype"] == "f64" else {"rel": 3.2e-5}


# ---------------------------------------------------------------- 64 bits
def _params(c):
    p = PARAMS[c["kind"]]
    return p if c["dtype"] == "f64" else tuple(float(np.float32(v)) for v in p)


def _ratio(c, d):
    return 1.0 / d if c["dtype"] == "f64" else float(np.float32(1) / np.float32(d))


NEIGHBOURS = ((-1, 0), (1, 0), (0, -1), (0, 1), (-1, -1), (1, -1), (-1, 1), (1, 1))


def _edge(ny, nx, dx, dy):
    """Slices of the points that have the neighbour (dx, dy), and of that neighbour."""
    def cut(n, d):
        return (slice(max(0, -d), n - max(0, d)), slice(max(0, d), n - max(0, -d)))
    (ys, yn), (xs, xn) = cut(ny, dy), cut(nx, dx)
    return (ys, xs), (yn, xn)


class _Steps:
    """One step of a (not in-place) kind, its transpose and its partials."""

    def __init__(self, c, K):
        self.c, self.K, self.p = c, K, _params(c)
        self.lim = BOUNDS[c["kind"]] if c["limit"] else None
        if self.lim and c["dtype"] == "f32":
            self.lim = tuple(float(np.float32(v)) for v in self.lim)

    def sums(self, x):
        """The sub-expression each point's update is built from."""
        k = self.c["kind"]
        if k == "jacobi":
            return (((x[1:-1, 1:-1] + x[1:-1, :-2]) + x[1:-1, 2:]) + x[:-2, 1:-1]) + x[2:, 1:-1]
        if k == "allencahn":
            return self.around(x) - 6.0 * x
        acc = torch.zeros_like(x)
        for q, (dx, dy) in enumerate(NEIGHBOURS):
            a, b = _edge(*x.shape, dx, dy)
            cn = _ratio(self.c, 3) if q < 4 else _ratio(self.c, 12)
            acc[a] += (cn * (self.K[a] + self.K[b])) * (x[b] - x[a])
        return acc

    @staticmethod
    def around(x):
        s = torch.zeros_like(x)
        s[:, :, 1:] += x[:, :, :-1]
        s[:, :, :-1] += x[:, :, 1:]
        s[:, 1:] += x[:, :-1]
        s[:, :-1] += x[:, 1:]
        s[1:] += x[:-1]
        s[:-1] += x[1:]
        return s

    def raw(self, x):
        k = self.c["kind"]
        s = self.sums(x)
        if k == "jacobi":
            y = x.clone()
            y[1:-1, 1:-1] = self.p[0] * s
            return y
        if k == "allencahn":
            s *= self.p[0]
            s += x
            s -= ((x * x) * x) * self.p[1]
            return s
        s *= self.p[0]
        return x + s

    def forward(self, x):
        y = self.raw(x)
        return y if self.lim is None else y.clamp_(*self.lim)

    def adjoint(self, x, g, dK, dp):
        """g_{t-1} from g_t and x = x_{t-1}; adds to dK and dp where wanted."""
        k = self.c["kind"]
        if self.lim is not None:
            y = self.raw(x)
            g = torch.where((y < self.lim[0]) | (y > self.lim[1]), torch.zeros_like(g), g)
            del y
        if dp is not None:
            s = self.sums(x)
            dp[0] += ((g[1:-1, 1:-1] if k == "jacobi" else g) * s).sum()
            if k == "allencahn":
                dp[1] -= (g * ((x * x) * x)).sum()
        if k == "jacobi":
            gi = torch.zeros_like(g)
            gi[1:-1, 1:-1] = self.p[0] * g[1:-1, 1:-1]
            out = g.clone()
            out[1:-1, 1:-1] = gi[1:-1, 1:-1]
            out[:, :-1] += gi[:, 1:]
            out[:, 1:] += gi[:, :-1]
            out[:-1] += gi[1:]
            out[1:] += gi[:-1]
            return out
        if k == "allencahn":
            out = self.around(g)
            out *= self.p[0]
            f = x * x
            f *= -3.0 * self.p[1]
            f += 1.0 - 6.0 * self.p[0]
            f *= g
            out += f
            return out
        out = torch.zeros_like(g)
        for q, (dx, dy) in enumerate(NEIGHBOURS):
            a, b = _edge(*g.shape, dx, dy)
            cn = _ratio(self.c, 3) if q < 4 else _ratio(self.c, 12)
            dg = g[b] - g[a]
            out[a] += (cn * (self.K[a] + self.K[b])) * dg
            if dK is not None:
                dK[a] -= self.p[0] * ((cn * (x[b] - x[a])) * dg)
        return g + self.p[0] * out


def _sweeps(c, x):
    """The in-place kind's sweeps, rows of several sweeps at a time: row j of
    sweep s goes at level j + 2s, when the rows it reads are what it needs. A
    row's own recurrence x'[i] = w*(b[i] + x'[i-1]) is one triangular product."""
    w, (ny, nx), T = _params(c)[0], x.shape, c["steps"]
    if ny < 3 or nx < 3:
        return x
    m = _powers(w, nx - 2, x.device)
    left = w ** torch.arange(1, nx - 1, dtype=torch.float64, device=x.device)
    for level in range(1, ny - 1 + 2 * (T - 1)):
        j = _rows(level, ny, T, x.device)
        row = x[j]
        b = ((row[:, 1:-1] + row[:, 2:]) + x[j + 1, 1:-1]) + x[j - 1, 1:-1]
        x[j, 1:-1] = (w * b) @ m.T + row[:, :1] * left
    return x


def _powers(w, n, device):
    """m[i, k] = w^(i-k) for k <= i, else 0."""
    d = torch.arange(n, device=device)
    d = (d[:, None] - d[None, :]).to(torch.float64)
    return torch.where(d >= 0, torch.full_like(d, w) ** d.clamp_min(0), torch.zeros_like(d))


def _rows(level, ny, T, device):
    s0 = max(0, -(-(level - (ny - 2)) // 2))
    s1 = min(T - 1, (level - 1) // 2)
    return level - 2 * torch.arange(s0, s1 + 1, device=device)


def _reverse_sweeps(c, g):
    """The transposed sweeps, from the last row down; row j of reverse sweep s
    goes at level (ny - 1 - j) + 2s. Interior rows hold h between sweeps."""
    w, (ny, nx), T = _params(c)[0], g.shape, c["steps"]
    if ny < 3 or nx < 3:
        return g
    m = _powers(w, nx - 2, g.device)

    def before(h, j):  # the gradient the sweep before left, from its h
        r = h[j, 1:-1].clone()
        r[:, 1:] += h[j, 1:-2]
        return w * (r + torch.where((j > 1)[:, None], h[j - 1, 1:-1], torch.zeros_like(r)))

    for level in range(1, ny - 1 + 2 * (T - 1)):
        up = _rows(level, ny, T, g.device)          # ny - 1 - j
        j = ny - 1 - up
        first = up == level                         # sweep 0: interior rows still hold g_T
        gin = torch.where(first[:, None], g[j, 1:-1], before(g, j))
        above = torch.where((j < ny - 2)[:, None], g[j + 1, 1:-1], torch.zeros_like(gin))
        h = (gin + w * above) @ m
        g[j, 1:-1] = h
        g[j, 0] += w * h[:, 0]
        g[j, -1] += w * h[:, -1]
        g[ny - 1, 1:-1] += w * (h * (j == ny - 2)[:, None]).sum(0)
        g[0, 1:-1] += w * (h * (j == 1)[:, None]).sum(0)
    j = torch.arange(1, ny - 1, device=g.device)
    g[1:-1, 1:-1] = before(g, j)
    return g


def _loss(c, x, aux):
    if c["loss"] == "half_sq":
        return (0.5 * (x * x)).sum(), x.clone()
    if c["loss"] == "half_sq_diff":
        d = x - aux
        return (0.5 * (d * d)).sum(), d
    return (aux * x).sum(), aux.clone()


def exact(case, seed):
    x0, K, aux = ((None if a is None else a.double()) for a in _inputs(case, seed))
    T, vjp = case["steps"], case["op"] == "vjp"
    if case["kind"] == "gs":
        xT = _sweeps(case, x0.clone())
        if not vjp:
            return {"xT": xT}
        loss, g = _loss(case, xT, aux)
        return {"dx0": _reverse_sweeps(case, g), "xT": xT, "loss": loss}
    f = _Steps(case, K)
    seg = max(1, math.isqrt(T))
    kept, x = {}, x0
    for t in range(T):  # every seg-th state is kept, the others formed again below
        if vjp and t % seg == 0:
            kept[t] = x
        x = f.forward(x)
    if not vjp:
        return {"xT": x}
    xT = x
    loss, g = _loss(case, xT, aux)
    dK = torch.zeros_like(x0) if case["dk"] else None
    dp = torch.zeros(2, dtype=torch.float64, device=DEVICE) if case["dparams"] else None
    for base in sorted(kept, reverse=True):
        states = [kept.pop(base)]
        while len(states) < min(seg, T - base):
            states.append(f.forward(states[-1]))
        while states:
            g = f.adjoint(states.pop(), g, dK, dp)
    out = {"dx0": g, "dK": dK, "xT": xT, "loss": loss, "dparams": dp}
    return {k: v for k, v in out.items() if v is not None}
