"""Performance cases of the solver: the calls a user's program makes, over the range it makes them.

The sizes are those of the benchmark workloads and the tests (or generic ones
between them).  ``listed`` names twelve of them, ``draw`` gives more of the same
ranges.  A pass goes through the public entry points only: a solver that holds
its operator on the device, new data per pass where the program has new data,
the solve, and the point copied out.  Solves run to ``eps`` or to ``steps`` ADMM
steps, whichever comes first.  Results of FP32 solvers are handed on as FP32
arrays, which is what their values are.

``exact`` repeats a solve in FP64 torch arithmetic without the package: the same
iteration (scaling, warm-started CG with the same tolerance schedule, the test
every ten steps) on explicit matrices or FFT convolutions.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_1609_03488_amd as P

_PRECISION = {"fp64": P.FP64, "fp32": P.FP32, "bf16": P.BF16}
_CHECK = 10                # steps between termination tests (library default)
_CG_MAX, _CG_TOL, _CG_RATE, _CG_FLOOR = 10, 0.1, 1.5, 1e-6   # library defaults
_ALPHA = 1.5


# ---------------------------------------------------------------- the cases
def listed():
    return [
        # the smallest whole call: a one-off solve from code that may not
        # allocate device memory (creation, upload, solve and download included)
        dict(name="noalloc_deconv_n300_k31", family="noalloc", n=300, k=31, density=0.05, noise_var=1e-4,
             precision="fp32", normalize=1, eps=1e-4, steps=200),
        # the paper's deconvolution size in FP64, one problem at a time (latency)
        dict(name="deconv_n1000_k101_fp64", family="deconv", n=1000, k=101, density=0.10, noise_var=1e-4,
             precision="fp64", normalize=2, eps=1e-6, steps=60, batch=1, fresh=False),
        # many small signals blurred by one kernel, solved together (throughput)
        dict(name="deconv_batch128_n1500_k151", family="deconv", n=1500, k=151, density=0.05, noise_var=1e-4,
             precision="fp32", normalize=1, eps=1e-4, steps=100, batch=128, fresh=False),
        # an ordinary signal, a new observation every pass on a kept operator
        dict(name="deconv_n20011_k201_fresh", family="deconv", n=20011, k=201, density=0.05, noise_var=1e-4,
             precision="fp32", normalize=1, eps=1e-4, steps=200, batch=1, fresh=True),
        # the same in FP64, where FP32's accuracy does not do
        dict(name="deconv_n30011_k257_fp64", family="deconv", n=30011, k=257, density=0.05, noise_var=1e-4,
             precision="fp64", normalize=1, eps=1e-6, steps=200, batch=1, fresh=False),
        # the largest signal, solved to its tolerance: the headline solve
        dict(name="deconv_n1M_k1025", family="deconv", n=1 << 20, k=1025, density=0.01, noise_var=1e-6,
             precision="fp32", normalize=1, eps=1e-4, steps=2000, batch=1, fresh=False),
        # the largest dense lasso, memory bound on the matrix
        dict(name="lasso_5000x10000", family="lasso", m=5000, n=10000, precision="fp32", normalize=2, eps=1e-5,
             steps=400, batch=1),
        # many lasso instances sharing one matrix, on the matrix cores
        dict(name="lasso_batch64_2000x8000_bf16", family="lasso", m=2000, n=8000, precision="bf16", normalize=2,
             eps=1e-3, steps=2000, batch=64),
        # lasso on a convolution operator with a long kernel
        dict(name="conv_lasso_n3000_k1365", family="conv_lasso", n=3000, k=1365, precision="fp32", normalize=1,
             eps=1e-4, steps=200),
        # regularized least squares to 1e-8 by CG, dense and convolution (FP64)
        dict(name="regls_dense_6000x3000", family="regls", kind="dense", m=6000, n=3000, precision="fp64", tol=1e-8),
        dict(name="regls_conv_n3000_k1365", family="regls", kind="conv", n=3000, k=1365, precision="fp64", tol=1e-8),
        # a burst of requests of different sizes through the server
        dict(name="server_24_requests", family="server", count=24, n_lo=1000, n_hi=100000, k_lo=11, k_hi=501,
             sizes=1, normalize=1, eps=1e-4, steps=100),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _odd(v):
    return v | 1


def draw(rng):
    family = rng.choice(("noalloc", "deconv", "deconv", "deconv", "batch", "lasso", "lasso", "lasso_batch",
                         "conv_lasso", "regls", "regls", "server"))
    if family == "noalloc":
        n = _log_int(rng, 100, 4000)
        return dict(family="noalloc", n=n, k=_odd(_log_int(rng, 5, max(7, n // 4))), density=0.05, noise_var=1e-4,
                    precision=rng.choice(("fp32", "fp64")), normalize=1, eps=1e-4, steps=rng.choice((100, 200)))
    if family == "deconv":
        precision = rng.choice(("fp32", "fp32", "fp64"))
        n = _log_int(rng, 300, 60000 if precision == "fp64" else 1 << 20)
        # (block equilibration makes the subspace solves of a blur run into the CG
        # limit, and rounding then grows by three digits in 60 steps: FP64 only)
        level = 2 if precision == "fp64" and n < 20000 and rng.random() < 0.5 else 1
        return dict(family="deconv", n=n, k=_odd(_log_int(rng, 11, min(1025, n // 3))), density=0.05,
                    noise_var=1e-4, precision=precision, normalize=level, eps=1e-6,
                    steps=60 if level == 2 else rng.choice((100, 200)), batch=1, fresh=rng.random() < 0.5)
    if family == "batch":
        n = _log_int(rng, 300, 5000)
        return dict(family="deconv", n=n, k=_odd(_log_int(rng, 11, min(301, n // 3))), density=0.05, noise_var=1e-4,
                    precision=rng.choice(("fp32", "fp64")), normalize=1, eps=1e-4, steps=100,
                    batch=rng.choice((8, 32, 128, 256)), fresh=False)
    if family == "lasso":
        m = _log_int(rng, 100, 5000)
        return dict(family="lasso", m=m, n=min(10000, int(m * rng.uniform(1.0, 4.0))),
                    precision=rng.choice(("fp32", "fp64")), normalize=rng.choice((1, 2)), eps=1e-5, steps=100, batch=1)
    if family == "lasso_batch":
        m = _log_int(rng, 250, 2000)
        return dict(family="lasso", m=m, n=int(m * rng.uniform(2.0, 4.0)), precision="bf16", normalize=2, eps=1e-3,
                    steps=200, batch=rng.randint(8, 64))
    if family == "conv_lasso":
        n = _log_int(rng, 500, 20000)
        return dict(family="conv_lasso", n=n, k=_odd(_log_int(rng, 11, min(1501, n // 2))),
                    precision=rng.choice(("fp32", "fp64")), normalize=1, eps=1e-4, steps=100)
    if family == "regls":
        if rng.random() < 0.5:
            n = _log_int(rng, 200, 3000)
            return dict(family="regls", kind="dense", m=int(n * rng.uniform(1.2, 2.0)), n=n, precision="fp64",
                        tol=1e-8)
        n = _log_int(rng, 300, 30000)
        return dict(family="regls", kind="conv", n=n, k=_odd(_log_int(rng, 11, min(1365, n // 2))),
                    precision="fp64", tol=1e-8)
    return dict(family="server", count=rng.randint(8, 24), n_lo=500, n_hi=_log_int(rng, 5000, 100000), k_lo=11,
                k_hi=_odd(_log_int(rng, 51, 501)), sizes=rng.randint(2, 1 << 30), normalize=1, eps=1e-4, steps=60)


# ---------------------------------------------------------------- inputs
def _generator(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _taps(k, sigma):
    j = torch.arange(k, dtype=torch.float64, device="cuda")
    c = torch.exp(-((j - (k - 1) / 2) ** 2) / (2.0 * sigma ** 2))
    return c / c.sum()


def _normal(g, *shape):
    return torch.randn(*shape, generator=g, device="cuda", dtype=torch.float64)


def _sparse(g, n, density, normal):
    x = torch.zeros(n, dtype=torch.float64, device="cuda")
    pos = torch.randperm(n, generator=g, device="cuda")[: int(density * n)]
    x[pos] = _normal(g, pos.numel()) if normal else torch.rand(pos.numel(), generator=g, device="cuda",
                                                               dtype=torch.float64)
    return x


class _Conv:
    """Full convolution with `taps` and its adjoint, FP64, by FFT."""

    def __init__(self, taps, n):
        self.n, self.rows = n, n + taps.numel() - 1
        self.size = 1 << (self.rows - 1).bit_length()
        self.spectrum = torch.fft.rfft(taps, self.size)
        self.frob2 = n * float((taps * taps).sum())

    def __call__(self, x):
        return torch.fft.irfft(torch.fft.rfft(x, self.size) * self.spectrum, self.size)[: self.rows]

    def adjoint(self, y):
        return torch.fft.irfft(torch.fft.rfft(y, self.size) * self.spectrum.conj(), self.size)[: self.n]


class _Dense:
    def __init__(self, a):
        self.a, self.n, self.rows = a, a.shape[1], a.shape[0]
        self.frob2 = float((a * a).sum())

    def __call__(self, x):
        return self.a @ x

    def adjoint(self, y):
        return self.a.t() @ y


def _deconv_data(case, seed):
    """taps and the observations of every instance (FP64, on the device)."""
    g = _generator(seed)
    taps = _taps(case["k"], case["k"] / 7.0)
    op = _Conv(taps, case["n"])
    obs = []
    for _ in range(case.get("batch", 1)):
        clean = op(_sparse(g, case["n"], case["density"], False))
        obs.append(clean + math.sqrt(case["noise_var"]) * _normal(g, op.rows))
    return taps, op, obs


def _lasso_data(case, seed):
    """the operator and (observation, lambda) of every instance"""
    g = _generator(seed)
    if case["family"] == "conv_lasso":
        taps = _taps(case["k"], case["k"] / 4.55)
        a, op, density = taps, _Conv(taps, case["n"]), 1.0
    else:
        a = _normal(g, case["m"], case["n"]) / math.sqrt(case["m"])
        if case["precision"] != "fp64":
            a = a.float()
        op, density = _Dense(a.double()), 0.05
    inst = []
    for _ in range(case.get("batch", 1)):
        b = op(_sparse(g, case["n"], density, True)) + 0.01 * _normal(g, op.rows)
        inst.append((b, 0.1 * float(op.adjoint(b).abs().max())))
    return a, op, inst


def _regls_data(case, seed):
    g = _generator(seed)
    if case["kind"] == "conv":
        a = _taps(case["k"], case["k"] / 4.55)
        op = _Conv(a, case["n"])
    else:
        a = _normal(g, case["m"], case["n"])
        op = _Dense(a)
    return a, op, op(_normal(g, case["n"])) + 0.01 * _normal(g, op.rows)


def _server_cases(case, seed):
    """the requests of a burst: sizes spread as in the serving trace, data from the seed"""
    r = np.random.Generator(np.random.PCG64(case["sizes"]))
    out = []
    for _ in range(case["count"]):
        n = int(round(math.exp(r.uniform(math.log(case["n_lo"]), math.log(case["n_hi"])))))
        k = int(r.integers(case["k_lo"] // 2, case["k_hi"] // 2 + 1)) * 2 + 1
        out.append(dict(n=n, k=k, density=0.05, noise_var=1e-4, seed=seed * 1000 + len(out)))
    return out


def _host(t):
    return t.cpu().numpy()


def _settings(case, **kw):
    return P.Settings.make(precision=_PRECISION[case.get("precision", "fp32")], normalize=case["normalize"],
                           eps=case["eps"], max_iters=case["steps"], **kw)


def prepare(case, seed):
    family = case["family"]
    state = {"case": case, "single": case.get("precision", "fp32") != "fp64"}
    stream = state["stream"] = torch.cuda.Stream()
    if family in ("deconv", "noalloc"):
        taps, _, obs = _deconv_data(case, seed)
        problems = [P.deconv_problem(_host(taps), _host(b)) for b in obs]
        state["data"] = [(p.b, p.c) for p in problems]
        if family == "noalloc":
            state["problem"], state["settings"] = problems[0], _settings(case)
            return state
    elif family == "lasso":
        a, _, inst = _lasso_data(case, seed)
        torch.cuda.synchronize()   # (the operator reads the matrix in place)
        problems = [P.lasso_problem(a, _host(inst[0][0]), inst[0][1])]
        p = problems[0]
        n = case["n"]
        state["data"] = []
        for b, lam in inst:
            c = p.c.copy()
            c[n:2 * n] = lam
            state["data"].append((np.concatenate([np.zeros(2 * n), [1.0], -2.0 * _host(b), [-1.0]]), c))
    elif family == "conv_lasso":
        taps, _, inst = _lasso_data(case, seed)
        problems = [P.conv_lasso_problem(_host(taps), _host(inst[0][0]), inst[0][1])]
        state["data"] = [(problems[0].b, problems[0].c)]
    elif family == "regls":
        a, _, b = _regls_data(case, seed)
        if case["kind"] == "conv":
            state["regls"] = P.RegLS(1e-2, taps=_host(a), n=case["n"], precision=P.FP64, stream=stream)
        else:
            state["regls"] = P.RegLS(1e-2, A=_host(a), precision=P.FP64, stream=stream)
        state["b"] = _host(b)
        return state
    else:
        state["problems"] = []
        for r in _server_cases(case, seed):
            taps, _, obs = _deconv_data(r, r["seed"])
            state["problems"].append(P.deconv_problem(_host(taps), _host(obs[0])))
        state["server"] = P.Server(1 << 29, 64, _settings(case, fused_max=3072), stream=stream)
        return state
    p = problems[0]
    solver = P.Solver(p.op, p.l, p.q, _settings(case), batch=case.get("batch", 1), stream=stream)
    for i, (b, c) in enumerate(state["data"]):
        solver.set_data(i, b, c)
    state["solver"], state["op"] = solver, p.op
    return state


# ---------------------------------------------------------------- a pass
def _points(state, points):
    """x, y, s of one or more instances, one array each, in the solver's precision"""
    dtype = np.float32 if state["single"] else np.float64
    return {name: np.concatenate([p[j] for p in points]).astype(dtype, copy=False)
            for j, name in enumerate(("x", "y", "s"))}


def run(state):
    case = state["case"]
    family = case["family"]
    if family == "noalloc":
        p = state["problem"]
        x, y, s, info = P.solve_noalloc(p.op, p.l, p.q, p.b, p.c, state["settings"], stream=state["stream"])
        return dict(_points(state, [(x, y, s)]), status=info["status"], iters=info["iters"])
    if family == "regls":
        x, iters = state["regls"].solve(state["b"], tol=case["tol"])
        return {"x": x, "iters": iters}
    if family == "server":
        server = state["server"]
        tickets = [server.submit(p.op, p.l, p.q, p.b, p.c) for p in state["problems"]]
        while server.step(_CHECK):
            pass
        done = [server.fetch(t) for t in tickets]
        return dict(_points(state, done), status=np.array([d[3]["status"] for d in done]),
                    iters=np.array([d[3]["iters"] for d in done]))
    solver = state["solver"]
    if case.get("fresh"):
        b, c = state["data"][0]
        solver.set_data(0, b, c)
    else:
        solver.reset()
    infos = solver.solve()
    out = _points(state, [solver.solution(i) for i in range(len(infos))])
    return dict(out, status=np.array([i["status"] for i in infos]), iters=np.array([i["iters"] for i in infos]))


# ---------------------------------------------------------------- work
def _apply_flops(case, n):
    """one product with the operator: the direct sum or, where it is less, the FFT's"""
    if "k" not in case:
        return 2.0 * case["m"] * n
    return min(2.0 * case["k"] * n, 20.0 * n * math.log2(4.0 * case["k"]))


def work(case):
    """Operator and data read and the point written once, and per ADMM step the
    iteration's state (u_x, u_y, v_s) read and written once, the dense matrix
    read once, and three products (the right-hand side and one CG iteration)."""
    size = 8 if case.get("precision", "fp32") == "fp64" else 4
    if case["family"] == "server":
        ratio = math.log(case["n_hi"] / case["n_lo"])
        n = (case["n_hi"] - case["n_lo"]) / ratio      # mean of the log-uniform sizes
        one = dict(case, k=(case["k_lo"] + case["k_hi"]) / 2)
        m = 2 * n + one["k"]
        return {"bytes": case["count"] * (8 * (n + m) * 2 + case["steps"] * 2 * size * (n + 2 * m)),
                "flops": case["count"] * case["steps"] * 3 * _apply_flops(one, n)}
    n, batch = case["n"], case.get("batch", 1)
    if case["family"] == "regls":
        rows = case["m"] if case["kind"] == "dense" else n + case["k"] - 1
        steps = 15 if case["kind"] == "conv" else 50
        entries = case["m"] * n if case["kind"] == "dense" else case["k"]
        return {"bytes": 8.0 * (steps * entries + rows + 2 * n), "flops": 2.0 * steps * _apply_flops(case, n)}
    if case["family"] in ("deconv", "noalloc"):
        nv, m, entries = n + 1, 2 * n + case["k"], case["k"]
    else:
        rows = case["m"] if case["family"] == "lasso" else n + case["k"] - 1
        nv, m = 2 * n + 1, 2 * n + rows + 2
        entries = case["m"] * n if case["family"] == "lasso" else case["k"]
    steps = 620 if case["steps"] == 2000 and "k" in case else min(case["steps"], 400)
    return {"bytes": float(batch * (8 * (nv + m) * 2 + steps * 2 * size * (nv + 2 * m)) + steps * entries * size),
            "flops": 3.0 * batch * steps * _apply_flops(case, n)}


# ---------------------------------------------------------------- the same in 64 bits
class _Program:
    """min c'x, A x + s = b, s in R_+^l x SOC of the rest; rows and columns in
    groups that share a scale, `weight` the groups' squared Frobenius norms."""

    def __init__(self, n, m, l, b, c, apply, adjoint, rows, cols, weight):
        self.n, self.m, self.l, self.b, self.c = n, m, l, b, c
        self.apply, self.adjoint = apply, adjoint
        self.rows, self.cols, self.weight = rows, cols, weight


def _deconv_program(op, obs):
    n, m = op.n, op.n + 1 + op.rows

    def apply(x):
        return torch.cat([-x, -op(x[:n])])

    def adjoint(y):
        return torch.cat([-y[:n] - op.adjoint(y[n + 1:]), -y[n:n + 1]])

    zero = obs.new_zeros(n + 1)
    c = zero.clone()
    c[n] = 1.0
    weight = np.array([[float(n), 0.0], [op.frob2, 1.0]])
    return _Program(n + 1, m, n, torch.cat([zero, -obs]), c, apply, adjoint, [n, m - n], [n, 1], weight)


def _lasso_program(op, obs, lam):
    n, m = op.n, 2 * op.n + op.rows + 2

    def apply(v):
        x, t, u = v[:n], v[n:2 * n], v[2 * n:]
        return torch.cat([x - t, -x - t, -u, -2.0 * op(x), -u])

    def adjoint(y):
        p, q, w = y[:n], y[n:2 * n], y[2 * n + 1:m - 1]
        return torch.cat([p - q - 2.0 * op.adjoint(w), -p - q, -y[2 * n:2 * n + 1] - y[m - 1:]])

    one = obs.new_ones(1)
    b = torch.cat([obs.new_zeros(2 * n), one, -2.0 * obs, -one])
    c = torch.cat([obs.new_zeros(n), obs.new_full((n,), lam), 0.5 * one])
    weight = np.array([[n, n, 0.0], [n, n, 0.0], [4.0 * op.frob2, 0.0, 2.0]])
    return _Program(2 * n + 1, m, 2 * n, b, c, apply, adjoint, [n, n, m - 2 * n], [n, n, 1], weight)


def _scaling(prog, level):
    """row and column scales of the groups (20 Ruiz passes at level 2), and of b and c"""
    rows, cols, w = np.array(prog.rows, float), np.array(prog.cols, float), prog.weight
    d, e = np.ones(len(rows)), np.ones(len(cols))

    def row_rms():
        return np.sqrt(d * d * (w @ (e * e)) / rows)

    def col_rms():
        return np.sqrt(e * e * (w.T @ (d * d)) / cols)

    for _ in range(20 if level == 2 else 0):
        d = d / np.sqrt(np.clip(row_rms(), 1e-4, 1e4))
        e = e / np.sqrt(np.clip(col_rms(), 1e-4, 1e4))
    dv = torch.tensor(np.repeat(d, prog.rows), device="cuda")
    ev = torch.tensor(np.repeat(e, prog.cols), device="cuda")
    sb = float(rows @ row_rms()) / prog.m / max(float((dv * prog.b).norm()), 1e-4)
    sc = float(cols @ col_rms()) / prog.n / max(float((ev * prog.c).norm()), 1e-4)
    return dv, ev, sb, sc


def _cg(kmul, z, rhs, tol, limit):
    """conjugate gradients on K z = rhs from z until ||r|| <= tol"""
    r = rhs - kmul(z)
    p, rr, it = r, float(r @ r), 0
    while math.sqrt(rr) > tol and it < limit:
        q = kmul(p)
        a = rr / float(p @ q)
        z, r, it = z + a * p, r - a * q, it + 1
        new = float(r @ r)
        p, rr = r + (new / rr) * p, new
    return z, it


def _admm(prog, case):
    """the whole solve: (x, y, s, status, iterations)"""
    dv, ev, sb, sc = _scaling(prog, case["normalize"])
    b, c, l = sb * dv * prog.b, sc * ev * prog.c, prog.l
    fp64 = case.get("precision", "fp32") == "fp64"
    floor = min(_CG_FLOOR, 1e-2 * case["eps"]) if fp64 else _CG_FLOOR
    nb, nc = 1.0 + float(prog.b.norm()), 1.0 + float(prog.c.norm())

    def apply(x):
        return dv * prog.apply(ev * x)

    def adjoint(y):
        return ev * prog.adjoint(dv * y)

    def kmul(x):
        return x + adjoint(apply(x))

    h = c - adjoint(b)
    gx, _ = _cg(kmul, torch.zeros_like(c), h, 1e-14 * float(h.norm()), 500)
    gy = b + apply(gx)
    eta = 1.0 + float(c @ gx) + float(b @ gy)
    ux, uy, vs, z = torch.zeros_like(c), torch.zeros_like(b), torch.zeros_like(b), torch.zeros_like(c)
    tau = kappa = 1.0
    status, it = 2, 0
    while it < case["steps"]:
        w = uy + vs
        h = ux - adjoint(w)
        tol = float(h.norm()) * max(floor, _CG_TOL / (it + 1.0) ** _CG_RATE)
        z, _ = _cg(kmul, z, h, tol, _CG_MAX)
        zy = w + apply(z)
        ut = (tau + kappa + float(c @ z) + float(b @ zy)) / eta
        ux = _ALPHA * (z - ut * gx) + (1.0 - _ALPHA) * ux
        v = _ALPHA * (zy - ut * gy) + (1.0 - _ALPHA) * uy - vs
        head, tail = v[l:l + 1], v[l + 1:]
        t, norm = float(head), float(tail.norm())
        if norm <= t:
            cone = v[l:]
        elif norm <= -t:
            cone = torch.zeros_like(v[l:])
        else:
            a = 0.5 * (t + norm)
            cone = torch.cat([torch.full_like(head, a), (a / norm) * tail])
        uy = torch.cat([v[:l].clamp_min(0.0), cone])
        vs = uy - v
        ubar = _ALPHA * ut + (1.0 - _ALPHA) * tau
        new = max(ubar - kappa, 0.0)
        kappa, tau, it = kappa - ubar + new, new, it + 1
        if it % _CHECK == 0 and tau > 0.0:
            rp = float(((apply(ux) + vs - tau * b) / dv).norm()) / (sb * tau) / nb
            rd = float(((adjoint(uy) + tau * c) / ev).norm()) / (sc * tau) / nc
            cx, by = float(c @ ux) / (sb * sc * tau), float(b @ uy) / (sb * sc * tau)
            if max(rp, rd, abs(cx + by) / (1.0 + abs(cx) + abs(by))) <= case["eps"]:
                status = 1
                break
    return _host(ev * ux / (sb * tau)), _host(dv * uy / (sc * tau)), _host(vs / (dv * sb * tau)), status, it


def _exact_regls(case, seed):
    _, op, b = _regls_data(case, seed)
    rhs = op.adjoint(b)
    if case["kind"] == "dense":
        gram = op.a.t().contiguous() @ op.a
        gram.diagonal().add_(1e-2)
        chol = torch.linalg.cholesky(gram)
        x = torch.cholesky_solve(rhs[:, None], chol)[:, 0]
    else:
        x, _ = _cg(lambda v: 1e-2 * v + op.adjoint(op(v)), torch.zeros_like(rhs), rhs, 1e-14 * float(rhs.norm()), 500)
    return {"x": _host(x), "iters": None}


def exact(case, seed):
    family = case["family"]
    if case.get("precision") == "bf16":
        return None   # (three phases on three operators: no single iteration to repeat)
    if family == "regls":
        return _exact_regls(case, seed)
    if family == "server":
        programs = []
        for r in _server_cases(case, seed):
            _, op, obs = _deconv_data(r, r["seed"])
            programs.append(_deconv_program(op, obs[0]))
    elif family in ("deconv", "noalloc"):
        _, op, obs = _deconv_data(case, seed)
        if case.get("batch", 1) * case["steps"] > 4000:
            return None   # (one instance after the other takes too long)
        programs = [_deconv_program(op, b) for b in obs]
    else:
        _, op, inst = _lasso_data(case, seed)
        programs = [_lasso_program(op, b, lam) for b, lam in inst]
    points = [_admm(p, case) for p in programs]
    out = {name: np.concatenate([p[j] for p in points]) for j, name in enumerate(("x", "y", "s"))}
    return dict(out, status=None, iters=None)
