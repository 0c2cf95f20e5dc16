"""The work that users of this solver have it do, as cases to be timed.

Every case goes through the public entry points (``binding.Plan``,
``binding.Server``) the way a program calls them: the plan (and the server)
is made once and kept, the data of each call is new.  The sizes, kernels and
distributions are those of the five workloads in ``workloads/configs.py`` and
of the fracture driver; grids are powers of two because the library takes no
others, so the ragged sizes are the numbers of requests, sequences and steps.

Solves ask for 1e-10, the default tolerance of ``Plan.solve``, in both
precisions (a mixed solve is certified by FP64 residuals like an FP64 one).
"""

from __future__ import annotations

import math
import time

import numpy as np
import torch

from paper_1305_3625_amd import binding

TOL = 1e-10
PREC = {"fp64": binding.FP64, "mixed": binding.MIXED}


# ---- the cases -------------------------------------------------------------

def listed():
    return [
        # one product on a small grid: what a program that runs its own Krylov
        # loop pays per call; launches and latency
        dict(name="apply small", kind="apply", L=64, padded=1, eps=1e-3, precision="fp64"),
        # one FP64 product at the benchmark's size: residual checks and
        # matrix-free loops of the caller
        dict(name="apply large", kind="apply", L=2048, padded=1, eps=1e-4, precision="fp64"),
        # the periodic L = 64 workload, one solve at a time (latency of the
        # smallest simulation)
        dict(name="solve periodic small", kind="solve", L=64, padded=0, eps=1e-2, precision="fp64", precond=0),
        # the smaller grids of the serving mix, solved one at a time
        dict(name="solve small mixed", kind="solve", L=128, padded=1, eps=1e-3, precision="mixed", precond=0),
        # the padded L = 512 FP64 workload
        dict(name="solve medium fp64", kind="solve", L=512, padded=1, eps=1e-3, precision="fp64", precond=0),
        # the benchmark's workload: padded L = 2048, mixed precision
        dict(name="solve large mixed", kind="solve", L=2048, padded=1, eps=1e-4, precision="mixed", precond=0),
        # the same with the circulant preconditioner, as a user who wants the
        # answer soonest runs it
        dict(name="solve large precond", kind="solve", L=2048, padded=1, eps=1e-4, precision="mixed", precond=1),
        # preconditioned FP64 at the middle size
        dict(name="solve medium precond", kind="solve", L=512, padded=1, eps=1e-3, precision="fp64", precond=1),
        # the largest padded grid (M = 8192)
        dict(name="solve largest mixed", kind="solve", L=4096, padded=1, eps=1e-4, precision="mixed", precond=0),
        # a burst of the serving mix, M in {128, 256, 512, 1024}
        dict(name="serve burst", kind="serve", count=48, eps=1e-3, precision="mixed"),
        # load-stepped sequences side by side through the server (warm starts)
        dict(name="load steps", kind="sequence", L=512, count=8, steps=6, eps=1e-3, precision="mixed"),
        # the fracture driver, preconditioned (warm starts, masked operator)
        dict(name="fracture", kind="fracture", L=512, steps=10, eps=1e-3, precision="mixed", precond=1),
    ]


def draw(rng):
    def pow2(lo, hi):
        return 1 << rng.randint(lo, hi)

    kind = rng.choices(("apply", "solve", "serve", "sequence", "fracture"), (3, 9, 1, 1, 1))[0]
    eps = float("%.4g" % math.exp(rng.uniform(math.log(1e-4), math.log(1e-2))))
    precision = rng.choice(("fp64", "mixed"))
    if kind == "apply":  # the operator in FP64: what a caller's own residuals and loops need
        return dict(kind=kind, L=pow2(4, 11), padded=rng.randint(0, 1), eps=eps, precision="fp64")
    if kind == "solve":
        precond = int(rng.random() < 0.3)
        return dict(kind=kind, L=pow2(4, 11), padded=int(rng.random() < 0.7), eps=eps, precision=precision,
                    precond=precond)
    if kind == "serve":
        return dict(kind=kind, count=rng.randint(5, 48), eps=eps, precision="mixed")
    if kind == "sequence":
        return dict(kind=kind, L=pow2(5, 9), count=rng.randint(1, 8), steps=rng.randint(2, 6), eps=eps,
                    precision="mixed")
    return dict(kind=kind, L=pow2(5, 9), steps=rng.randint(2, 10), eps=eps, precision=precision,
                precond=rng.randint(0, 1))


# ---- inputs ------------------------------------------------------------------

def _spectrum(M, eps):
    """ghat(m, n) = 1 / sqrt(4 - 2 cos(2 pi m / M) - 2 cos(2 pi n / M) + eps) on the GPU, exactly even."""
    m = torch.arange(M, device="cuda", dtype=torch.float64)
    c = torch.cos(torch.minimum(m, M - m) * (2.0 * math.pi / M))
    return torch.rsqrt(4.0 - 2.0 * (c[:, None] + c[None, :]) + eps)


def _plan(L, padded, eps):
    return binding.Plan(L, padded, _spectrum(2 * L if padded else L, eps).cpu().numpy())


def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(seed & 0x7FFFFFFFFFFFFFFF)


def _d(L, padded, g):
    """d ~ U(0.5, 1.5), 30% zeros on the padded grids (broken bonds)."""
    d = torch.rand(L, L, dtype=torch.float64, device="cuda", generator=g) + 0.5
    if padded:
        d[torch.rand(L, L, dtype=torch.float64, device="cuda", generator=g) < 0.3] = 0.0
    return d


def _mix(case):
    """FFT grid of each request of a burst: one of each of {128, 256, 512, 1024}, the others drawn from them with
    p {.4, .3, .2, .1}, in mixed order; the same burst for every seed."""
    r = np.random.default_rng([4, case["count"]])
    sizes = [128, 256, 512, 1024] + r.choice([128, 256, 512, 1024], size=case["count"] - 4, p=[.4, .3, .2, .1]).tolist()
    return [sizes[i] for i in np.argsort(r.random(case["count"]), kind="stable")]


def _data(case, seed):
    """The data of one call, on the GPU (served requests: host arrays)."""
    g = _gen(seed)
    if case["kind"] in ("apply", "solve"):
        L = case["L"]
        d = _d(L, case["padded"], g)
        return d, torch.randn(L, L, dtype=torch.float64, device="cuda", generator=g)
    if case["kind"] == "serve":
        out = []
        for M in _mix(case):
            d = _d(M // 2, 1, g)
            b = torch.rand(M // 2, M // 2, dtype=torch.float64, device="cuda", generator=g)
            out.append((M, d.cpu().numpy(), b.cpu().numpy()))
        return out
    L = case["L"]
    if case["kind"] == "sequence":
        return [torch.rand(L, L, dtype=torch.float64, device="cuda", generator=g).cpu().numpy()
                for _ in range(case["count"])]
    front = torch.arange(L, dtype=torch.float64, device="cuda")[:, None] / L
    return 1e-3 + torch.rand(L, L, dtype=torch.float64, device="cuda", generator=g) + front


def prepare(case, seed):
    """The state of one case.  A server comes before its plans: it is closed first."""
    kind = case["kind"]
    data = _data(case, seed)
    if kind == "serve":
        plans = {M: _plan(M // 2, 1, case["eps"]) for M in (128, 256, 512, 1024)}
        srv = binding.Server(memory_budget=4 << 30)
        sizes = [M for M, _, _ in data]
        for M, p in plans.items():
            srv.reserve(p, sizes.count(M), PREC[case["precision"]])
        return dict(case=case, data=data, server=srv, plans=plans)
    if kind == "sequence":
        plan = _plan(case["L"], 1, case["eps"])
        srv = binding.Server(memory_budget=4 << 30)
        srv.reserve(plan, case["count"], PREC[case["precision"]])
        one = np.ones((case["L"], case["L"]))
        return dict(case=case, data=data, server=srv, plan=plan, one=one)
    plan = _plan(case["L"], case.get("padded", 1), case["eps"])
    if case.get("precond"):
        plan.set_precond(binding.PRECOND_CIRCULANT)
    out = torch.empty(case["L"], case["L"], dtype=torch.float64, device="cuda")
    return dict(case=case, data=data, plan=plan, out=out)


# ---- one pass ----------------------------------------------------------------

def _collect(server, left, take):
    """Polls finished tickets until none of `left` (ticket -> position) is left."""
    out = [None] * len(left)
    while left:
        done = server.completed()
        for ticket in done:
            k = left.pop(ticket)
            out[k] = take(ticket, k)
        if not done:
            time.sleep(2e-4)
    return out


def run(state):
    case, data = state["case"], state["data"]
    kind, prec = case["kind"], PREC[case["precision"]]
    if kind == "apply":
        return state["plan"].apply(data[0], data[1], state["out"], precision=prec)
    if kind == "solve":
        state["plan"].solve(data[0], data[1], state["out"], tol=TOL, precision=prec)
        return state["out"]
    if kind == "serve":
        srv, plans = state["server"], state["plans"]
        left = {srv.submit(plans[M], d, b, tol=TOL, precision=prec)[1]: k for k, (M, d, b) in enumerate(data)}
        return _collect(srv, left, lambda t, k: srv.poll(t, data[k][0] // 2).x)
    if kind == "sequence":
        srv, plan, one, steps = state["server"], state["plan"], state["one"], case["steps"]
        left = {srv.submit_sequence(plan, one, one, t, steps, tol=TOL, precision=prec)[1]: k
                for k, t in enumerate(data)}
        return _collect(srv, left, lambda t, k: srv.poll_sequence(t, case["L"], steps).x[:2])
    _, broken, dbreak, _ = state["plan"].fracture(1.0, data, state["out"], case["steps"], tol=TOL, precision=prec)
    return dict(f=state["out"], broken=broken, dbreak=dbreak)


# ---- what a pass cannot do without --------------------------------------------

def _iterations(case):
    """Iterations of a solve from zero to TOL: the CG bound from the condition number (with the preconditioner the
    operator's spectrum lies within about [0.25, 1.75], whatever eps is)."""
    lo, hi = (0.0 if case.get("padded", 1) else 0.5) + 1 / math.sqrt(8.0 + case["eps"]), 1.5 + case["eps"] ** -0.5
    if case.get("precond"):
        lo, hi = 0.25, 1.75
    return math.ceil(0.5 * math.sqrt(hi / lo) * math.log(2.0 / TOL))


def _product_flops(M):
    """A forward and an inverse real M x M transform (half of 5 n log2 n each) and the multiply."""
    n = M * M
    return 5.0 * n * math.log2(n) + n


def work(case):
    kind = case["kind"]
    if kind == "serve":
        grids = _mix(case)
        return dict(bytes=sum(24.0 * (M // 2) ** 2 for M in grids) + sum(2.0 * M * M for M in set(grids)),
                    flops=sum(_iterations(case) * _product_flops(M) for M in grids))
    L, padded = case["L"], case.get("padded", 1)
    M = 2 * L if padded else L
    # d, b (or x) and the spectrum's quarter read, the result written
    size = 24.0 * L * L + 2.0 * M * M
    if kind == "apply":
        return dict(bytes=size, flops=_product_flops(M))
    solves = case.get("steps", 1) * (case["count"] if kind == "sequence" else 1)
    # the steps after the first start from the previous one's solution: about half the iterations
    iters = _iterations(case) * (solves if solves == 1 else 0.5 * (solves + 1))
    each = 2 if case.get("precond") else 1
    bytes_ = size if kind == "solve" else 2.0 * M * M + 16.0 * L * L * case.get("count", 1)
    return dict(bytes=bytes_, flops=iters * each * _product_flops(M))


# ---- the same in 64 bits, without the library ----------------------------------

def _conv(v, s, M):
    L = v.shape[0]
    return torch.fft.irfft2(s * torch.fft.rfft2(v, s=(M, M)), s=(M, M))[:L, :L]


def _exact_solve(g, d, b, M, keep=None):
    """(diag(d) + C) x = b, on the entries of `keep` if given: circulant-preconditioned CG and one refinement."""
    keep = torch.ones_like(b) if keep is None else keep
    pre = 1.0 / (float(d.mean()) + g)
    x, r = torch.zeros_like(b), keep * b
    top = float(r.norm())
    for goal in (1e-12, 1e-15):
        e, rho_old, p = torch.zeros_like(b), 0.0, None
        for _ in range(200):
            z = keep * _conv(r, pre, M)
            rho = float((r * z).sum())
            p = z if p is None else z + (rho / rho_old) * p
            q = keep * (d * p + _conv(p, g, M))
            a = rho / float((p * q).sum())
            e += a * p
            r = r - a * q
            rho_old = rho
            if float(r.norm()) <= goal * top:
                break
        x = x + e
        r = keep * (b - d * x - _conv(x, g, M))
    return x


def exact(case, seed):
    kind = case["kind"]
    data = _data(case, seed)
    if kind == "serve":
        gs = {M: _spectrum(M, case["eps"])[:, : M // 2 + 1] for M in (128, 256, 512, 1024)}
        return [_exact_solve(gs[M], torch.from_numpy(d).cuda(), torch.from_numpy(b).cuda(), M).cpu().numpy()
                for M, d, b in data]
    L = case["L"]
    M = 2 * L if case.get("padded", 1) else L
    g = _spectrum(M, case["eps"])[:, : M // 2 + 1].contiguous()
    if kind == "apply":
        return data[0] * data[1] + _conv(data[1], g, M)
    if kind == "solve":
        return _exact_solve(g, data[0], data[1], M)
    one = torch.ones(L, L, dtype=torch.float64, device="cuda")
    if kind == "sequence":
        out = []
        for t in data:
            t, d, broken = torch.from_numpy(t).cuda(), one.clone(), []
            for _ in range(case["steps"]):
                x = _exact_solve(g, d, one, M)
                k = int(torch.where(d != 0, x / t, -math.inf).argmax())
                broken.append(k)
                d.view(-1)[k] = 0.0
            out.append((x.cpu().numpy(), np.array(broken, dtype=np.int32)))
        return out
    keep, broken, dbreak = one.clone(), [], []
    for _ in range(case["steps"]):
        f = _exact_solve(g, one, one, M, keep)
        ratio = torch.where(keep != 0, f / data, -math.inf)
        k = int(ratio.argmax())
        broken.append(k)
        dbreak.append(1.0 / float(ratio.view(-1)[k]))
        keep.view(-1)[k] = 0.0
    return dict(f=f, broken=np.array(broken, dtype=np.int32), dbreak=np.array(dbreak))
