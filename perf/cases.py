"""Performance cases of the Anderson-acceleration library: whole calls through
its public entry points, from one small solve to vectors of 2^26 entries.

``listed()`` names the cases that are tracked, ``draw(rng)`` gives others of
the same ranges, ``prepare``/``run`` set one up and take one pass through it,
``work`` states the bytes and operations a pass cannot do without and
``exact`` the same outputs in 64-bit torch arithmetic.
"""
from __future__ import annotations

import math

import torch

from paper_2110_09667_amd import aa

F64 = torch.float64
FUSED = aa.FUSE_RHS | aa.FUSE_DELETE
VARIANTS = ["mgs", "cgs2", "dcgs2", "icwy", "dcgs2_lag"]


# --------------------------------------------------------------------------
# the cases
# --------------------------------------------------------------------------

def listed():
    return [
        # A small 2D problem inside a larger program: every launch counts.
        _solve("tiny 2d 24^2 m3 mgs", 2, 24, 3, "mgs", 0, 12),
        # The 1D Poisson solve (linear, n = 4096, m = 5) of the parity and
        # latency workload: one workgroup per step.
        _solve("poisson1d 4096 m5 icwy", 1, 4096, 5, "icwy", 0, 40),
        # The 3D nonlinear problem at the sizes where an iteration is a chain
        # of short dependent passes: a coarse grid, and a ragged middle one
        # with both pass fusions.
        _solve("cube 32^3 m10 icwy", 3, 32, 10, "icwy", 0, 20),
        _solve("cube 101^3 m20 dcgs2 fused", 3, 101, 20, "dcgs2", FUSED, 24),
        # The 3D benchmark itself: 256^3 unknowns, window of 20.
        _solve("cube 256^3 m20 icwy", 3, 256, 20, "icwy", 0, 24),
        # Streaming least squares: a window of 50 columns of odd length is
        # filled, then slides (QRDelete, QRAdd, solve).
        _window("window 3000001 k50 cgs2", 3_000_001, 50, 6, "cgs2", 0),
        # The QRAdd microbenchmark: twenty columns of 2^26 entries.
        _window("qradd 2^26 k20 icwy", 1 << 26, 20, 1, "icwy", 0),
        # The paper's EM mixture: 100,000 samples, 1.5 million entries.
        _em("em 1.5M m3 mgs", 500_000, 100_000, 3, "mgs", 10),
        # The 2D heat equation (term 1) on the paper's 1024^2 grid, each map
        # evaluation a multigrid-preconditioned conjugate-gradient solve ...
        _pde("heat 1024^2 m5 icwy", aa.PDE_HEAT_NL1, 1024, 5, "icwy", 5),
        # ... and the Bratu problem on a small grid, where it is all latency.
        _pde("bratu 96^2 m8 cgs2", aa.PDE_BRATU, 96, 8, "cgs2", 5),
        # Many independent 2D instances of uneven size (the batched table's
        # recipe), windows filling and then recycling.
        _batch("batch 512 icwy fused", "plain", 512, 32, 512, "icwy", FUSED, 24),
        # Training the mixing-weight network along plain trajectories.
        _batch("train 256 icwy", "train", 256, 8, 32, "icwy", 0, 6),
    ]


def draw(rng):
    kind = rng.choice(["solve", "solve", "solve", "window", "window", "em", "pde", "pde",
                       "batch", "batch"])
    if kind == "solve":
        dim = rng.choice([1, 2, 3])
        s = {1: _log(rng, 64, 200_000), 2: _log(rng, 12, 2048), 3: _log(rng, 8, 176)}[dim]
        m = rng.randint(2, 20)
        variant = rng.choice(VARIANTS)
        c = _solve("", dim, s, m, variant, _flags(rng, variant), min(m, 12) + rng.randint(3, 6))
    elif kind == "window":
        n = _log(rng, 1000, 1 << 24)
        k = rng.randint(2, min(62, max(2, (1 << 28) // n)))
        variant = rng.choice(VARIANTS)
        c = _window("", n, k, rng.randint(1, 6), variant, _flags(rng, variant) & ~FUSED)
    elif kind == "em":
        c = _em("", _log(rng, 1, 700_000), _log(rng, 1000, 1_000_000), rng.randint(2, 3),
                rng.choice(VARIANTS), rng.randint(6, 12))
    elif kind == "pde":
        N = rng.choice([o << j for o in range(3, 32, 2) for j in range(0, 9) if 12 <= o << j <= 1024])
        problem = rng.choice([aa.PDE_HEAT_NL1, aa.PDE_HEAT_NL2, aa.PDE_BRATU])
        c = _pde("", problem, N, rng.randint(2, 10), rng.choice(VARIANTS), rng.randint(2, 5))
    else:
        mode = rng.choice(["plain", "plain", "learned", "train"])
        lo = _log(rng, 8, 64)
        variant = rng.choice(VARIANTS[:4])
        c = _batch("", mode, _log(rng, 1, 512), lo, lo * rng.randint(1, 6), variant,
                   rng.choice([0, aa.FUSE_RHS, aa.FUSE_DELETE, FUSED]), rng.randint(4, 16))
    del c["name"]
    return c


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _flags(rng, variant):
    f = rng.choice([0, 0, aa.FUSE_RHS, FUSED])
    if variant == "icwy" and rng.random() < 0.3:
        f = (f & ~aa.FUSE_DELETE) | aa.ICWY_T_TRANSFORM
    if variant == "dcgs2_lag":
        f &= ~aa.FUSE_DELETE
    return f


def _solve(name, dim, s, m, variant, flags, iters):
    return dict(name=name, kind="solve", dim=dim, s=s, m=m, variant=variant, flags=flags, iters=iters)


def _window(name, n, k, slides, variant, flags):
    return dict(name=name, kind="window", n=n, k=k, slides=slides, variant=variant, flags=flags)


def _em(name, replicas, samples, m, variant, iters):
    return dict(name=name, kind="em", replicas=replicas, samples=samples, m=m, variant=variant,
                iters=iters)


def _pde(name, problem, N, m, variant, iters):
    return dict(name=name, kind="pde", problem=problem, N=N, m=m, variant=variant, iters=iters)


def _batch(name, mode, count, lo, hi, variant, flags, iters):
    return dict(name=name, kind="batch", mode=mode, count=count, lo=lo, hi=hi, variant=variant,
                flags=flags, iters=iters)


# --------------------------------------------------------------------------
# inputs and state
# --------------------------------------------------------------------------

def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed))


def _uniform(g, n):
    return torch.rand(n, dtype=F64, device="cuda", generator=g)


def _stencil(dim, s):
    """Spacing and relaxation weight 0.9 / lambda_max of the Dirichlet Laplacian."""
    h = 1.0 / (s + 1)
    lam = dim * (4.0 / (h * h)) * math.cos(math.pi / (2.0 * (s + 1))) ** 2
    return h, 0.9 / lam


def prepare(case, seed):
    return {"solve": _prepare_solve, "window": _prepare_window, "em": _prepare_em,
            "pde": _prepare_pde, "batch": _prepare_batch}[case["kind"]](case, seed)


def _solve_inputs(case, seed):
    n = case["s"] ** case["dim"]
    f = _uniform(_gen(seed), n)
    if case["dim"] == 1:
        f = 2.0 * f - 1.0                       # the linear problem's right-hand side
    c = 0.0 if case["dim"] == 1 else 1.0
    return n, f, c


def _prepare_solve(case, seed):
    n, f, c = _solve_inputs(case, seed)
    h, omega = _stencil(case["dim"], case["s"])
    x = torch.zeros(n, dtype=F64, device="cuda")
    return dict(case=case, ctx=aa.AAContext(n, case["m"], case["variant"], case["flags"]), f=f,
                x=x, g=torch.empty_like(x), h=h, omega=omega, c=c)


def _window_inputs(case, seed):
    """Gaussian columns and right-hand side."""
    g = _gen(seed)
    V = torch.empty((case["k"] + case["slides"], case["n"]), dtype=F64, device="cuda")
    for v in V:
        v.normal_(generator=g)
    return V, torch.randn(case["n"], dtype=F64, device="cuda", generator=g)


def _prepare_window(case, seed):
    V, f = _window_inputs(case, seed)
    k = case["k"]
    ctx = aa.AAContext(case["n"], k, case["variant"], case["flags"] | aa.QR_ONLY)
    return dict(case=case, ctx=ctx, V=V, f=f, gamma=torch.zeros(k, dtype=F64, device="cuda"))


EM_ALPHA, EM_SIGMA, EM_MU = (0.3, 0.3, 0.4), (1.0, 1.0, 1.0), (0.0, 0.5, 1.0)


def _em_inputs(case, seed):
    g = _gen(seed)
    u = _uniform(g, case["samples"])
    z = torch.randn(case["samples"], dtype=F64, device="cuda", generator=g)
    comp = (u > EM_ALPHA[0]).to(F64) + (u > EM_ALPHA[0] + EM_ALPHA[1]).to(F64)
    x = z + 0.5 * comp                           # means 0, 0.5 and 1, deviations 1
    srt = torch.sort(x).values
    u0 = torch.stack([srt[int(q * (x.numel() - 1))] for q in (1 / 6, 1 / 2, 5 / 6)])
    return x, u0.repeat(case["replicas"])


def _prepare_em(case, seed):
    samples, u0 = _em_inputs(case, seed)
    return dict(case=case, ctx=aa.AAContext(u0.numel(), case["m"], case["variant"], 0),
                samples=samples, u0=u0, x=torch.empty_like(u0), g=torch.empty_like(u0),
                work=torch.empty(aa.EM_WORK_DOUBLES, dtype=F64, device="cuda"))


def _c_term(problem, u):
    if problem == aa.PDE_HEAT_NL1:
        eu = torch.exp(u)
        return u + u * eu + u * torch.exp(-u) + (u - eu) ** 2
    return 100.0 * (u - u * u)


def _pde_inputs(case, seed):
    """Source of the manufactured solution a sin^2(pi x) sin^2(pi y) (heat),
    parameter lambda and a smooth start (Bratu)."""
    N = case["N"]
    r = _uniform(_gen(seed), 2).tolist()
    a, lam = 0.75 + 0.5 * r[0], 5.0 + r[1]
    t = torch.arange(1, N + 1, dtype=F64, device="cuda") / (N + 1)
    s2, c2 = torch.sin(math.pi * t) ** 2, torch.cos(math.pi * t) ** 2
    d2 = 2 * math.pi ** 2 * (c2 - s2)
    if case["problem"] == aa.PDE_BRATU:
        return None, lam, (0.1 * a * s2[:, None] * s2[None, :]).reshape(-1)
    u = a * s2[:, None] * s2[None, :]
    lap = a * (d2[:, None] * s2[None, :] + s2[:, None] * d2[None, :])
    return (lap + _c_term(case["problem"], u)).reshape(-1), lam, torch.zeros(N * N, dtype=F64, device="cuda")


def _prepare_pde(case, seed):
    b, lam, u0 = _pde_inputs(case, seed)
    return dict(case=case, ctx=aa.AAContext(u0.numel(), case["m"], case["variant"], 0), b=b, u0=u0,
                pde=aa.PDE2D(case["N"], case["problem"], lam=lam), x=torch.empty_like(u0),
                g=torch.empty_like(u0))


def _batch_table(case):
    """Side, window and cubic coefficient of each instance: sides spread over
    [lo, hi] logarithmically, windows over 3..20."""
    lo, hi = case["lo"], max(case["lo"], case["hi"])
    tab = []
    for j in range(case["count"]):
        u, v, c = ((j + 0.5) * q % 1.0 for q in (0.6180339887498949, 0.4142135623730951, 0.7320508075688772))
        tab.append((int(round(lo * (hi / lo) ** u)), 3 + int(18 * v), c))
    return tab


def _batch_inputs(case, seed):
    offs, tot = [], 0
    for s, _, _ in _batch_table(case):
        offs.append(tot)
        tot += (s * s + 1) // 2 * 2              # instances start on 16 bytes
    return offs, _uniform(_gen(seed), tot)


def _prepare_batch(case, seed):
    offs, f = _batch_inputs(case, seed)
    x = torch.zeros_like(f)
    insts = []
    for (s, m, c), o in zip(_batch_table(case), offs):
        h, omega = _stencil(2, s)
        insts.append(aa.BatchInstance(s * s, m, 2, s, h, omega, c, f.data_ptr() + 8 * o,
                                      x.data_ptr() + 8 * o))
    variant = aa.VARIANTS[case["variant"]]
    flags = case["flags"] | (aa.BATCH_LEARNED if case["mode"] != "plain" else 0)
    nbytes = aa.aa_batch_workspace_size(insts, variant, flags)
    st = dict(case=case, f=f, x=x, insts=insts, variant=variant, flags=flags,
              stream=torch.cuda.Stream(),
              workspace=torch.empty((nbytes + 7) // 8, dtype=F64, device="cuda"))
    if case["mode"] != "plain":
        st["net"] = aa.AAMlp(case["count"], seed=seed, stream=st["stream"])
        st["params"] = _net_params(st["net"], seed)
    st["stream"].wait_stream(torch.cuda.current_stream())
    return st


def _net_params(net, seed):
    """The library's initialization with a small seeded last layer, as a few
    training steps leave it."""
    p = net.get_params()
    w3 = 3 * (256 * 256 + 256)
    g = torch.Generator().manual_seed(int(seed))
    w = torch.zeros(256, 64)
    w[:, :aa.MLP_OUTPUTS] = 1e-3 * torch.randn(256, aa.MLP_OUTPUTS, generator=g)
    p[w3:w3 + 256 * 64] = w.reshape(-1).numpy()
    return p


# --------------------------------------------------------------------------
# one pass
# --------------------------------------------------------------------------

def run(state):
    return {"solve": _run_solve, "window": _run_window, "em": _run_em, "pde": _run_pde,
            "batch": _run_batch}[state["case"]["kind"]](state)


def _run_solve(st):
    """A solve of the model problem from x_0 = 0, one G evaluation a step."""
    case, ctx, x, g = st["case"], st["ctx"], st["x"], st["g"]
    ctx.reset()
    x.zero_()
    for _ in range(case["iters"] + 1):
        aa.aa_problem_apply(case["dim"], case["s"], st["h"], st["omega"], st["c"], st["f"], x, g)
        ctx.step(x, g, x)
    return {"x": x, "g": g, "status": int(ctx.info().status)}


def _run_window(st):
    """Fill the window column by column, slide it, solve after every slide."""
    case, ctx, V, gamma = st["case"], st["ctx"], st["V"], st["gamma"]
    k = case["k"]
    ctx.reset()
    for j in range(k):
        ctx.qr_add(V[j])
    ctx.qr_solve(st["f"], gamma)
    for j in range(k, k + case["slides"]):
        ctx.qr_delete()
        ctx.qr_add(V[j])
        ctx.qr_solve(st["f"], gamma)
    return {"gamma": gamma, "Q": ctx.basis(k).T}


def _run_em(st):
    case, ctx, x, g = st["case"], st["ctx"], st["x"], st["g"]
    ctx.reset()
    x.copy_(st["u0"])
    for _ in range(case["iters"] + 1):
        aa.aa_em_apply(EM_ALPHA, EM_SIGMA, st["samples"], x, g, st["work"])
        ctx.step(x, g, x)
    return {"x": x, "g": g}


def _run_pde(st):
    case, ctx, pde, x, g = st["case"], st["ctx"], st["pde"], st["x"], st["g"]
    ctx.reset()
    x.copy_(st["u0"])
    for _ in range(case["iters"] + 1):
        pde.apply(st["b"], x, g)
        ctx.step(x, g, x)
    return {"x": x, "g": g}


def _run_batch(st):
    """A new batch over kept memory: start, iterate, read the states."""
    case = st["case"]
    with torch.cuda.stream(st["stream"]):
        st["x"].zero_()
        b = aa.aa_batch_init(st["insts"], st["variant"], st["flags"], 1e-8, 5000, st["workspace"],
                             st["stream"])
        out = {"x": st["x"]}
        if case["mode"] == "plain":
            for _ in range(case["iters"] // 4):
                aa.aa_batch_run(b, 4)
            aa.aa_batch_run(b, case["iters"] % 4 + 1)
        else:
            net = st["net"]
            net.set_params(st["params"])
            go = aa.lib().aa_batch_run_learned if case["mode"] == "learned" else aa.lib().aa_batch_train
            args = () if case["mode"] == "learned" else (1e-3,)
            if go(b, net.net, case["iters"] + 1, *args) != 0:
                raise RuntimeError("the learned batch failed")
            if case["mode"] == "train":
                out["params"] = net.get_params()
        states, out["active"] = aa.aa_batch_read(b, case["count"])
        out["k"] = torch.tensor([s.k for s in states])
        aa.aa_batch_destroy(b)
    return out


# --------------------------------------------------------------------------
# what a pass cannot do without
# --------------------------------------------------------------------------

def _aa_work(n, m, iters):
    """Steps of Alg. 1: x, G(x), the previous pair, Q and the history read
    once, the new vectors and the rotated basis written once."""
    vecs = flops = 0.0
    for i in range(iters + 1):
        k = min(i, m)
        vecs += 3 if i == 0 else 4 + 4 + 2 * k + (k if i > m else 1)
        flops += 2.0 * n * 6 * k
    return {"bytes": 8.0 * n * vecs, "flops": flops}


def work(case):
    kind = case["kind"]
    if kind == "solve":
        n = case["s"] ** case["dim"]
        w = _aa_work(n, case["m"], case["iters"])
        g = case["iters"] + 1
        return {"bytes": w["bytes"] + 24.0 * n * g, "flops": w["flops"] + (4 * case["dim"] + 8.0) * n * g}
    if kind == "window":
        n, k, s = case["n"], case["k"], case["slides"]
        vecs = sum(j + 2 for j in range(k)) + (k + 1) + s * (2 * k + 4)
        return {"bytes": 8.0 * n * vecs, "flops": 4.0 * n * k * k / 2 + s * 2.0 * n * 6 * k}
    if kind == "em":
        n, g = 3 * case["replicas"], case["iters"] + 1
        w = _aa_work(n, case["m"], case["iters"])
        return {"bytes": w["bytes"] + 8.0 * (n + case["samples"]) * g,
                "flops": w["flops"] + 100.0 * case["samples"] * g}
    if kind == "pde":
        n, g = case["N"] ** 2, case["iters"] + 1
        w = _aa_work(n, case["m"], case["iters"])
        # ten conjugate-gradient iterations an evaluation; each reads and
        # writes x, r, p, q and takes one cycle (r read, z written)
        return {"bytes": w["bytes"] + g * 10 * 8.0 * 10 * n, "flops": w["flops"] + g * 10 * 60.0 * n}
    tot = {"bytes": 0.0, "flops": 0.0}
    for s, m, _ in _batch_table(case):
        w = _aa_work(s * s, m, case["iters"])
        tot["bytes"] += w["bytes"] + 24.0 * s * s * (case["iters"] + 1)
        tot["flops"] += w["flops"] + 16.0 * s * s * (case["iters"] + 1)
    if case["mode"] != "plain":
        per = 2.0 * (3 * 256 * 256 + 256 * 64) * (3 if case["mode"] == "train" else 1)
        tot["flops"] += per * case["count"] * (case["iters"] + 1)
    return tot


# --------------------------------------------------------------------------
# the same in 64-bit torch
# --------------------------------------------------------------------------

def _dots(A, B):
    """A^T B, a million rows at a time."""
    rows = range(0, A.shape[0], 1 << 20)
    return sum(A[r:r + (1 << 20)].T @ B[r:r + (1 << 20)] for r in rows)


def _orthonormal(F):
    """Q and R of an n x k matrix (R with a positive diagonal)."""
    if F.shape[0] * F.shape[1] <= 1 << 20:
        Q, R = torch.linalg.qr(F)
        sg = torch.sign(torch.diagonal(R))
        return Q * sg, R * sg[:, None]
    eye = torch.eye(F.shape[1], dtype=F64, device=F.device)
    R, Q = eye, F
    for _ in range(2):
        L = torch.linalg.cholesky(_dots(Q, Q))
        inv = torch.linalg.solve_triangular(L, eye, upper=False).T
        Q = torch.cat([q @ inv for q in Q.split(1 << 20)])
        R = L.T @ R
    return Q, R


def _aa_exact(G, x, m, iters):
    g = G(x)
    f = g - x
    x = g
    dF, dG = [], []
    for _ in range(iters):
        gp, fp = g, f
        g = G(x)
        f = g - x
        dF, dG = (dF + [f - fp])[-m:], (dG + [g - gp])[-m:]
        Q, R = _orthonormal(torch.stack(dF, 1))
        c = _dots(Q, f[:, None])
        gam = torch.linalg.solve_triangular(R, c, upper=True)[:, 0]
        x = g - sum(d * c for d, c in zip(dG, gam))
    return x, g


def _stencil_map(dim, s, h, omega, c, f):
    shape = (s,) * dim

    def G(u):
        v = u.reshape(shape)
        a = 2.0 * dim * v
        for d in range(dim):
            lo, hi = [slice(None)] * dim, [slice(None)] * dim
            lo[d], hi[d] = slice(0, s - 1), slice(1, s)
            a[tuple(hi)] -= v[tuple(lo)]
            a[tuple(lo)] -= v[tuple(hi)]
        return u - omega * (a.reshape(-1) / (h * h) + c * u ** 3 - f)
    return G


def exact(case, seed):
    kind = case["kind"]
    if kind == "solve":
        n, f, c = _solve_inputs(case, seed)
        h, omega = _stencil(case["dim"], case["s"])
        x, g = _aa_exact(_stencil_map(case["dim"], case["s"], h, omega, c, f), torch.zeros_like(f),
                         case["m"], case["iters"])
        return {"x": x, "g": g, "status": None}
    if kind == "window":
        V, f = _window_inputs(case, seed)
        Q, R = _orthonormal(V[case["slides"]:].T)
        gam = torch.linalg.solve_triangular(R, _dots(Q, f[:, None]), upper=True)[:, 0]
        return {"gamma": gam, "Q": Q.T}
    if kind == "em":
        samples, u0 = _em_inputs(case, seed)
        al, sg = (torch.tensor(v, dtype=F64, device="cuda") for v in (EM_ALPHA, EM_SIGMA))

        def G(u):
            p = al / sg * torch.exp(-(samples[:, None] - u[:3]) ** 2 / (2 * sg * sg))
            w = p / p.sum(1, keepdim=True)
            return ((w * samples[:, None]).sum(0) / w.sum(0)).repeat(u.numel() // 3)
        x, g = _aa_exact(G, u0, case["m"], case["iters"])
        return {"x": x, "g": g}
    if kind == "pde":
        b, lam, u0 = _pde_inputs(case, seed)
        N = case["N"]
        j = torch.arange(1, N + 1, dtype=F64, device="cuda")
        S = math.sqrt(2.0 / (N + 1)) * torch.sin(math.pi / (N + 1) * ((j[:, None] * j) % (2 * N + 2)))
        ev = 4.0 * (N + 1) ** 2 * torch.sin(j * math.pi / (2 * (N + 1))) ** 2

        def G(u):
            r = lam * torch.exp(u) if b is None else _c_term(case["problem"], u) - b
            return (S @ ((S @ r.reshape(N, N) @ S) / (ev[:, None] + ev)) @ S).reshape(-1)
        x, g = _aa_exact(G, u0, case["m"], case["iters"])
        return {"x": x, "g": g}
    if case["mode"] == "learned" or case["count"] * case["iters"] > 2000:
        return None
    offs, f = _batch_inputs(case, seed)
    x = torch.zeros_like(f)
    for (s, m, c), o in zip(_batch_table(case), offs):
        h, omega = _stencil(2, s)
        fj = f[o:o + s * s]
        x[o:o + s * s] = _aa_exact(_stencil_map(2, s, h, omega, c, fj), torch.zeros_like(fj), m,
                                   case["iters"])[0]
    return {"x": x, "params": None, "active": None, "k": None}
