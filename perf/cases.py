"""The work that a user of this library has it do: implicit steps through
``Context.step``, over the equations, grids and precisions of the repository's
workloads and paper examples, and a batch of serving requests.

A case is a plain dict.  ``op`` is "step" (one implicit step on one grid) or
"serve" (a mixed batch of trajectories, opened, advanced and closed).
"""
import math

import numpy as np
import torch

# Equation parameters of the repository's workloads on the unit square.
AC = dict(kind="allen_cahn", L=1.0, d0=0.01 ** 2, d1=0.0, b=1.0, a=0.0, sb=0.0, kappa=1.0, tau=0.9)
CH = dict(kind="cahn_hilliard", L=1.0, d0=0.02 ** 2, d1=0.0, b=1.0, a=0.0, sb=0.0, kappa=1.0, tau=0.7)
SCHNAK = dict(kind="schnakenberg", L=1.0, d0=1.0, d1=10.0, b=0.0, a=0.1, sb=0.9, kappa=1.0, tau=0.9)
FCH = dict(kind="fch", L=2.0 * math.pi, d0=0.18 ** 2, d1=0.0, b=0.0, a=0.0, sb=0.0, kappa=1.0, tau=0.58)


def step_case(base, N, precision, ht, tol, bc="periodic", dim=2, init="noise", amp=0.1, **over):
    c = dict(base, op="step", N=N, dim=dim, bc=bc, precision=precision, ht=ht, tol=tol, init=init, amp=amp)
    c.update(over)
    return c


def listed():
    def named(name, c):
        return dict(c, name=name)

    return [
        # The smallest calls: a 64^2 grid solved to 1e-10, in both precisions (latency).
        named("ac64_fp64", step_case(AC, 64, "fp64", 1e-2, 1e-10, amp=0.9, d0=0.05 ** 2)),
        named("ac64_mixed", step_case(AC, 64, "mixed", 1e-2, 1e-10, amp=0.9, d0=0.05 ** 2)),
        # The paper's own examples at their 128^2 size: Schnakenberg with kappa = 100 on a
        # Neumann grid, and the sixth-order FCH equation (hundreds of iterations a step).
        named("schnak128_fp64", step_case(SCHNAK, 128, "fp64", 2e-4, 1e-7, bc="neumann", init="bump", amp=1e-3,
                                          d0=0.05, d1=1.0, a=0.1305, sb=0.7695, kappa=100.0)),
        named("fch128_fp64", step_case(FCH, 128, "fp64", 1e-3, 5e-6, init="fch", amp=1.0)),
        # Ordinary grids of phase-field and pattern runs.
        named("ch512_neumann_fp64", step_case(CH, 512, "fp64", 1e-4, 1e-2, bc="neumann", amp=0.05)),
        named("schnak1024_fp64", step_case(SCHNAK, 1024, "fp64", 1e-3, 1e-4, init="steady", amp=0.01)),
        named("schnak1024_mixed", step_case(SCHNAK, 1024, "mixed", 1e-3, 1e-4, init="steady", amp=0.01)),
        # Large grids: the headline 2048^2 Allen-Cahn step in both precisions, and 4096^2,
        # whose fields exceed the last-level cache.
        named("ac2048_fp64", step_case(AC, 2048, "fp64", 1e-3, 1e-6)),
        named("ac2048_mixed", step_case(AC, 2048, "mixed", 1e-3, 1e-6)),
        named("ac4096_mixed", step_case(AC, 4096, "mixed", 1e-3, 1e-6)),
        # A 3-D grid.
        named("ac3d128_mixed", step_case(AC, 128, "mixed", 1e-3, 1e-6, dim=3)),
        # Continuous batching: trajectories of every equation and several sizes arrive
        # together, take a few steps each and leave.
        dict(name="serve_mix", op="serve", n_traj=18, steps=3, max_n=512, ht=1e-3),
    ]


def draw(rng):
    """One more case: an equation, a grid and a precision that the listed ones stand for."""
    def logu(lo, hi):
        return float("%.4g" % math.exp(rng.uniform(math.log(lo), math.log(hi))))

    which = rng.choice(["ac", "ac", "ac", "schnak", "schnak", "ch", "fch", "ac3d", "serve"])
    bc = rng.choice(["periodic", "neumann"])
    precision = rng.choice(["fp64", "mixed"])
    if which == "ac":
        N = rng.choice([16, 32, 64, 128, 256, 512, 1024, 2048, 4096])
        # the tolerance of the small grids is the 64^2 workload's order, of the others the 2048^2 one's
        return step_case(AC, N, precision, logu(1e-4, 1e-3), 1e-8 if N <= 128 else 1e-6, bc=bc,
                         amp=rng.choice([0.1, 0.5, 0.9]), d0=logu(0.01 ** 2, 0.05 ** 2))
    if which == "schnak":
        N = rng.choice([32, 64, 128, 256, 512, 1024])
        return step_case(SCHNAK, N, precision, logu(2e-4, 1e-3), 1e-4 * (N / 1024.0) ** 2, bc=bc, init="steady",
                         amp=0.01)
    if which == "ch":
        # FP64: the faster precision for this equation, and the one whose result is not set by
        # the round-off floor of the other's inner loop
        N = rng.choice([32, 64, 128, 256, 512])
        return step_case(CH, N, "fp64", logu(5e-5, 1e-4), 1e-2, bc=bc, amp=0.05)
    if which == "fch":
        N = rng.choice([32, 64, 128])
        return step_case(FCH, N, "fp64" if N == 128 else precision, logu(5e-4, 1e-3), 5e-6, bc="periodic", init="fch",
                         amp=1.0)
    if which == "ac3d":
        return step_case(AC, rng.choice([16, 32, 64, 128]), precision, logu(1e-4, 1e-3), 1e-6, bc=bc, dim=3,
                         d0=logu(0.01 ** 2, 0.05 ** 2))
    return dict(op="serve", n_traj=rng.randint(4, 18), steps=rng.randint(1, 3), max_n=rng.choice([128, 256, 512]),
                ht=logu(5e-4, 1e-3))


# ---------------------------------------------------------------- inputs
def field(c, seed, gen=None):
    """The initial state of a step, FP64, on the GPU where there is one."""
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    if gen is None:
        gen = torch.Generator(device="cpu").manual_seed(int(seed))
    N, dim = c["N"], c["dim"]
    shape = (N,) * dim

    def uniform(shape, amp):
        if math.prod(shape) <= 1 << 20 or dev == "cpu":
            return (torch.rand(shape, generator=gen, dtype=torch.float64) * 2 - 1).mul_(amp).to(dev)
        big = torch.Generator(device=dev).manual_seed(int(torch.randint(1 << 40, (1,), generator=gen)))
        return (torch.rand(shape, generator=big, dtype=torch.float64, device=dev) * 2 - 1).mul_(amp)

    if c["init"] == "noise":
        return uniform(shape, c["amp"])
    if c["init"] == "steady":
        # the steady state with noise
        u = c["a"] + c["sb"] + uniform(shape, c["amp"])
        v = c["sb"] / (c["a"] + c["sb"]) ** 2 + uniform(shape, c["amp"])
        return torch.stack([u, v])
    r = torch.rand(4, generator=gen, dtype=torch.float64).tolist()
    if c["init"] == "bump":
        # Sec. 3.4.1 of the paper: the steady state with a Gaussian bump on u, its place and height drawn
        x = (torch.arange(N, dtype=torch.float64, device=dev) + 0.5) / N
        Y, X = torch.meshgrid(x, x, indexing="ij")
        cx, cy = 0.3 + 0.4 * r[0], 0.3 + 0.4 * r[1]
        u = c["a"] + c["sb"] + c["amp"] * (0.5 + r[2]) * torch.exp(-100 * ((X - cx) ** 2 + (Y - cy) ** 2))
        return torch.stack([u, torch.full_like(u, c["sb"] / (c["a"] + c["sb"]) ** 2)])
    # Sec. 3.3 of the paper: two bumps on the periodic square, shifted by a drawn phase
    x = torch.arange(N, dtype=torch.float64, device=dev) * (c["L"] / N)
    Y, X = torch.meshgrid(x + c["L"] * r[0], x + c["L"] * r[1], indexing="ij")
    s = torch.sin(X) + torch.sin(Y)
    return 2 * torch.exp(s - 2) + (2.1 + 0.1 * r[2]) * torch.exp(-s - 2) - 1


def requests(c, seed):
    """The trajectories of a serving batch: (step case, initial state)."""
    rng = np.random.default_rng(int(seed))
    sizes = [n for n in (64, 128, 256, 512) if n <= c["max_n"]]
    out = []
    for i in range(c["n_traj"]):
        # every equation, size and boundary in turn, so that two batches cost alike
        which, N, bc = i % 3, sizes[(i // 3 + i) % len(sizes)], ("periodic", "neumann")[(i // 2) % 2]
        if which == 0:
            s = step_case(AC, N, "mixed", c["ht"], 1e-8 if N <= 128 else 1e-6, bc=bc)
        elif which == 1:
            s = step_case(CH, N, "fp64", 1e-4, 1e-2, bc=bc, amp=0.05)
        else:
            s = step_case(SCHNAK, N, "mixed", c["ht"], 1e-4 * (N / 1024.0) ** 2, bc=bc, init="steady", amp=0.01)
        out.append((s, field(s, int(rng.integers(1 << 40)))))
    return out


# ---------------------------------------------------------------- the calls
def problem_and_opts(c):
    from paper_2305_03945_amd import rd
    p = rd.make_problem(c["kind"], c["N"], L=c["L"], bc=c["bc"], diff=(c["d0"], c["d1"]) if c["d1"] else (c["d0"],),
                        b=c["b"], a=c["a"], sb=c["sb"], kappa=c["kappa"], dim=c["dim"])
    return p, rd.make_opts(tol=c["tol"], tau_u=c["tau"], tau_p=c["tau"], precision=c["precision"], max_iter=5000)


def prepare(case, seed):
    from paper_2305_03945_amd import rd
    ctx = rd.Context(0)
    if case["op"] == "serve":
        reqs = [problem_and_opts(s) + (u, s["ht"]) for s, u in requests(case, seed)]
        return dict(op="serve", ctx=ctx, reqs=reqs, steps=case["steps"])
    p, o = problem_and_opts(case)
    u = field(case, seed)
    return dict(op="step", ctx=ctx, p=p, o=o, ht=case["ht"], u=u, out=torch.empty_like(u))


def run(state):
    ctx = state["ctx"]
    if state["op"] == "step":
        out, info = ctx.step(state["u"], state["ht"], state["p"], state["o"], out=state["out"])
        if info["status"] != "ok":
            raise RuntimeError("step: %s" % info)
        return out
    trajs = [ctx.open(p, o, u) for p, o, u, _ in state["reqs"]]
    waiting = [t.submit(r[3]) for t, r in zip(trajs, state["reqs"]) for _ in range(state["steps"])]
    while waiting:
        ctx.pump()
        infos = [(t, ctx.poll(t)) for t in waiting]
        for _, info in infos:
            if info is not None and info["status"] != "ok":
                raise RuntimeError("served step: %s" % info)
        waiting = [t for t, info in infos if info is None]
    outs = [t.read() for t in trajs]
    for t in trajs:
        t.close()
    return outs


# ---------------------------------------------------------------- what a pass cannot do without
# Iterations that a step of the equation takes in double precision, about.
ITERATIONS = {"allen_cahn": 30, "schnakenberg": 25, "cahn_hilliard": 80, "fch": 280}


def step_work(c):
    comps = 2 if c["kind"] == "schnakenberg" else 1
    pts = comps * c["N"] ** c["dim"]
    # one forward and one inverse real transform, two stencils and a few updates an iteration
    flops = pts * (2 * 2.5 * c["dim"] * math.log2(c["N"]) + 40) * ITERATIONS[c["kind"]]
    return pts * 16.0, flops


def work(case):
    if case["op"] == "step":
        b, f = step_work(case)
        return {"bytes": b, "flops": f}
    sizes = [n for n in (64, 128, 256, 512) if n <= case["max_n"]]
    b = f = 0.0
    for i in range(case["n_traj"]):
        base = (AC, CH, SCHNAK)[i % 3]
        bi, fi = step_work(dict(base, N=sizes[(i // 3 + i) % len(sizes)], dim=2))
        b, f = b + bi, f + fi * case["steps"]
    return {"bytes": b, "flops": f}


# ---------------------------------------------------------------- the step's root in 64 bits
def laplacian(u, h, dim):
    s = -2.0 * dim * u
    for ax in range(-dim, 0):
        s = s + torch.roll(u, 1, ax) + torch.roll(u, -1, ax)
    return s / (h * h)


def residual_of(c, h, uk):
    """F and the product of its transposed Jacobian, on a periodic grid."""
    ht, dim, lap = c["ht"], c["dim"], lambda v: laplacian(v, h, c["dim"])
    d = c["d0"]
    if c["kind"] == "allen_cahn":
        F = lambda u: u - uk - ht * (d * lap(u) + c["b"] * (u - u ** 3))  # noqa: E731
        J = lambda u, p: p - ht * (d * lap(p) + c["b"] * (1 - 3 * u * u) * p)  # noqa: E731
    elif c["kind"] == "cahn_hilliard":
        F = lambda u: u - uk + ht * lap(d * lap(u) - c["b"] * (u ** 3 - u))  # noqa: E731

        def J(u, p):
            q = lap(p)
            return p + ht * (d * lap(q) - c["b"] * (3 * u * u - 1) * q)
    elif c["kind"] == "fch":
        def F(u):
            m = d * lap(u) - (u ** 3 - u)
            return u - uk - ht * lap(d * lap(m) - (3 * u * u - 1) * m + d * m)

        def J(u, p):
            q, D, B = lap(p), 3 * u * u - 1, d * lap(u) - (u ** 3 - u)
            a = d * lap(q) - D * q + d * q
            return p - ht * (d * lap(a) - D * a) + ht * 6 * u * B * q
    else:
        e, kap = c["d1"], c["kappa"]

        def F(w):
            u, v = w[0], w[1]
            r = u * u * v
            return torch.stack([u - uk[0] - ht * (d * lap(u) + kap * (c["a"] - u + r)),
                                v - uk[1] - ht * (e * lap(v) + kap * (c["sb"] - r))])

        def J(w, p):
            u, v, s = w[0], w[1], p[0] - p[1]
            return torch.stack([p[0] - ht * (d * lap(p[0]) + kap * (-p[0] + 2 * u * v * s)),
                                p[1] - ht * (e * lap(p[1]) + kap * u * u * s)])
    # symbol of A, per component, over the half spectrum
    N = uk.shape[-1]
    s = 4.0 / (h * h) * torch.sin(math.pi * torch.arange(N, dtype=torch.float64, device=uk.device) / N) ** 2
    mu = s[: N // 2 + 1]
    for ax in range(1, dim):
        mu = mu + s.reshape((N,) + (1,) * ax)
    if c["kind"] == "cahn_hilliard":
        A = 1 + ht * d * mu ** 2
    elif c["kind"] == "fch":
        A = 1 + ht * d * mu ** 2 * (d * mu + 2 - d)
    elif c["kind"] == "schnakenberg":
        A = torch.stack([1 + ht * d * mu, 1 + ht * c["d1"] * mu])
    else:
        A = 1 + ht * d * mu
    return F, J, A * A


def root(c, u0):
    """The root of the implicit step, by the same iteration run on to a residual far below the
    tolerance (or to the round-off of 64 bits)."""
    dim, N = c["dim"], c["N"]
    axes = tuple(range(-dim, 0))
    uk = u0
    if c["bc"] == "neumann":  # the half-sample symmetric extension is periodic
        for ax in axes:
            uk = torch.cat([uk, uk.flip(ax)], ax)
    F, J, G = residual_of(c, c["L"] / N, uk)
    u, p = uk.clone(), torch.zeros_like(uk)
    best, since, out = math.inf, 0, u
    for _ in range(6000):
        w = F(u)
        res = float(w.norm())
        if res < best:
            since = 0 if res < 0.95 * best else since + 1
            best, out = res, u
        else:
            since += 1
        if res <= 1e-4 * c["tol"] * c["ht"] or since > 60:
            break
        y = torch.fft.irfftn(torch.fft.rfftn(w, dim=axes) / G, s=[uk.shape[a] for a in axes], dim=axes)
        p = p + c["tau"] * y
        u = u - c["tau"] * J(u, p + c["tau"] * y)
    for ax in axes:
        out = out.narrow(ax, 0, N)
    return out.contiguous()


def exact(case, seed):
    if case["op"] == "step":
        return root(case, field(case, seed))
    outs = []
    for s, u in requests(case, seed):
        for _ in range(case["steps"]):
            u = root(s, u)
        outs.append(u)
    return outs
