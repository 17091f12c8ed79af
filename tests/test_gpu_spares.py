"""Memory of closed trajectories serves later ones of the same shape: a trajectory that
takes over another's workspace and state, of another equation, boundary or precision
history, gives bitwise the results of rd_step alone; and a budget bounds what is kept."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def run_one(rd, ctx, p, o, u, ht, steps):
    t = ctx.open(p, o, u)
    tickets = [t.submit(ht) for _ in range(steps)]
    while any(ctx.poll(k) is None for k in tickets):
        ctx.pump()
    infos = [ctx.poll(k) for k in tickets]
    out = t.read()
    return t, out, infos


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("budget", [0, 1])
def test_reused_memory_gives_the_same_results(precision, budget):
    from paper_2305_03945_amd import rd
    rng = np.random.default_rng(3)
    alone, ctx = rd.Context(0), rd.Context(0)
    # one shape, three equations and two boundaries in turn; the first step of each is long
    # and the next trajectory's short, so a workspace's history must not carry over
    cases = [("allen_cahn", "periodic", (1e-4,), 1e-8), ("cahn_hilliard", "neumann", (4e-4,), 1e-2),
             ("heat", "neumann", (1e-4,), 1e-3), ("allen_cahn", "neumann", (1e-4,), 1e-6)]
    if budget:
        p, o = rd.make_problem("heat", 128), rd.make_opts(precision=precision)
        ctx.set_budget(rd.footprint_bytes(p, o) + (1 << 20))
    for kind, bc, diff, tol in cases * 2:
        p = rd.make_problem(kind, 128, bc=bc, diff=diff)
        tau = 0.7 if kind == "cahn_hilliard" else 0.9
        o = rd.make_opts(tol=tol, tau_u=tau, tau_p=tau, precision=precision)
        u = torch.tensor(rng.uniform(-0.05, 0.05, (128, 128)), device="cuda")
        t, out, infos = run_one(rd, ctx, p, o, u, 1e-4, 2)
        v = u
        for info in infos:
            v, ref = alone.step(v, 1e-4, p, o)
            assert info["status"] == ref["status"] == "ok" and info["iters"] == ref["iters"]
        assert torch.equal(out, v)
        t.close()
        assert ctx.serve_stats()["resident_bytes"] == 0
    ctx.close()
    alone.close()


def test_closed_trajectories_leave_the_others_running():
    """Closing one trajectory waits for its own group only and drops nothing of the others."""
    from paper_2305_03945_amd import rd
    rng = np.random.default_rng(4)
    ctx, alone = rd.Context(0), rd.Context(0)
    o = rd.make_opts(tol=1e-6)
    probs = [rd.make_problem("allen_cahn", n, diff=(1e-4,)) for n in (128, 256, 128)]
    us = [torch.tensor(rng.uniform(-0.1, 0.1, (p.nx, p.nx)), device="cuda") for p in probs]
    ts = [ctx.open(p, o, u) for p, u in zip(probs, us)]
    ks = [t.submit(1e-3) for t in ts]
    ctx.pump()
    ts[0].close()
    with pytest.raises(rd.RDError):
        ctx.poll(ks[0])
    while any(ctx.poll(k) is None for k in ks[1:]):
        ctx.pump()
    for t, p, u in list(zip(ts, probs, us))[1:]:
        assert torch.equal(t.read(), alone.step(u, 1e-3, p, o)[0])
        t.close()
    ctx.close()
    alone.close()
