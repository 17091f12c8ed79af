"""A closed trajectory's memory goes to one of another batch group, which runs on another
stream, while other groups have rounds in flight: every result is bitwise rd_step's."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_memory_moves_between_running_groups(precision):
    from paper_2305_03945_amd import rd
    rng = np.random.default_rng(11)
    ctx, alone = rd.Context(0), rd.Context(0)
    o = rd.make_opts(tol=1e-6, precision=precision)
    kinds = [("allen_cahn", "periodic"), ("allen_cahn", "neumann"), ("heat", "periodic"), ("heat", "neumann")]

    def start(i, N=256):
        kind, bc = kinds[i % len(kinds)]
        p = rd.make_problem(kind, N, bc=bc, diff=(1e-4,))
        u = torch.tensor(rng.uniform(-0.1, 0.1, (N, N)), device="cuda")
        t = ctx.open(p, o, u)
        return t, p, u, [t.submit(1e-3) for _ in range(3)]

    def check(t, p, u, tickets):
        for k in tickets:
            u, ref = alone.step(u, 1e-3, p, o)
            info = ctx.poll(k)
            assert info["status"] == "ok" and info["iters"] == ref["iters"]
        assert torch.equal(t.read(), u)
        t.close()

    live = [start(i) for i in range(4)]
    for i in range(4, 12):
        ctx.pump()                           # rounds of every group are in flight
        live.pop(0)[0].close()               # its steps are dropped, its memory kept
        live.append(start(i + i // 4))       # taken by a trajectory of another group
    while any(ctx.poll(k) is None for run in live for k in run[3]):
        ctx.pump()
    for run in live:
        check(*run)
    assert ctx.serve_stats()["resident_bytes"] == 0
    ctx.close()
    alone.close()
