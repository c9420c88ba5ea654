"""GMRES restarts raised on a live context (swr_set_schedule, a schedule cache):
the workspaces are those of the restart in use, so the solve is bitwise that of
a context made with it."""
import numpy as np
import pytest

from paper_1503_02564_amd import workloads as W
from tests.gpu_util import say, to_dev, to_np

pytestmark = pytest.mark.gpu


def _solve(wl, vkind, restart, raised=None, cache=None):
    import torch
    from paper_1503_02564_amd import swr
    o = swr.swr_default_opts()
    o.batch, o.restart, o.tol, o.precond = wl.B, restart, 1e-12, 0
    if vkind == W.V_STATIC:
        o.solver = swr.SWR_SOLVER_GMRES
    if cache is not None:
        o.tune_cache = cache.encode()
    pb = swr.Problem(wl.a0, wl.b0, tuple(int(j) for j in wl.J), wl.dt, wl.dt * wl.nt, wl.vkind, wl.trans,
                     wl.sigma, o, to_dev(np.asarray(wl.V, np.float64)))
    u0 = to_dev(wl.u0)
    uT = torch.zeros_like(u0)
    g = torch.zeros((wl.B, pb.ns, wl.nt), dtype=torch.complex128, device="cuda")
    if raised is not None:
        swr.swr_set_schedule(pb.ctx, restart=raised)
    st, info = swr.swr_solve(pb.ctx, u0, uT, g)
    assert st == swr.SWR_OK
    out = (to_np(uT), to_np(g), info.iters, info.history)
    pb.close()
    return out


@pytest.mark.parametrize("vkind", [W.V_STATIC, W.V_TIME])
@pytest.mark.parametrize("how", ["set_schedule", "cache"])
def test_restart_raised_after_setup(dev, tmp_path, vkind, how):
    """More inner steps in a cycle than the restart of swr_setup has room for."""
    from paper_1503_02564_amd import swr
    wl = W.small_case(J=[12] * 40, nt=64, vkind=vkind, trans=W.S02, B=2, seed=13, a0=-12.0, b0=12.0)
    want = _solve(wl, vkind, 60)
    assert want[2] > 10                       # (outputs per reduction that a restart of 8 has room for)
    say("restart", vkind, how, "iterations", want[2])
    if how == "set_schedule":
        got = _solve(wl, vkind, 8, raised=60)
    else:
        cache = str(tmp_path / "schedules.txt")
        o = swr.swr_default_opts()
        o.batch, o.restart, o.tune_cache = wl.B, 8, cache.encode()
        if vkind == W.V_STATIC:
            o.solver = swr.SWR_SOLVER_GMRES
        pb = swr.Problem(wl.a0, wl.b0, tuple(int(j) for j in wl.J), wl.dt, wl.dt * wl.nt, wl.vkind, wl.trans,
                         wl.sigma, o, to_dev(np.asarray(wl.V, np.float64)))
        swr.swr_tune(pb.ctx, to_dev(wl.u0), budget_ms=1.0)
        pb.close()
        f = open(cache).read().split()        # key, pipeline, help_max, restart, ...
        f[3] = "60"
        open(cache, "w").write(" ".join(f) + "\n")
        got = _solve(wl, vkind, 8, cache=cache)
    assert got[2] == want[2]
    assert np.array_equal(got[0], want[0]) and np.array_equal(got[1], want[1])
    assert np.array_equal(got[3], want[3])


def test_a_refused_restart_leaves_the_context_usable(dev, monkeypatch):
    """swr_tune goes on to other candidates after one without room: a restart
    whose basis is refused leaves no half of a workspace behind, and restarts
    tried one after the other do not pile up."""
    import torch
    from paper_1503_02564_amd import swr
    wl = W.small_case(J=[12] * 40, nt=64, trans=W.S02, B=2, seed=13, a0=-12.0, b0=12.0)
    o = swr.swr_default_opts()
    o.batch, o.restart, o.tol, o.solver = wl.B, 8, 1e-12, swr.SWR_SOLVER_GMRES
    # a basis of 101 vectors takes 16 MB, one of 4001 640 MB
    monkeypatch.setenv("SWR_DEBUG_ALLOC_LIMIT", str(64 << 20))
    pb = swr.Problem(wl.a0, wl.b0, tuple(int(j) for j in wl.J), wl.dt, wl.dt * wl.nt, wl.vkind, wl.trans,
                     wl.sigma, o, to_dev(np.asarray(wl.V, np.float64)))
    u0 = to_dev(wl.u0)

    def solve():
        uT = torch.zeros_like(u0)
        st, _ = swr.swr_solve(pb.ctx, u0, uT)
        assert st == swr.SWR_OK
        return to_np(uT)

    first = solve()
    say("restart refused")
    swr.swr_set_schedule(pb.ctx, restart=4000)
    with pytest.raises(swr.SwrError) as e:
        solve()
    assert e.value.status == swr.SWR_ENOMEM
    swr.swr_set_schedule(pb.ctx, restart=8)
    assert np.array_equal(solve(), first)
    for k in range(8):
        swr.swr_set_schedule(pb.ctx, restart=100 + k % 2)
        solve()
    pb.close()
