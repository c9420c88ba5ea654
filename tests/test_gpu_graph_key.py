"""A captured solve is kept when a schedule parameter changes that no launch of a
static solve depends on, and captured anew for another pipeline chunk."""
import numpy as np
import pytest

from paper_1503_02564_amd import workloads as W
from tests.gpu_util import make_problem, say, to_dev, to_np

pytestmark = pytest.mark.gpu


def test_graph_survives_parameters_without_effect(dev):
    import torch
    from paper_1503_02564_amd import swr
    wl = W.small_case(J=[60, 90, 75, 128], nt=200, trans=W.S02, B=2, seed=41, a0=-12.0, b0=12.0)
    pb = make_problem(wl, pipeline=64)
    u0 = to_dev(wl.u0)
    uT = torch.zeros_like(u0)

    def solve():
        uT.fill_(float("nan"))
        st, info = swr.swr_solve(pb.ctx, u0, uT)
        assert st == swr.SWR_OK
        return to_np(uT), info

    def replayed(info):              # (a replay has no per-stage times)
        return info.t_factor_ms == 0 and info.t_total_ms > 0

    want, info = solve()
    assert not replayed(info)
    swr.swr_set_schedule(pb.ctx, graph=1)
    assert replayed(solve()[1])
    for kw in (dict(pair_from=3), dict(group=2), dict(help_max=0)):
        say("graph key", kw)
        swr.swr_set_schedule(pb.ctx, **kw)
        got, info = solve()
        assert replayed(info), kw
        assert np.array_equal(got, want)
    swr.swr_set_schedule(pb.ctx, pipeline=128)
    got, info = solve()
    assert not replayed(info) and np.array_equal(got, want)
    got, info = solve()
    assert replayed(info) and np.array_equal(got, want)
    pb.close()
