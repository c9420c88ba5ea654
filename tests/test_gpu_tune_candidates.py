"""The schedules that swr_tune times are different launches: helper-wave bounds
count only where a sweep has helper waves, V(t,x) that refactors in every step."""
import pytest

from paper_1503_02564_amd import workloads as W
from tests.gpu_util import make_problem, say, to_dev

pytestmark = pytest.mark.gpu

RESTARTS_CHECKS = 4 * 3        # restarts 20, 30, 60, 120; residual read-backs every 1, 4, 16 steps


@pytest.mark.parametrize("vkind,trans,limit,want", [
    (W.V_CUBIC, W.S02, None, 1),
    (W.V_TIME, W.S02, None, RESTARTS_CHECKS),
    (W.V_TIME, W.S02, 3 << 20, 2 * RESTARTS_CHECKS),       # no room for the records (3.2 MiB)
    (W.V_TIME, W.ROBIN, 3 << 20, RESTARTS_CHECKS),
])
def test_candidates(dev, monkeypatch, vkind, trans, limit, want):
    from paper_1503_02564_amd import swr
    wl = W.small_case(J=[40, 50, 60], nt=64, vkind=vkind, trans=trans, sigma=2 - 3j, B=1, seed=3)
    say("tune candidates", vkind, trans, limit)
    pb = make_problem(wl)
    if limit is not None:
        pb.close()
        monkeypatch.setenv("SWR_DEBUG_ALLOC_LIMIT", str(limit))
        pb = make_problem(wl)
    chosen = swr.swr_tune(pb.ctx, to_dev(wl.u0), budget_ms=60000.0)
    assert chosen.candidates == want
    pb.close()
