"""V(t,x) contexts without room for their factor records (SWR_DEBUG_ALLOC_LIMIT
makes the runtime refuse memory): they set up and solve as before, refactoring in
every step, and no refused allocation surfaces in a later call."""
import numpy as np
import pytest

from paper_1503_02564_amd import workloads as W
from tests.gpu_util import make_problem, rel, say, to_dev, to_np

pytestmark = pytest.mark.gpu

MIB = 1 << 20


def _case(nt, J=(200,) * 6):
    return W.small_case(J=list(J), nt=nt, vkind=W.V_TIME, B=1, seed=5, a0=-10.0, b0=10.0)


def _sweep(wl, limit, monkeypatch, solve=False, **kw):
    import torch
    from paper_1503_02564_amd import swr
    if limit is None:
        monkeypatch.delenv("SWR_DEBUG_ALLOC_LIMIT", raising=False)
    else:
        monkeypatch.setenv("SWR_DEBUG_ALLOC_LIMIT", str(int(limit)))
    ns, nt = 2 * wl.N - 2, wl.nt
    rng = np.random.default_rng(2)
    gd = to_dev(0.3 * (rng.standard_normal((1, ns, nt)) + 1j * rng.standard_normal((1, ns, nt))))
    pb = make_problem(wl, **kw)
    u0 = to_dev(wl.u0)
    out, uT, uS = torch.zeros_like(gd), torch.zeros_like(u0), torch.zeros_like(u0)
    swr.swr_apply_R(pb.ctx, u0, gd, out, uT)
    res = [to_np(out)[0], to_np(uT)[0]]
    if solve:
        for _ in range(2):
            st, info = swr.swr_solve(pb.ctx, u0, uS)
            assert st == swr.SWR_OK
        res.append(to_np(uS)[0])
    pb.close()
    return res


@pytest.mark.parametrize("nt", [300, 2100])       # 2100: far history in super-chunks as well
def test_refactors_without_room_for_records(dev, monkeypatch, nt):
    """Records of 300 steps take 53 MiB here, the rest of the context less than
    12 MiB (2100 steps: 372 and 64).  Both sweeps carry one rounding chain a
    step: 1e-11, the bar of the sweeps of moving potentials."""
    import oracle as O
    wl = _case(nt)
    say("no records", nt)
    got = _sweep(wl, (24 if nt == 300 else 128) * MIB, monkeypatch)
    ref = _sweep(wl, None, monkeypatch)
    for x, y in zip(got, ref):
        assert rel(x, y) < 1e-11
    rng = np.random.default_rng(2)
    ns = 2 * wl.N - 2
    g = 0.3 * (rng.standard_normal((1, ns, nt)) + 1j * rng.standard_normal((1, ns, nt)))
    uref, gref = O.local_solution(wl, wl.u0[0], g[0])
    assert rel(got[0], gref) < 1e-11 and rel(got[1], uref) < 1e-11


def test_records_make_room_for_a_later_buffer(dev, monkeypatch):
    """A GMRES basis of 2001 vectors (153 MiB with its Hessenberg matrix) that fits
    only without the records."""
    import oracle as O
    wl = _case(300)
    say("records given back")
    got = _sweep(wl, 200 * MIB, monkeypatch, solve=True, restart=2000)
    assert rel(got[2], O.mono(wl, wl.u0[0])) < 1e-9


def test_refused_setup_leaves_nothing_behind(dev, monkeypatch):
    """SWR_ENOMEM without room for the mandatory buffers; the next setup and
    sweep on the same thread see no pending error."""
    from paper_1503_02564_amd import swr
    wl = _case(300)
    monkeypatch.setenv("SWR_DEBUG_ALLOC_LIMIT", str(MIB))
    with pytest.raises(swr.SwrError) as e:
        make_problem(wl)
    assert e.value.status == swr.SWR_ENOMEM
    say("after a refused setup")
    _sweep(wl, None, monkeypatch)
