"""A call that is refused memory half-way (SWR_ENOMEM) leaves no half-made
workspace behind: with room again, the same context gives the bits of one that was
never refused.  swr_tune relies on it, which goes on after a refusal."""
import numpy as np
import pytest

from paper_1503_02564_amd import workloads as W
from tests.gpu_util import say, to_dev, to_np

pytestmark = pytest.mark.gpu

S02 = dict(J=[40] * 6, nt=300, trans=W.S02, B=64)
CASES = {
    # (problem, solver, pipeline, call)
    "pipelined": (S02, "causal", 64, "solve"),
    "march": (dict(J=[6] * 70, nt=300, trans=W.S02, B=2), "causal", 0, "solve"),
    "dense": (dict(J=[2] * 60, nt=64, trans=W.S02, B=2, a0=-0.6, b0=0.6), "causal", 0, "solve"),
    "bicgstab": (S02, "bicgstab", 0, "solve"),
    "gmres": (S02, "gmres", 0, "solve"),
    "gradient": (S02, "causal", 64, "grad"),
    "gradient-robin": (dict(S02, trans=W.ROBIN), "causal", 0, "grad"),
}


class _Call:
    def __init__(self, wl, solver, pipeline, call):
        import torch
        from paper_1503_02564_amd import swr
        o = swr.swr_default_opts()
        o.batch, o.pipeline = wl.B, pipeline
        o.solver = dict(causal=swr.SWR_SOLVER_CAUSAL, bicgstab=swr.SWR_SOLVER_BICGSTAB,
                        gmres=swr.SWR_SOLVER_GMRES)[solver]
        self.pb = swr.Problem(wl.a0, wl.b0, tuple(int(j) for j in wl.J), wl.dt, wl.dt * wl.nt, wl.vkind,
                              wl.trans, wl.sigma, o, to_dev(np.asarray(wl.V, np.float64)))
        self.u0, self.call = to_dev(wl.u0), call
        self.out = [torch.zeros_like(self.u0)]
        if call == "grad":
            self.out.insert(0, torch.zeros(wl.u0.shape, dtype=torch.float64, device="cuda"))

    def run(self):
        """The call's outputs, or None where it met SWR_ENOMEM."""
        from paper_1503_02564_amd import swr
        try:
            if self.call == "grad":
                st, _ = swr.swr_grad(self.pb.ctx, self.u0, self.u0, *self.out)
            else:
                st, _ = swr.swr_solve(self.pb.ctx, self.u0, *self.out)
        except swr.SwrError as e:
            assert e.status == swr.SWR_ENOMEM
            return None
        assert st == swr.SWR_OK
        return [to_np(x) for x in self.out]


@pytest.mark.parametrize("name", list(CASES))
def test_a_refused_call_can_be_repeated(dev, monkeypatch, name):
    prob, solver, pipeline, call = CASES[name]
    wl = W.small_case(**dict(dict(seed=13, a0=-10.0, b0=10.0, sigma=2 - 3j), **prob))
    say("refused", name, "reference")
    c = _Call(wl, solver, pipeline, call)
    want = c.run()
    c.pb.close()
    # the least limit with which the call goes through (setup has no limit)
    lo, hi = 0, 1 << 30
    while hi - lo > 1024:
        mid = (lo + hi) // 2
        c = _Call(wl, solver, pipeline, call)
        monkeypatch.setenv("SWR_DEBUG_ALLOC_LIMIT", str(mid))
        lo, hi = (lo, mid) if c.run() is not None else (mid, hi)
        monkeypatch.delenv("SWR_DEBUG_ALLOC_LIMIT")
        c.pb.close()
    refused = 0
    for less in [0] + [1 << k for k in range(10, 26)] + [3 << k for k in range(9, 25)]:
        if less > lo:
            continue
        c = _Call(wl, solver, pipeline, call)
        monkeypatch.setenv("SWR_DEBUG_ALLOC_LIMIT", str(lo - less))
        assert c.run() is None
        monkeypatch.delenv("SWR_DEBUG_ALLOC_LIMIT")
        refused += 1
        say("refused", name, less, "bytes below", lo)
        for x, y in zip(want, c.run()):
            assert np.array_equal(x, y), (name, less)
        c.pb.close()
    assert refused > 8
