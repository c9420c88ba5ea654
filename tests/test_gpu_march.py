"""Causal interface solve above 64 interfaces: the forms of the march (one
workgroup of 256, 512 or 1024 threads; windows with halos and blocks of 8 or 4
steps), at the edges of their interface counts and for every number of
doublings that a block-dominant system needs, against the monodomain oracle."""
import numpy as np
import pytest

from paper_1503_02564_amd import workloads as W
from tests.gpu_util import make_problem, rel, say, to_dev, to_np

pytestmark = pytest.mark.gpu

# (subdomains, cells of each, dt, doublings of the prefix sums, problems)
CASES = [
    (66, 16, 1e-5, 1, 1), (66, 4, 1e-2, 4, 3), (66, 4, 1e-1, 6, 1),
    (257, 16, 1e-5, 2, 3), (257, 1, 1e-3, 5, 1),
    (258, 4, 1e-5, 3, 1), (300, 1, 1e-3, 6, 2), (513, 4, 1e-5, 3, 9),
    (514, 16, 1e-5, 2, 1), (600, 4, 1e-5, 3, 3), (600, 2, 1e-5, 4, 1), (600, 2, 1e-4, 5, 1),
    (600, 1, 1e-3, 6, 1),
    (1025, 16, 1e-5, 3, 1), (1025, 2, 1e-4, 5, 2), (1025, 1, 1e-4, 6, 1),
]


def _doublings(cols, N):
    """Doublings until no product of the block elimination's multipliers over
    2^l interfaces exceeds 2^-60, from the lag-0 entries of the blocks."""
    x, ni = cols[:, :, 0], N - 1
    al, be = np.zeros(ni, complex), np.zeros(ni, complex)
    A = w = 0
    for j in range(ni):
        al[j] = x[j, 2] * w if j else 0
        A = x[j, 3] + (al[j] * A * x[j, 1] if j else 0)
        w = 1 / (1 - A * x[j + 1, 0])
        be[j] = w * x[j + 1, 1] if j + 1 < ni else 0
    lev = 0
    while max(abs(al).max(), abs(be).max()) > 2.0 ** -60:
        d = 1 << lev
        al[d:], al[:d] = al[d:] * al[:-d], 0
        be[:-d], be[-d:] = be[:-d] * be[d:], 0
        lev += 1
    return lev


@pytest.mark.parametrize("N,J,dt,doublings,B", CASES)
def test_solution_equals_the_monodomain(dev, N, J, dt, doublings, B):
    """u(T) of random initial data at 1e-10, the bar of the suite's solves
    against the monodomain, over ragged blocks."""
    import torch
    import oracle as O
    from paper_1503_02564_amd import swr
    nt = 21
    base = W.small_case(J=[J] * N, nt=nt, trans=W.S02, B=B, seed=5, a0=-10.0, b0=10.0)
    rng = np.random.default_rng(N)
    u0 = rng.standard_normal((B, base.nx)) + 1j * rng.standard_normal((B, base.nx))
    u0[:, 0] = u0[:, -1] = 0
    wl = W.Workload("m", base.a0, base.b0, base.J, dt, nt, W.V_STATIC, base.V, base.trans, base.sigma, u0)
    pb = make_problem(wl)
    cols = torch.zeros((1, N, 4, nt), dtype=torch.complex128, device=dev)
    d = torch.zeros((B, 2 * N - 2, nt), dtype=torch.complex128, device=dev)
    swr.swr_build_interface(pb.ctx, to_dev(u0), cols, d)
    assert _doublings(to_np(cols)[0], N) == doublings
    say("march", N, J, dt, "B", B)
    uT = torch.zeros((B, wl.nx), dtype=torch.complex128, device=dev)
    st, info = swr.swr_solve(pb.ctx, to_dev(u0), uT)
    assert st == swr.SWR_OK
    for b in range(B):
        e = rel(to_np(uT)[b], O.mono(wl, u0[b]))
        say("march", N, J, dt, b, e, info.residual)
        assert e < 1e-10
    pb.close()
