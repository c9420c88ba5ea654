"""The side outputs of a solve (end-node traces, snapshots, u(T), g) in every form
of the row and wide sweeps, against the oracle's monodomain steps: the snapshot
stride divides no block length (16, 32, 64), and the pipelined solve, whose
sweeps are cut into chunks, gives the staged solve's bits."""
import numpy as np
import pytest

from paper_1503_02564_amd import workloads as W
from tests.gpu_util import rel, say, to_dev, to_np

pytestmark = pytest.mark.gpu

STRIDE = 7
# (label, J, B, potential per problem, transmission, nt): with B as in the sweep tests
# of these forms, both task lists together are past the count from which a form is taken
CASES = [
    ("whole-wave", [1, 2, 40, 62, 63, 64, 127, 255, 300, 511], 2, False, W.S02, 150),
    ("one-row", [1, 2, 14, 15, 16, 30, 31, 32, 47, 62, 63, 64, 79, 95, 111, 126, 127], 101, False, W.S02, 300),
    ("one-row-robin", [3, 15, 16, 31, 46, 63, 64, 127], 251, False, W.ROBIN, 150),
    ("one-row-per-problem", [15, 40, 64, 100, 127], 257, True, W.S02, 150),
    ("two-rows", [128, 129, 159, 160, 191, 223, 224, 255, 100], 191, False, W.S02, 150),
    ("two-rows-lds", [256, 257, 287, 288, 320, 383, 384, 416, 447, 480, 511], 223, False, W.S02, 150),
    ("one-row-lds", [128, 143, 144, 159, 160, 175, 176, 191, 207, 208, 223], 571, False, W.S02, 150),
    ("wide", [512, 640, 1152, 100, 2304, 4608], 2, False, W.S02, 135),
    ("wide-robin", [520, 1151, 300, 2303], 1, False, W.ROBIN, 100),
]


def _solve(wl, per_problem, pipeline):
    import torch
    from paper_1503_02564_amd import swr
    o = swr.swr_default_opts()
    o.batch, o.tol, o.pipeline, o.snapshot_stride, o.v_per_problem = wl.B, 1e-13, pipeline, STRIDE, int(per_problem)
    V = None if wl.V is None else to_dev(np.asarray(wl.V, np.float64))
    pb = swr.Problem(wl.a0, wl.b0, tuple(int(j) for j in wl.J), wl.dt, wl.dt * wl.nt, wl.vkind, wl.trans,
                     wl.sigma, o, V)
    nan = complex(np.nan, np.nan)
    u0 = to_dev(wl.u0)
    uT = torch.full_like(u0, nan)
    g = torch.full((wl.B, pb.ns, wl.nt), nan, dtype=torch.complex128, device="cuda")
    tr = torch.full((wl.B, wl.N, 2, wl.nt + 1), nan, dtype=torch.complex128, device="cuda")
    sn = torch.full((wl.B, wl.nt // STRIDE + 1, wl.nx), nan, dtype=torch.complex128, device="cuda")
    st, info = swr.swr_solve(pb.ctx, u0, uT, g, tr, sn)
    assert st == swr.SWR_OK
    out = [to_np(x) for x in (uT, g, tr, sn)]
    pb.close()
    return out


def _check(wl, out, members, V=None):
    """The bar of the snapshot test: 1e-10 of the largest value."""
    import oracle as O
    uT, g, tr, sn = out
    off = np.concatenate([[0], np.cumsum(wl.J)])
    for x in out:
        assert np.isfinite(x).all()
    for b in members:
        kw = {} if V is None else dict(V=V[b])
        want, u_all, _ = O.mono(wl, wl.u0[b], want_u=True, **kw)
        top = np.max(np.abs(u_all))
        assert rel(uT[b], want) < 1e-10
        assert np.max(np.abs(sn[b] - u_all[::STRIDE])) < 1e-10 * top
        assert np.array_equal(sn[b][0], wl.u0[b])
        for k in range(wl.N):
            assert np.max(np.abs(tr[b, k, 0] - u_all[:, off[k]])) < 1e-10 * top, (b, k)
            assert np.max(np.abs(tr[b, k, 1] - u_all[:, off[k + 1]])) < 1e-10 * top, (b, k)


@pytest.mark.parametrize("label,J,B,per_problem,trans,nt", CASES, ids=[c[0] for c in CASES])
def test_outputs_of_every_form(dev, label, J, B, per_problem, trans, nt):
    wl = W.small_case(J=J, nt=nt, trans=trans, sigma=2 - 3j, B=B, seed=5, a0=-10.0, b0=10.0)
    Vs = None
    if per_problem:
        Vs = np.stack([(0.5 + b / B) * np.asarray(wl.V) for b in range(B)])
        wl = W.Workload("pp", wl.a0, wl.b0, wl.J, wl.dt, wl.nt, W.V_STATIC, Vs, trans, wl.sigma, wl.u0)
    say("row outputs", label, "staged")
    staged = _solve(wl, per_problem, 0)
    _check(wl, staged, sorted({0, 1 % B, B // 2, B - 1}), Vs)
    if max(J) < 512:
        say("row outputs", label, "pipelined")
        for x, y in zip(staged, _solve(wl, per_problem, 64)):
            assert np.array_equal(x, y)


@pytest.mark.parametrize("vkind,trans", [(W.V_TIME, W.S02), (W.V_TIME, W.ROBIN), (W.V_CUBIC, W.S02),
                                         (W.V_CUBIC, W.ROBIN)])
def test_outputs_of_moving_potentials(dev, vkind, trans):
    wl = W.small_case(J=[40, 63, 64, 100, 31, 200], nt=90, vkind=vkind, trans=trans, sigma=2 - 3j, B=1, seed=23,
                      a0=-12.0, b0=12.0)
    say("row outputs", vkind, trans)
    _check(wl, _solve(wl, False, -1), [0])
