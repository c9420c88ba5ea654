"""Row form of the static sweep: contexts with enough tasks run a subdomain on
one or two rows of 16 lanes (two to four tasks per wave), interior coefficients
in registers or in LDS.  One sweep at the edges of every form's widths against
the oracle's sweep, element by element, and independence of the tasks of a wave."""
import numpy as np
import pytest

from paper_1503_02564_amd import workloads as W
from tests.gpu_util import make_problem, rel, say, to_dev, to_np

pytestmark = pytest.mark.gpu

# (label, J, B, potential per problem, transmission): node counts J + 1 at the
# first and last of a width, fewer nodes than lanes, every width up to the
# form's widest; batches that leave waves partly filled
CASES = [
    # 2560 tasks: one row, registers (up to 128 nodes)
    ("one-row", [1, 2, 14, 15, 16, 30, 31, 32, 47, 62, 63, 64, 79, 95, 111, 126, 127], 101, False, W.S02),
    ("one-row-robin", [3, 15, 16, 31, 46, 63, 64, 127], 251, False, W.ROBIN),
    ("one-row-per-problem", [15, 40, 64, 100, 127], 257, True, W.S02),
    # 3072 / 4608 tasks: two rows, registers (129 to 256 nodes) and LDS (above)
    ("two-rows", [128, 129, 159, 160, 191, 223, 224, 255, 100], 191, False, W.S02),
    ("two-rows-lds", [256, 257, 287, 288, 320, 383, 384, 416, 447, 480, 511], 223, False, W.S02),
    ("two-rows-robin", [255, 300, 128, 511], 643, False, W.ROBIN),
    # 12288 tasks: one row, LDS (129 to 224 nodes)
    ("one-row-lds", [128, 143, 144, 159, 160, 175, 176, 191, 207, 208, 223], 571, False, W.S02),
]


@pytest.mark.parametrize("label,J,B,per_problem,trans", CASES, ids=[c[0] for c in CASES])
def test_one_sweep_equals_the_oracle(dev, label, J, B, per_problem, trans):
    import torch
    import oracle as O
    from paper_1503_02564_amd import swr
    nt = 300          # a ragged last block of every block length; past one far-history super-chunk
    wl = W.small_case(J=J, nt=nt, trans=trans, B=B, seed=5, a0=-10.0, b0=10.0)
    Vs = None
    if per_problem:
        Vs = np.stack([(0.5 + b / B) * np.asarray(wl.V) for b in range(B)])
        wl = W.Workload("pp", wl.a0, wl.b0, wl.J, wl.dt, wl.nt, W.V_STATIC, Vs, trans, wl.sigma, wl.u0)
    rng = np.random.default_rng(9)
    ns = 2 * len(J) - 2
    g = rng.standard_normal((B, ns, nt)) + 1j * rng.standard_normal((B, ns, nt))
    say("rows", label, "tasks", 2 * B * len(J))
    pb = make_problem(wl, v_per_problem=per_problem)
    gd = to_dev(g)
    out = torch.zeros_like(gd)
    uT = torch.zeros((B, wl.nx), dtype=torch.complex128, device=dev)
    swr.swr_apply_R(pb.ctx, to_dev(wl.u0), gd, out, uT)
    got = to_np(out)
    for b in (0, 1, 2, 3, B // 2, B - 2, B - 1):
        one = W.Workload("one", wl.a0, wl.b0, wl.J, wl.dt, wl.nt, W.V_STATIC,
                         wl.V if Vs is None else Vs[b], trans, wl.sigma, wl.u0[b:b + 1])
        uref, ref = O.local_solution(one, one.u0[0], g[b])
        assert rel(got[b], ref) < 1e-12, (label, b)
        assert rel(to_np(uT)[b], uref) < 1e-12, (label, b)
    # a problem with a non-finite flux leaves the other tasks of its waves, and
    # its own steps before it, as they were
    gd[1, :, 40] = float("nan")
    out2 = torch.zeros_like(gd)
    swr.swr_apply_R(pb.ctx, to_dev(wl.u0), gd, out2, None)
    keep = [b for b in range(B) if b != 1]
    got2 = to_np(out2)
    assert np.array_equal(got2[keep], got[keep])
    assert np.array_equal(got2[1][:, :40], got[1][:, :40])
    assert not np.isfinite(got2[1][:, 40]).any()
    pb.close()


# node counts J + 1 at the first and last width of every workgroup size of the
# wide form (2, 4, 8 waves; 5 to 9, for 8 waves to 12 nodes per lane), with and
# without copied slots, the first size past it, and a short neighbour
WIDE = [
    ("two-waves", [512, 639, 640, 700, 1023, 1151, 99], W.S02),
    ("two-waves-robin", [520, 1151, 300], W.ROBIN),
    ("four-waves", [1152, 1279, 1280, 1900, 2303], W.S02),
    ("eight-waves", [2304, 2559, 4200, 4607], W.S02),
    ("eight-waves-long", [4608, 5119, 6143, 6144], W.S02),
]


@pytest.mark.parametrize("label,J,trans", WIDE, ids=[c[0] for c in WIDE])
def test_one_wide_sweep_equals_the_oracle(dev, label, J, trans):
    """Long subdomains on a workgroup of 2, 4 or 8 waves: one sweep against the
    oracle's at 1e-11, the bar of the streaming form's test (chunks of many
    nodes), and steps before a non-finite flux unchanged."""
    import torch
    import oracle as O
    from paper_1503_02564_amd import swr
    nt, B = 135, 2
    wl = W.small_case(J=J, nt=nt, trans=trans, sigma=2 - 3j, B=B, seed=5, a0=-12.0, b0=12.0)
    rng = np.random.default_rng(3)
    ns = 2 * len(J) - 2
    g = 0.3 * (rng.standard_normal((B, ns, nt)) + 1j * rng.standard_normal((B, ns, nt)))
    say("wide", label)
    pb = make_problem(wl)
    gd = to_dev(g)
    out = torch.zeros_like(gd)
    uT = torch.zeros((B, wl.nx), dtype=torch.complex128, device=dev)
    swr.swr_apply_R(pb.ctx, to_dev(wl.u0), gd, out, uT)
    got = to_np(out)
    for b in range(B):
        uref, ref = O.local_solution(wl, wl.u0[b], g[b])
        eg, eu = rel(got[b], ref), rel(to_np(uT)[b], uref)
        say("wide", label, b, "g", eg, "uT", eu)
        assert eg < 1e-11 and eu < 1e-11
    gd[1, :, 70] = float("nan")
    out2 = torch.zeros_like(gd)
    swr.swr_apply_R(pb.ctx, to_dev(wl.u0), gd, out2, None)
    got2 = to_np(out2)
    assert np.array_equal(got2[0], got[0]) and np.array_equal(got2[1][:, :70], got[1][:, :70])
    pb.close()


# the same forms in the adjoint sweep (node counts J + 1 at the edges of their
# widths); few tasks: one task on the whole wave
ADJ = [
    ("whole-wave", [1, 2, 62, 63, 64, 127, 255, 300, 511], 2, True, W.S02),
    ("one-row", [1, 2, 14, 15, 16, 31, 32, 63, 64, 79, 100, 126, 127], 127, False, W.S02),
    ("one-row-robin-per-problem", [3, 15, 16, 63, 64, 127], 430, True, W.ROBIN),
    ("two-rows", [128, 129, 160, 191, 224, 255, 100], 240, False, W.S02),
    ("two-rows-lds", [256, 288, 320, 384, 447, 480, 511], 350, False, W.S02),
    ("one-row-lds", [128, 143, 144, 160, 176, 191, 208, 223], 790, False, W.S02),
]


@pytest.mark.parametrize("label,J,B,per_problem,trans", ADJ, ids=[c[0] for c in ADJ])
def test_adjoint_of_every_form(dev, label, J, B, per_problem, trans):
    """Gradients against the oracle's monodomain adjoint at the bar of the
    suite's adjoint tests, over several checkpoint segments with a ragged last
    one, for an arbitrary upstream gradient."""
    import torch
    import oracle as O
    from paper_1503_02564_amd import swr
    nt = 70 if trans == W.ROBIN else 150
    wl = W.small_case(J=J, nt=nt, trans=trans, sigma=2 - 3j, B=B, seed=11, a0=-10.0, b0=10.0)
    Vs = None
    if per_problem:
        Vs = np.stack([(0.5 + b / B) * np.asarray(wl.V) for b in range(B)])
        wl = W.Workload("pp", wl.a0, wl.b0, wl.J, wl.dt, wl.nt, W.V_STATIC, Vs, trans, wl.sigma, wl.u0)
    rng = np.random.default_rng(4)
    gbar = rng.standard_normal((B, wl.nx)) + 1j * rng.standard_normal((B, wl.nx))
    say("adjoint rows", label, "tasks", B * len(J))
    pb = make_problem(wl, v_per_problem=per_problem)
    dV = torch.zeros((B, wl.nx), dtype=torch.float64, device=dev)
    du0 = torch.zeros((B, wl.nx), dtype=torch.complex128, device=dev)
    st, info = swr.swr_grad(pb.ctx, to_dev(wl.u0), to_dev(gbar), dV, du0)
    assert st == swr.SWR_OK
    for b in (0, 1, B // 2, B - 1):
        V = wl.V if Vs is None else Vs[b]
        one = W.Workload("one", wl.a0, wl.b0, wl.J, wl.dt, wl.nt, W.V_STATIC, V, trans, wl.sigma, wl.u0[b:b + 1])
        dV_ref, du0_ref = O.adjoint_mono(one, one.u0[0], gbar[b])
        ev, eu = rel(to_np(dV)[b], dV_ref), rel(to_np(du0)[b], du0_ref)
        say("adjoint rows", label, b, "dV", ev, "du0", eu)
        assert ev < 1e-10 and eu < 1e-10
    pb.close()


WIDTHS = [1, 2, 40, 62, 63, 64, 100, 127, 128, 190, 255, 256, 320, 383, 384, 447, 448, 511]


@pytest.mark.parametrize("vk,trans,J,nt", [
    (W.V_TIME, W.S02, WIDTHS, 135), (W.V_TIME, W.ROBIN, WIDTHS, 64), (W.V_TIME, W.S02, [5, 70, 7], 2100),
    (W.V_CUBIC, W.S02, WIDTHS, 135), (W.V_CUBIC, W.ROBIN, WIDTHS, 65), (W.V_CUBIC, W.S02, [5, 70, 7], 2100),
    (W.V_TIME, W.S02, [9, 8], 1), (W.V_CUBIC, W.S02, [9, 8], 1),
])
def test_sweeps_of_moving_potentials(dev, vk, trans, J, nt):
    """V(t,x) with its records read step by step and |u|^2 with its inner
    iteration, in every width and past the window where the history is split:
    one sweep against the oracle's, 1e-11 (|u|^2: 1e-10, the inner iteration
    stops at 1e-12 of the largest value in either)."""
    import torch
    import oracle as O
    from paper_1503_02564_amd import swr
    wl = W.small_case(J=J, nt=nt, vkind=vk, trans=trans, sigma=2 - 3j, B=1, seed=5, a0=-10.0, b0=10.0)
    rng = np.random.default_rng(2)
    ns = 2 * len(J) - 2
    g = 0.3 * (rng.standard_normal((1, ns, nt)) + 1j * rng.standard_normal((1, ns, nt)))
    say("moving", vk, trans, len(J), nt)
    pb = make_problem(wl)
    out = torch.zeros((1, ns, nt), dtype=torch.complex128, device=dev)
    uT = torch.zeros((1, wl.nx), dtype=torch.complex128, device=dev)
    swr.swr_apply_R(pb.ctx, to_dev(wl.u0), to_dev(g), out, uT)
    uref, ref = O.local_solution(wl, wl.u0[0], g[0])
    bar = 1e-10 if vk == W.V_CUBIC else 1e-11
    assert rel(to_np(out)[0], ref) < bar and rel(to_np(uT)[0], uref) < bar
    pb.close()


def test_records_in_pieces_equal_refactoring(dev):
    """V(t,x) whose records do not all fit at once (240 subdomains of 500 cells:
    384 steps) against two problems with the same data, above the task count of
    the records: both sweeps carry one rounding chain of 390 steps, 1e-11."""
    import torch
    from paper_1503_02564_amd import swr
    N, nt = 240, 390
    wl = W.small_case(J=[500] * N, nt=nt, vkind=W.V_TIME, B=1, seed=5, a0=-100.0, b0=100.0)
    rng = np.random.default_rng(2)
    g = 0.3 * (rng.standard_normal((1, 2 * N - 2, nt)) + 1j * rng.standard_normal((1, 2 * N - 2, nt)))
    res = []
    for B in (1, 2):
        w2 = W.Workload("p", wl.a0, wl.b0, wl.J, wl.dt, nt, wl.vkind, wl.V, wl.trans, wl.sigma,
                        np.repeat(wl.u0, B, axis=0))
        pb = make_problem(w2)
        gd = to_dev(np.repeat(g, B, axis=0))
        out = torch.zeros_like(gd)
        uT = torch.zeros((B, wl.nx), dtype=torch.complex128, device=dev)
        swr.swr_apply_R(pb.ctx, to_dev(w2.u0), gd, out, uT)
        res.append((to_np(out)[0], to_np(uT)[0]))
        pb.close()
    assert rel(res[0][0], res[1][0]) < 1e-11 and rel(res[0][1], res[1][1]) < 1e-11
