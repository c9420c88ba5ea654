"""Products with the interface operator (block-Toeplitz, on the matrix cores)
over step counts at the edges of its tiles of 16 and 256 outputs and of its
stages of 16 lag blocks, against convolutions, and the causal solve whose history
comes in one or several partials."""
import numpy as np
import pytest

from paper_1503_02564_amd import workloads as W
from tests.gpu_util import make_problem, rel, say, to_dev, to_np

pytestmark = pytest.mark.gpu


def _apply(cols, g):
    """y = g - L g by FFT convolution of the blocks' first columns."""
    from scipy.signal import fftconvolve
    B, ns, nt = g.shape
    N = ns // 2 + 1
    y = g.copy()
    for b in range(B):
        c = cols[b if len(cols) > 1 else 0]
        for k in range(N):
            for p in range(4):
                src = 2 * k - 1 if p % 2 == 0 else 2 * k
                dst = 2 * k - 2 if p < 2 else 2 * k + 1
                if 0 <= src < ns and 0 <= dst < ns and (k > 0 or src == 0) and (k < N - 1 or src == ns - 1):
                    y[b, dst] -= fftconvolve(c[k, p], g[b, src])[:nt]
    return y


@pytest.mark.parametrize("nt", [1, 15, 16, 17, 127, 129, 255, 256, 257, 272, 500, 513, 800])
@pytest.mark.parametrize("B,per_problem", [(1, False), (3, True), (9, False)])
def test_product_equals_the_convolution(dev, nt, B, per_problem):
    """1e-12 of the largest entry: 2 nt terms of relative rounding 1e-16 each,
    and the same again for the transform."""
    import torch
    from paper_1503_02564_amd import swr
    J = [9, 30, 17, 12]
    wl = W.small_case(J=J, nt=nt, trans=W.S02, B=B, seed=3)
    wl = W.Workload("c", wl.a0, wl.b0, wl.J, 1e-2, nt, W.V_STATIC, wl.V, wl.trans, wl.sigma, wl.u0)
    if per_problem:
        Vs = np.stack([(0.5 + b) * np.asarray(wl.V) for b in range(B)])
        wl = W.Workload("c", wl.a0, wl.b0, wl.J, 1e-2, nt, W.V_STATIC, Vs, wl.trans, wl.sigma, wl.u0)
    N, ns = len(J), 2 * len(J) - 2
    say("product", nt, B, per_problem)
    pb = make_problem(wl, v_per_problem=per_problem)
    cols = torch.zeros((B if per_problem else 1, N, 4, nt), dtype=torch.complex128, device=dev)
    d = torch.zeros((B, ns, nt), dtype=torch.complex128, device=dev)
    swr.swr_build_interface(pb.ctx, to_dev(wl.u0), cols, d)
    rng = np.random.default_rng(nt)
    g = rng.standard_normal((B, ns, nt)) + 1j * rng.standard_normal((B, ns, nt))
    y = torch.zeros_like(d)
    swr.swr_interface_matvec(pb.ctx, to_dev(g), y)
    ref = _apply(to_np(cols), g)
    assert np.abs(to_np(y) - ref).max() < 1e-12 * np.abs(ref).max()
    pb.close()


@pytest.mark.parametrize("N,B,per_problem,nt", [(4, 1, False, 1300), (40, 2, True, 1100), (40, 8, False, 800),
                                               (120, 5, True, 700), (40, 26, True, 300),
                                               (100, 31, False, 300), (64, 48, False, 300)])
def test_causal_solution_meets_the_convolution(dev, N, B, per_problem, nt):
    """(I - L) g = d over several super-blocks: certified residual, u(T) against the
    monodomain oracle at the bar of the suite's solves, and the staged solve equal
    to the pipelined one."""
    import torch
    from paper_1503_02564_amd import swr
    wl = W.small_case(J=[20] * N, nt=nt, trans=W.S02, B=B, seed=3, a0=-10.0, b0=10.0)
    if per_problem:
        Vs = np.stack([(0.5 + b) * np.asarray(wl.V) for b in range(B)])
        wl = W.Workload("c", wl.a0, wl.b0, wl.J, wl.dt, nt, W.V_STATIC, Vs, wl.trans, wl.sigma, wl.u0)
    say("causal", N, B, per_problem, nt)
    out = []
    for ch in (0, 256):
        pb = make_problem(wl, v_per_problem=per_problem, pipeline=ch)
        uT = torch.zeros((B, wl.nx), dtype=torch.complex128, device=dev)
        st, info = swr.swr_solve(pb.ctx, to_dev(wl.u0), uT)
        assert st == swr.SWR_OK and info.residual < 1e-12
        out.append(to_np(uT))
        pb.close()
    assert np.array_equal(out[0], out[1])
    import oracle as O
    for b in range(B):
        V = wl.V[b] if per_problem else wl.V
        one = W.Workload("one", wl.a0, wl.b0, wl.J, wl.dt, nt, W.V_STATIC, V, wl.trans, wl.sigma, wl.u0[b:b + 1])
        assert rel(out[0][b], O.mono(one, one.u0[0])) < 1e-10
