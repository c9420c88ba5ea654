"""Factors at dt / h^2 = 21: on this mesh the row sums of the subdomain matrices
are 60 times smaller than their couplings, and a pivot formed by subtraction
loses them by the same error in every step.  A 64-bit Thomas sweep over the whole
domain does so (5.8e-12 of u after 2000 steps, against extended precision); the
row form and the wide form carry the sums and stay a factor of ten below it."""
import numpy as np
import pytest

from paper_1503_02564_amd import workloads as W
from tests.gpu_util import make_problem, rel, say, to_dev, to_np

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def reference():
    import oracle as O
    wl = W.adjoint_batch()
    ld = O.mono_ld(wl, wl.u0[0], V=wl.V[0])
    return wl, ld, rel(O.mono(wl, wl.u0[0], V=wl.V[0]), ld)


@pytest.mark.parametrize("label,J,B", [("one-row", [64] * 256, 16), ("whole-wave", [64] * 256, 1),
                                       ("whole-wave-256", [256] * 64, 1), ("wide", [4096] * 4, 1)])
def test_factors_keep_the_row_sums(dev, reference, label, J, B):
    import torch
    from paper_1503_02564_amd import swr
    wl, ld, thomas = reference
    assert thomas > 2e-12                     # the mesh shows the loss
    one = W.Workload(label, wl.a0, wl.b0, np.asarray(J, np.int32), wl.dt, wl.nt, W.V_STATIC,
                     wl.V if B > 1 else wl.V[0], wl.trans, wl.sigma, wl.u0[:B])
    pb = make_problem(one, v_per_problem=B > 1)
    uT = torch.zeros((B, wl.nx), dtype=torch.complex128, device=dev)
    st, _ = swr.swr_solve(pb.ctx, to_dev(one.u0), uT)
    assert st == swr.SWR_OK
    err = rel(to_np(uT)[0], ld)
    say("row sums", label, "error", err, "64-bit Thomas", thomas)
    assert err < thomas / 10
    pb.close()
