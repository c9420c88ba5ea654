// swr_adjoint.hip -- launches the adjoint sweep (swr_adjoint_kernel.h),
// instantiated one kind of the row form per file, and joins the gradients of
// the subdomains at their shared nodes.
#include "swr_rows.h"
#include "swr_sweep_rows_kernel.h"

namespace swr {

hipError_t launch_adjoint_rows4(const AdjArgs& a, int trans, int nitems, size_t lds, hipStream_t st);
hipError_t launch_adjoint_rows1_reg(const AdjArgs& a, int trans, int nitems, size_t lds, hipStream_t st);
hipError_t launch_adjoint_rows1_lds(const AdjArgs& a, int trans, int nitems, size_t lds, hipStream_t st);
hipError_t launch_adjoint_rows2_reg(const AdjArgs& a, int trans, int nitems, size_t lds, hipStream_t st);
hipError_t launch_adjoint_rows2_lds(const AdjArgs& a, int trans, int nitems, size_t lds, hipStream_t st);

// dJ/dV and dJ/du0 at nodes shared by two subdomains: the two local parts
// add (element sums of dJ/dV; pieces of the assembled dual vector P_0).
__global__ void finalize_grad_kernel(int N, int nx, int B, const int* off, const double* gends,
                                     const cd* wends, double* dV, cd* du0) {
    const int idx = blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= B * (N + 1)) return;
    const int b = idx / (N + 1), j = idx % (N + 1);
    const double* ge = gends + (size_t)b * N * 2;
    const cd* we = wends + (size_t)b * N * 2;
    double* v = dV + (size_t)b * nx;
    cd* u = du0 + (size_t)b * nx;
    if (j == 0) { v[0] = ge[0]; u[0] = conjc(we[0]); }
    else if (j == N) { v[nx - 1] = ge[(N - 1) * 2 + 1]; u[nx - 1] = conjc(we[(N - 1) * 2 + 1]); }
    else {
        v[off[j]] = ge[(j - 1) * 2 + 1] + ge[j * 2 + 0];
        u[off[j]] = conjc(we[(j - 1) * 2 + 1] + we[j * 2 + 0]);
    }
}

// the workgroups are those of the forward sweep
hipError_t launch_adjoint(const AdjArgs& a, int kind, int trans, int nitems, int pmax, hipStream_t st) {
    if (nitems == 0) return hipSuccess;
    if (kind < 0 || kind >= kRowsKinds || !a.items || !a.fac || (trans != TR_S02 && trans != TR_ROBIN))
        return hipErrorInvalidValue;
    const RowsKind& k = kRowsKind[kind];
    if (pmax < 1 || pmax > k.pmax) return hipErrorInvalidValue;
    if (trans == TR_S02 && (!a.hist || !a.beta)) return hipErrorInvalidValue;
    if ((a.m_begin > 0 || a.m_end < a.nt) && !a.state) return hipErrorInvalidValue;
    if (a.grad && (!a.ckpt || !a.bsum || !a.seg)) return hipErrorInvalidValue;
    const size_t lds = rows_lds_bytes(k, pmax);
    switch (kind) {
        case 0: return launch_adjoint_rows4(a, trans, nitems, lds, st);
        case 1: return launch_adjoint_rows1_reg(a, trans, nitems, lds, st);
        case 2: return launch_adjoint_rows1_lds(a, trans, nitems, lds, st);
        case 3: return launch_adjoint_rows2_reg(a, trans, nitems, lds, st);
        case 4: return launch_adjoint_rows2_lds(a, trans, nitems, lds, st);
    }
    return hipErrorInvalidValue;
}

hipError_t launch_finalize_grad(int N, int nx, int B, const int* off, const double* gends,
                                const cd* wends, double* dV, cd* du0, hipStream_t st) {
    const int tot = B * (N + 1);
    finalize_grad_kernel<<<(tot + 255) / 256, 256, 0, st>>>(N, nx, B, off, gends, wends, dV, du0);
    return hipGetLastError();
}

}  // namespace swr
