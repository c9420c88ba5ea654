// swr_sweep_rows.hip -- launches the row form of the static sweep
// (swr_sweep_rows_kernel.h), instantiated one kind per file.
#include "swr_sweep_rows_kernel.h"

namespace swr {

hipError_t launch_sweep_rows4(const SweepArgs& a, int trans, int nitems, size_t lds, hipStream_t st);
hipError_t launch_sweep_rows1_reg(const SweepArgs& a, int trans, int nitems, size_t lds, hipStream_t st);
hipError_t launch_sweep_rows1_lds(const SweepArgs& a, int trans, int nitems, size_t lds, hipStream_t st);
hipError_t launch_sweep_rows2_reg(const SweepArgs& a, int trans, int nitems, size_t lds, hipStream_t st);
hipError_t launch_sweep_rows2_lds(const SweepArgs& a, int trans, int nitems, size_t lds, hipStream_t st);

hipError_t launch_sweep_rows_cubic(const SweepArgs& a, int trans, int nitems, size_t lds, hipStream_t st);
hipError_t launch_sweep_rows_time(const SweepArgs& a, int trans, int nitems, size_t lds, hipStream_t st);

hipError_t launch_sweep_rows(const SweepArgs& a, int kind, int trans, int vk, int nitems, int pmax,
                             hipStream_t st) {
    if (nitems == 0) return hipSuccess;
    if (kind < 0 || kind >= kRowsKinds || !a.items || (!a.fac && vk != VK_TIME) || (trans != TR_S02 && trans != TR_ROBIN))
        return hipErrorInvalidValue;
    const RowsKind& k = kRowsKind[kind];
    if (pmax < 1 || pmax > k.pmax) return hipErrorInvalidValue;
    if (trans == TR_S02 && (!a.hist || !a.beta)) return hipErrorInvalidValue;
    if ((a.n_begin > 0 || a.n_end < a.nt) && !a.state) return hipErrorInvalidValue;
    const size_t lds = rows_lds_bytes(k, pmax);
    // V(t,x), |u|^2: one task per wave; V(t,x) with two records in LDS
    if (vk != VK_STATIC && kind != 0) return hipErrorInvalidValue;
    if (vk == VK_CUBIC) return launch_sweep_rows_cubic(a, trans, nitems, lds, st);
    if (vk == VK_TIME)
        return launch_sweep_rows_time(a, trans, nitems, lds + sizeof(cd) * 2 * rows_fields(pmax, 4) * kWave, st);
    switch (kind) {
        case 0: return launch_sweep_rows4(a, trans, nitems, lds, st);
        case 1: return launch_sweep_rows1_reg(a, trans, nitems, lds, st);
        case 2: return launch_sweep_rows1_lds(a, trans, nitems, lds, st);
        case 3: return launch_sweep_rows2_reg(a, trans, nitems, lds, st);
        case 4: return launch_sweep_rows2_lds(a, trans, nitems, lds, st);
    }
    return hipErrorInvalidValue;
}

}  // namespace swr
