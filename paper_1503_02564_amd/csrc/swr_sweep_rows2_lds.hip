// swr_sweep_rows2_lds.hip -- instantiates the row form of the static sweep: two tasks per wave, widths 9 to 16 from LDS.
#include "swr_sweep_rows_kernel.h"

namespace swr {

hipError_t launch_sweep_rows2_lds(const SweepArgs& a, int trans, int nitems, size_t lds, hipStream_t st) {
    if (trans == TR_S02) sweep_rows_kernel<2, 9, 16, 9, 2, 2, TR_S02><<<nitems, kRowsKind[4].waves * kWave, lds, st>>>(a);
    else sweep_rows_kernel<2, 9, 16, 9, 2, 2, TR_ROBIN><<<nitems, kRowsKind[4].waves * kWave, lds, st>>>(a);
    return hipGetLastError();
}

}  // namespace swr
