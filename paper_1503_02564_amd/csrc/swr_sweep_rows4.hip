// swr_sweep_rows4.hip -- instantiates the row form of the static sweep: one task per wave, widths 1 to 8 in registers.
#include "swr_sweep_rows_kernel.h"

namespace swr {

hipError_t launch_sweep_rows4(const SweepArgs& a, int trans, int nitems, size_t lds, hipStream_t st) {
    if (trans == TR_S02) sweep_rows_kernel<4, 1, 8, 99, 1, 1, TR_S02><<<nitems, kRowsKind[0].waves * kWave, lds, st>>>(a);
    else sweep_rows_kernel<4, 1, 8, 99, 1, 1, TR_ROBIN><<<nitems, kRowsKind[0].waves * kWave, lds, st>>>(a);
    return hipGetLastError();
}

}  // namespace swr
