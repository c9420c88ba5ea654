// swr_sweep_rows1_reg.hip -- instantiates the row form of the static sweep: four tasks per wave, widths 1 to 8 in registers.
#include "swr_sweep_rows_kernel.h"

namespace swr {

hipError_t launch_sweep_rows1_reg(const SweepArgs& a, int trans, int nitems, size_t lds, hipStream_t st) {
    if (trans == TR_S02) sweep_rows_kernel<1, 1, 8, 99, 1, 2, TR_S02><<<nitems, kRowsKind[1].waves * kWave, lds, st>>>(a);
    else sweep_rows_kernel<1, 1, 8, 99, 1, 2, TR_ROBIN><<<nitems, kRowsKind[1].waves * kWave, lds, st>>>(a);
    return hipGetLastError();
}

}  // namespace swr
