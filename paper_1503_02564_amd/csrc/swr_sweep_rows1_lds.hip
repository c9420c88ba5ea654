// swr_sweep_rows1_lds.hip -- instantiates the row form of the static sweep: four tasks per wave, widths 9 to 14 from LDS.
#include "swr_sweep_rows_kernel.h"

namespace swr {

hipError_t launch_sweep_rows1_lds(const SweepArgs& a, int trans, int nitems, size_t lds, hipStream_t st) {
    if (trans == TR_S02) sweep_rows_kernel<1, 9, 14, 9, 2, 2, TR_S02><<<nitems, kRowsKind[2].waves * kWave, lds, st>>>(a);
    else sweep_rows_kernel<1, 9, 14, 9, 2, 2, TR_ROBIN><<<nitems, kRowsKind[2].waves * kWave, lds, st>>>(a);
    return hipGetLastError();
}

}  // namespace swr
