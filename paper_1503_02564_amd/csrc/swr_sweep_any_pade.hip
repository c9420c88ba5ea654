// swr_sweep_any_pade.hip -- instantiates the static sweep with the Pade strategy, all chunk
// widths in one launch.
#include "swr_sweep_kernel.h"

namespace swr {

hipError_t launch_sweep_any_pade(const SweepArgs& a, hipStream_t st) {
    sweep_any_kernel<TR_PADE><<<a.ntasks, kWave, 0, st>>>(a);
    return hipGetLastError();
}

}  // namespace swr
