// swr_sweep_any_gen.hip -- instantiates the static sweep with the higher-order operators, all chunk
// widths in one launch.
#include "swr_sweep_kernel.h"

namespace swr {

hipError_t launch_sweep_any_gen(const SweepArgs& a, hipStream_t st) {
    sweep_any_kernel<TR_GEN><<<a.ntasks, kWave, 0, st>>>(a);
    return hipGetLastError();
}

}  // namespace swr
