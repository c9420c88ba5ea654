// swr_sweep_static.hip -- instantiates the subdomain sweep for a time-independent
// potential with the higher-order transmissions (the Pade strategy is in
// swr_sweep_static_pade.hip; Robin and S0^2 have the row form, swr_sweep_rows.hip).
#include "swr_sweep_kernel.h"

namespace swr {

template <int P>
static void launch_p(const SweepArgs& a, hipStream_t st) {
    sweep_kernel<P, TR_GEN, VK_STATIC><<<a.ntasks, sweep_threads(false), 0, st>>>(a);
}

hipError_t launch_sweep_any_gen(const SweepArgs& a, hipStream_t st);
hipError_t launch_sweep_any_pade(const SweepArgs& a, hipStream_t st);

hipError_t launch_sweep_any(const SweepArgs& a, int trans, hipStream_t st) {
    if (a.ntasks == 0) return hipSuccess;
    if (!a.endc) return hipErrorInvalidValue;
    if (trans == TR_GEN) return launch_sweep_any_gen(a, st);
    if (trans == TR_PADE && a.pade && a.pade_m >= 1 && a.pade_m <= kPadeMax) return launch_sweep_any_pade(a, st);
    return hipErrorInvalidValue;
}

hipError_t launch_sweep_static(const SweepArgs& a, int trans, hipStream_t st) {
    if (trans == TR_PADE) return launch_sweep_static_pade(a, st);
    if (trans != TR_GEN || !a.endc) return hipErrorInvalidValue;
    switch (a.P) {
        case 1: launch_p<1>(a, st); break;
        case 2: launch_p<2>(a, st); break;
        case 3: launch_p<3>(a, st); break;
        case 4: launch_p<4>(a, st); break;
        case 5: launch_p<5>(a, st); break;
        case 6: launch_p<6>(a, st); break;
        case 7: launch_p<7>(a, st); break;
        case 8: launch_p<8>(a, st); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace swr
