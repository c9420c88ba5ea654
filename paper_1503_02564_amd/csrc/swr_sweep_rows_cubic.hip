// swr_sweep_rows_cubic.hip -- instantiates the row form of the sweep for the |u|^2
// potential (Robin and S0^2): one task per wave, the V-free record in
// registers, the inner iteration of eq. AvMNL on it.
//
// Bound: the chain of an inner iteration (nodal weights, chunk solve, reduction
// over the lanes, convergence maxima), one wave per task.  128 x 256 cells, 600
// steps: 4.1 ms a sweep in the 64-lane form with history on a second wave, 2.6 ms
// now; the solve 56.7 -> 30.4 ms (its iterations, so its time, depend on the data).
#include "swr_sweep_rows_kernel.h"

namespace swr {

template <int TR>
__global__ __launch_bounds__(kWave, 1) void sweep_rows_cubic_kernel(SweepArgs a) {
    extern __shared__ cd smem[];
    const int4 it = a.items[blockIdx.x];
    auto run = [&](auto pc) { rows_body<decltype(pc)::value, 4, false, 1, TR, VK_CUBIC>(a, it.x, it.y, smem); };
    switch (it.z) {
        case 1: run(std::integral_constant<int, 1>{}); break;
        case 2: run(std::integral_constant<int, 2>{}); break;
        case 3: run(std::integral_constant<int, 3>{}); break;
        case 4: run(std::integral_constant<int, 4>{}); break;
        case 5: run(std::integral_constant<int, 5>{}); break;
        case 6: run(std::integral_constant<int, 6>{}); break;
        case 7: run(std::integral_constant<int, 7>{}); break;
        case 8: run(std::integral_constant<int, 8>{}); break;
    }
}

hipError_t launch_sweep_rows_cubic(const SweepArgs& a, int trans, int nitems, size_t lds, hipStream_t st) {
    if (trans == TR_S02) sweep_rows_cubic_kernel<TR_S02><<<nitems, kWave, lds, st>>>(a);
    else sweep_rows_cubic_kernel<TR_ROBIN><<<nitems, kWave, lds, st>>>(a);
    return hipGetLastError();
}

}  // namespace swr
