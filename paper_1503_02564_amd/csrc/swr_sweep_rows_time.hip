// swr_sweep_rows_time.hip -- the row form of the sweep for V(t,x) (Robin and
// S0^2), with the factor record of every step read from memory.
//
// The potential is given in advance, so the matrices of all steps are factored
// by one launch (launch_rows_factor over steps), which fills the GPU, before the
// first sweep of a call instead of inside every step of every sweep, where one
// wave per task waits for a chain of P + 6 reciprocals.  A sweep is then that of
// a static potential whose record changes from step to step: wave 0 of a
// workgroup sweeps, three helper waves fetch records, each every third one,
// three steps ahead into registers and one step ahead into LDS.
//
// Bound: a record is 16 KB (P = 1) to 46 KB (P = 8) per task and step, so memory
// bandwidth from about 100 tasks on.  128 x 256 cells, 400 steps: 1626 us a sweep
// that refactored, 416 us now (4.2 TB/s) and 201 us once per solve for the records;
// the preconditioned GMRES solve with 20 sweeps 45.0 -> 21.6 ms.
// The line to the refactoring sweep (swr_sweep_kernel.h) is kTimeRecordTasks.
#include "swr_sweep_rows_kernel.h"

namespace swr {

// The records of the launch's steps, in step order, into two alternating LDS
// slots: record n is in its slot before barrier n (the step's), which the
// sweeping wave passes before it reads it; that wave has done with the slot's
// last record before barrier n - 1.
template <int P>
__device__ __forceinline__ void time_helper(const SweepArgs& a, int first, cd* slots) {
    constexpr int NF = rows_fields(P, 4), HELPERS = 3;
    const int lane = threadIdx.x & (kWave - 1);
    const int h = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave) - 1;
    const int steps = a.n_end - a.n_begin;
    const size_t stride = (size_t)a.N * a.rstride;
    const cd* src = a.tfac + ((size_t)(a.n_begin - a.tfac_begin) * a.N + a.tasks[first].k) * a.rstride + lane;
    // (reads past the last step repeat it)
    cd r[NF];
    auto read = [&](int n) __attribute__((always_inline)) {
        const cd* p = src + (size_t)min(n, steps - 1) * stride;
#pragma unroll
        for (int f = 0; f < NF; ++f) r[f] = mk(p[f * kWave].x, p[f * kWave].y);
    };
    read(h);
    __syncthreads();                                  // rows_body's first
    for (int n = 0; n < steps; ++n) {
        if (n % HELPERS == h) {
            // (by component: copies of whole entries, memory to memory by way of r,
            // would leave r in scratch memory)
            cd* dst = slots + (n & 1) * (NF * kWave) + lane;
#pragma unroll
            for (int f = 0; f < NF; ++f) dst[f * kWave] = mk(r[f].x, r[f].y);
            read(n + HELPERS);
        }
        __syncthreads();
    }
}

template <int TR>
__global__ __launch_bounds__(4 * kWave, 1) void sweep_rows_time_kernel(SweepArgs a) {
    extern __shared__ cd smem[];
    const int4 it = a.items[blockIdx.x];
    cd* slots = smem + kRowsBetaLds / 2 + kRowsWaveLds;
    auto run = [&](auto pc) {
        constexpr int P = decltype(pc)::value;
        if (threadIdx.x >= kWave) time_helper<P>(a, it.x, slots);
        else rows_body<P, 4, false, 1, TR, VK_TIME>(a, it.x, it.y, smem);
    };
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

hipError_t launch_sweep_rows_time(const SweepArgs& a, int trans, int nitems, size_t lds, hipStream_t st) {
    if (!a.tfac || a.n_begin < a.tfac_begin) return hipErrorInvalidValue;
    if (trans == TR_S02) sweep_rows_time_kernel<TR_S02><<<nitems, 4 * kWave, lds, st>>>(a);
    else sweep_rows_time_kernel<TR_ROBIN><<<nitems, 4 * kWave, lds, st>>>(a);
    return hipGetLastError();
}

}  // namespace swr
