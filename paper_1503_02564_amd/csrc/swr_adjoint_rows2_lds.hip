// swr_adjoint_rows2_lds.hip -- instantiates the adjoint sweep; kind 4: two tasks per wave, records in LDS.
#include "swr_adjoint_kernel.h"

namespace swr {

hipError_t launch_adjoint_rows2_lds(const AdjArgs& a, int trans, int nitems, size_t lds, hipStream_t st) {
    return launch_adj<2, 9, 16, true, kRowsKind[4].waves, 1>(a, trans, nitems, lds, st);
}

}  // namespace swr
