// swr_adjoint_rows4.hip -- instantiates the adjoint sweep; kind 0: one task per wave, widths 1 to 8.
#include "swr_adjoint_kernel.h"

namespace swr {

hipError_t launch_adjoint_rows4(const AdjArgs& a, int trans, int nitems, size_t lds, hipStream_t st) {
    return launch_adj<4, 1, 8, false, kRowsKind[0].waves, 1>(a, trans, nitems, lds, st);
}

}  // namespace swr
