// swr_adjoint_rows2_reg.hip -- instantiates the adjoint sweep; kind 3: two tasks per wave, widths 1 to 8.
#include "swr_adjoint_kernel.h"

namespace swr {

hipError_t launch_adjoint_rows2_reg(const AdjArgs& a, int trans, int nitems, size_t lds, hipStream_t st) {
    return launch_adj<2, 1, 8, false, kRowsKind[3].waves, 1>(a, trans, nitems, lds, st);
}

}  // namespace swr
