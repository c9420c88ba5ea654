// swr_adjoint_rows1_lds.hip -- instantiates the adjoint sweep; kind 2: four tasks per wave, records in LDS.
#include "swr_adjoint_kernel.h"

namespace swr {

hipError_t launch_adjoint_rows1_lds(const AdjArgs& a, int trans, int nitems, size_t lds, hipStream_t st) {
    return launch_adj<1, 9, 14, true, kRowsKind[2].waves, 1>(a, trans, nitems, lds, st);
}

}  // namespace swr
