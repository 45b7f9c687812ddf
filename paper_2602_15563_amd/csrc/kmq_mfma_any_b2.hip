// 2-bit instances of the matrix-core kernel for any row length.
#include "kmq_mfma_any.h"

namespace kmq {
hipError_t launch_canon_b2(const GemmArgs& a, hipStream_t s) { return canon_dispatch<2>(a, s); }
}  // namespace kmq
