// 3-bit instances of the matrix-core kernel for any row length.
#include "kmq_mfma_any.h"

namespace kmq {
hipError_t launch_canon_b3(const GemmArgs& a, hipStream_t s) { return canon_dispatch<3>(a, s); }
}  // namespace kmq
