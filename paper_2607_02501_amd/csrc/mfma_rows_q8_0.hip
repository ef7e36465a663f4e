// mfma_rows_q8_0.hip -- the small-m kernels (mfma_rows.h) for Q8_0 weights.
// Built with the MFMA results in VGPRs: they are scaled by the VALU at once,
// and from accumulation registers each would take a move first (64 per step
// and wave of the largest tile).
#include "mfma_rows.h"

namespace eb {

template hipError_t rows_lone<EB_Q8_0>(int32_t, const RowsTiles &, const MMOp &, int, float *, int64_t,
                                       hipStream_t);
template hipError_t rows_multi<EB_Q8_0>(int32_t, const RowsTiles &, const MMOp *, int, int64_t,
                                        hipStream_t);

}  // namespace eb
