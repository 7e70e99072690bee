// Causal softmax attention over the kept tokens, bf16 inputs: tiles of 128 queries by eight waves of 16
// (plan_attend() says when).
#include "attend_bf16.h"

namespace tf {

hipError_t launch_attend_bf16_halves(const Dims& d, float scale_log2, int n_qt, int grid, const uint16_t* Q,
                                     const uint16_t* K, const uint16_t* V, const int32_t* kept_idx, uint16_t* O,
                                     int n_cu, int n_xcd, const int32_t* counts, long long idx_stride, hipStream_t s)
{
    attend_bf16_kernel<8, 1, true><<<dim3(grid), dim3(512), 0, s>>>(d, scale_log2, n_qt, n_xcd, n_cu, Q, K, V, kept_idx,
                                                                    O, counts, idx_stride);
    return hipGetLastError();
}

}  // namespace tf
