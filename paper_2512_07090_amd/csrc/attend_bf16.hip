// Causal softmax attention over the kept tokens, bf16 inputs: which form of the kernel (attend_bf16.h) a call
// gets, and its launch.
#include "attend_bf16.h"
#include "attend_plan.h"

#include <algorithm>

namespace tf {

hipError_t launch_attend_bf16_halves(const Dims& d, float scale_log2, int n_qt, int grid, const uint16_t* Q,
                                     const uint16_t* K, const uint16_t* V, const int32_t* kept_idx, uint16_t* O,
                                     int n_cu, int n_xcd, const int32_t* counts, long long idx_stride, hipStream_t s);

hipError_t launch_attend_bf16(const Dims& d, float scale, const void* Q, const void* K,
                              const void* V, const int32_t* kept_idx, void* O, int n_cu, int n_xcd,
                              const int32_t* counts, int expected, long long idx_stride, hipStream_t s)
{
    // the tile gathers address a row as a 32-bit byte offset from its (batch, head) slice
    if (d.n > (1 << 24) || d.kvs[2] * 2 >= (1 << 24) || (long long)d.n * d.kvs[2] * 2 >= (1ll << 32))
        return hipErrorInvalidValue;
    n_xcd = std::max(n_xcd, 1);
    n_cu = std::max(n_cu, 1);
    const AttendForm form = plan_attend(d.B, d.Hq, counts ? std::min(expected, d.m) : d.m, counts != nullptr, n_cu, n_xcd);
    // with per-row counts d.m is the bound (the longest possible row)
    const int tile = form == kHalves || form == kNarrow ? 128 : 256, n_qt = (d.m + tile - 1) / tile;
    // persistent workgroups: as many as are resident at once; where there is less to do, as many as the XCD with the
    // most groups has tiles, on every XCD (a lone group's tiles are all one XCD's: with a workgroup per
    // tile in all, one eighth of them, 1 head x 1024 took 108 us instead of 22, and 82 with tiles of 256)
    const long long per_xcd = ((long long)d.B * d.Hq + n_xcd - 1) / n_xcd * n_qt;
    const int grid = (int)std::max<long long>(n_xcd, std::min<long long>(per_xcd * n_xcd, (long long)(form == kNarrow ? 2 : 1) * n_cu));
    const float scale_log2 = scale * 1.44269504088896340736f;
    if (!counts) idx_stride = d.m;
#define TF_ATTEND(NW, SINGLES)                                                                 \
    attend_bf16_kernel<NW, 2, SINGLES><<<dim3(grid), dim3(64 * NW), 0, s>>>(                   \
        d, scale_log2, n_qt, n_xcd, n_cu, (const uint16_t*)Q, (const uint16_t*)K,              \
        (const uint16_t*)V, kept_idx, (uint16_t*)O, counts, idx_stride)
    switch (form) {
    case kPairs: TF_ATTEND(8, false); break;
    case kSingles: TF_ATTEND(8, true); break;
    case kNarrow: TF_ATTEND(4, true); break;
    case kHalves:
        return launch_attend_bf16_halves(d, scale_log2, n_qt, grid, (const uint16_t*)Q, (const uint16_t*)K,
                                         (const uint16_t*)V, kept_idx, (uint16_t*)O, n_cu, n_xcd, counts, idx_stride, s);
    }
#undef TF_ATTEND
    return hipGetLastError();
}

}  // namespace tf
