// Causal softmax attention over the kept tokens, bf16 inputs: which form of the kernel (attend_bf16.h) a call gets, and its
// launch.
#include "attend_bf16.h"

#include <algorithm>

namespace tf {

// How the query tiles are dealt out.  Costs are in key tiles of 64 on one compute unit; a tile of 256
// queries costs its key tiles (4 per 256 ranks) and kItemCost more for its first loads, the masked and
// the finishing iteration and its output rows (fitted: 11 us an item, 1.47 us a key tile).
constexpr double kItemCost = 7.5, kKeyTiles = 4.0;
enum AttendForm {
    kPairs,    // tiles of 256 queries in pairs of equal work
    kSingles,  // the same one by one, longest first
    kHalves,   // tiles of 128 queries, one by one, eight waves of 16
    kNarrow,   // the same, four waves of 32, two workgroups on a compute unit
};

hipError_t launch_attend_bf16_halves(const Dims& d, float scale_log2, int n_qt, int grid, const uint16_t* Q,
                                     const uint16_t* K, const uint16_t* V, const int32_t* kept_idx, uint16_t* O,
                                     int n_cu, int n_xcd, const int32_t* counts, long long idx_stride, hipStream_t s);

static AttendForm plan_attend(int groups, int m, bool ragged, int n_cu, int n_xcd)
{
    const int nq = (m + 255) / 256, n_pairs = (nq + 1) / 2;
    const long long items8 = (long long)groups * nq, items4 = (long long)groups * ((m + 127) / 128);
    // one XCD: its groups, workgroups and pairs
    const int ng = (groups + n_xcd - 1) / n_xcd, nwx = std::max(1, n_cu / n_xcd);
    const long long entries = (long long)ng * n_pairs;
    bool singles = false;
    // Pairs are all alike, so they are best when they fill whole rounds (1 x 40 heads x 2500 kept tokens: 83 us
    // against 97 one by one) and when there are many of them; with few, the last round, or the only
    // one, keeps some workgroups busy with a whole pair while the others have nothing
    // (1 x 32 x 1024: 44 against 35 us; 3 x 32 x 2048: 140 against 131).
    if (nq > 1 && entries <= 16 * nwx) {
        auto tile = [](int t) { return kItemCost + kKeyTiles * t; };   // t: in tiles of 256 ranks, 1-based
        const int full = (int)(entries / nwx), rest = (int)(entries % nwx);
        double in_pairs = 0;
        if (!ragged && full >= 2 && rest > 0 && 2 * rest <= nwx && rest <= ng && nq % 2 == 0)
            in_pairs = full * (tile(nq) + tile(1)) + tile(nq / 2 + 1);   // the kernel splits the last round's pairs
        else
            for (int j = 0; j < nwx; ++j) {
                double sum = 0;
                for (long long e = j; e < entries; e += nwx) {
                    const int pr = (int)(e % n_pairs);
                    sum += tile(nq - pr) + (pr != nq - 1 - pr ? tile(pr + 1) : 0.0);
                }
                in_pairs = std::max(in_pairs, sum);
            }
        double one_by_one = 0;
        for (int j = 0; j < nwx; ++j) {   // (odd rounds backwards)
            double sum = 0;
            for (long long r = 0, e; r * nwx < (long long)ng * nq; ++r)
                if ((e = r * nwx + (r & 1 ? nwx - 1 - j : j)) < (long long)ng * nq) sum += tile(nq - (int)(e / ng));
            one_by_one = std::max(one_by_one, sum);
        }
        // (ragged rows are listed row by row, not by length: only where every tile has a place at once)
        singles = one_by_one < 0.97 * in_pairs && (!ragged || items8 <= n_cu);
    }
    // Tiles of 128 queries while there are at most two for each compute unit: beyond, they load every key tile
    // twice as often (8 x 32 x 2048: 410 against 326 us; 8 x 32 x 700: 78 against 66).  A row that half fills a
    // tile of 256 never pays for the other half (8 x 40 x 120: 16.7 against 20.5); one that fills it
    // is best left whole when there is one for each compute unit (8 x 32 x 240: 22 against 19.5).
    const bool small = (nq == 1 || singles) && (m <= 128 || items4 <= n_cu || (nq >= 2 && items4 <= 2 * n_cu));
    if (!small) return singles ? kSingles : kPairs;
    // One for each: by eight waves, which take about as long for a key tile as four but share the first loads and the
    // output rows (1 x 32 x 167: 11.4 -> 8.7 us, x 1024: 28.1 -> 24.9).  More: two rounds of these, or by four waves with two
    // workgroups on a compute unit, whichever the longest sequence of tiles in an XCD says (us, fitted within a tenth: 1 x 32 x
    // 1536: 32 and 36; 2 x 32 x 600: 18.4 and 21; 2 x 40 x 700: 25.3 and 22.6; 1 x 32 x 2048: 48 and 47).
    if (items4 <= n_cu) return kHalves;
    if (nq == 1) return kNarrow;
    const int n_tiles = (m + 127) / 128, n_items = ng * n_tiles;
    auto keys = [&](int e) { return 2 * (n_tiles - e / ng); };   // key tiles of the e-th tile of the list
    double halves = 0, narrow = 0;
    for (int j = 0; j < nwx; ++j) {
        const int with = std::min(n_items, 2 * nwx) - 1 - j;    // the tile that goes with the j-th in the four waves' plan
        narrow = std::max(narrow, with >= nwx ? 8.5 + 1.42 * keys(with) + 1.2 * (keys(j) - keys(with)) : 7.5 + 1.2 * keys(j));
        const int next = 2 * nwx - 1 - j;                       // in the second round of the eight waves'
        halves = std::max(halves, 6.0 + 1.1 * keys(j) + (next < n_items ? 6.0 + 1.1 * keys(next) : 0.0));
    }
    return halves <= narrow ? kHalves : kNarrow;
}

hipError_t launch_attend_bf16(const Dims& d, float scale, const void* Q, const void* K,
                              const void* V, const int32_t* kept_idx, void* O, int n_cu, int n_xcd,
                              const int32_t* counts, int expected, long long idx_stride, hipStream_t s)
{
    // the tile gathers address a row as a 32-bit byte offset from its (batch, head) slice
    if (d.n > (1 << 24) || d.kvs[2] * 2 >= (1 << 24) || (long long)d.n * d.kvs[2] * 2 >= (1ll << 32))
        return hipErrorInvalidValue;
    n_xcd = std::max(n_xcd, 1);
    n_cu = std::max(n_cu, 1);
    const AttendForm form = plan_attend(d.B * d.Hq, counts ? std::min(expected, d.m) : d.m, counts != nullptr, n_cu, n_xcd);
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
