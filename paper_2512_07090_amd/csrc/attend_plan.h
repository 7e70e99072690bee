// Which form of the bf16 attention kernel (attend_bf16.h) a call gets.  Host code only.
#pragma once
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

// The list of single tiles that the workgroups of an XCD share, as the kernel lists it: uniform rows longest
// tiles of all groups first, ragged rows one row after the other (every row taken as long as expected).
struct TileList {
    int first_group, groups;   // the XCD's (batch row, head) groups
    int Hq, tiles;             // tiles of a row
    bool ragged;
    int size() const { return groups * tiles; }
    int length(int e) const    // of the keys that the e-th entry walks, in tiles
    {
        if (!ragged) return tiles - e / groups;
        int of_row = std::min(groups, Hq - first_group % Hq);   // groups of the first row
        if (e >= of_row * tiles) {
            e -= of_row * tiles;
            const int rows = e / (Hq * tiles);
            e -= rows * Hq * tiles;
            of_row = std::min(Hq, groups - of_row - rows * Hq);
        }
        return tiles - e / of_row;
    }
};

// Cost of the longest sequence of tiles when `workgroups` walk a list in rounds, the odd ones backwards.
inline double longest_sequence(const TileList& list, int workgroups, double item, double per_tile)
{
    double most = 0;
    for (int j = 0; j < workgroups; ++j) {
        double sum = 0;
        for (int r = 0, e; r * workgroups < list.size(); ++r)
            if ((e = r * workgroups + (r & 1 ? workgroups - 1 - j : j)) < list.size()) sum += item + per_tile * list.length(e);
        most = std::max(most, sum);
    }
    return most;
}

// The same of the four waves' form, in us: two workgroups on a compute unit, of which the second walks each
// round backwards; together they take 1.42 us for a key tile of 64, the one that is left alone 1.2.
inline double longest_of_two(const TileList& list, int n_cu)
{
    const int workgroups = std::min(list.size(), 2 * n_cu);
    double most = 0;
    for (int j = 0; j < n_cu; ++j) {
        int keys[2] = {0, 0};
        for (int r = 0; r < list.size(); r += workgroups)
            for (int i = 0; i < 2; ++i) {
                const int at = i ? workgroups - 1 - j : j, e = r + at;
                if (at >= i * n_cu && e < list.size()) keys[i] += 2 * list.length(e);
            }
        const int both = std::min(keys[0], keys[1]);
        most = std::max(most, (both ? 8.5 : 7.5) + 1.42 * both + 1.2 * (std::max(keys[0], keys[1]) - both));
    }
    return most;
}

inline AttendForm plan_attend(int B, int Hq, int m, bool ragged, int n_cu, int n_xcd)
{
    const int groups = B * Hq;
    const int nq = (m + 255) / 256, n_pairs = (nq + 1) / 2;
    const long long items8 = (long long)groups * nq, items4 = (long long)groups * ((m + 127) / 128);
    // one XCD: its groups, workgroups and pairs
    const int ng = (groups + n_xcd - 1) / n_xcd, nwx = std::max(1, n_cu / n_xcd);
    const long long entries = (long long)ng * n_pairs;
    // the largest of cost(list) over the XCDs with the most groups (their lists are all alike for uniform
    // rows, and where rows and XCDs meet at the same groups)
    const bool alike = !ragged || (groups % n_xcd == 0 && (Hq % ng == 0 || ng % Hq == 0));
    auto over_xcds = [&](int tiles, auto cost) {
        double most = 0;
        for (int x = alike ? n_xcd - 1 : 0; x < n_xcd; ++x) {
            const int g_lo = (int)((long long)x * groups / n_xcd), g_hi = (int)((x + 1ll) * groups / n_xcd);
            if (g_hi - g_lo == ng) most = std::max(most, cost(TileList{g_lo, ng, Hq, tiles, ragged}));
        }
        return most;
    };
    bool singles = false;
    double one_by_one = 0;
    // Pairs are all alike, so they are best when they fill whole rounds (1 x 40 heads x 2500 kept tokens: 83
    // us against 97 one by one) and when there are many of them; with few, the last round, or the only one,
    // keeps some workgroups busy with a whole pair while the others have nothing (1 x 32 x 1024: 44 against
    // 35 us; 3 x 32 x 2048: 140 against 131).  Ragged rows are listed row by row: only where there is a
    // compute unit for every tile on the chip, and an XCD that lists two rows may still give its workgroups
    // two long ones (9 rows of 1 head x 7000: 249 us, 173 in pairs; 1 row of 9 heads 163 and 172).
    if (nq > 1 && entries <= 16 * nwx && (!ragged || items8 <= n_cu)) {
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
        one_by_one = over_xcds(nq, [&](const TileList& list) { return longest_sequence(list, nwx, kItemCost, kKeyTiles); });
        singles = one_by_one < 0.97 * in_pairs;
    }
    // Tiles of 128 queries while there are at most two for each compute unit: beyond, they load every key
    // tile twice as often (8 x 32 x 2048: 410 against 326 us; 8 x 32 x 700: 78 against 66).  A row that half
    // fills a tile of 256 never pays for the other half (8 x 40 x 120: 16.7 against 20.5); one that fills it
    // is best left whole when there is one for each compute unit (8 x 32 x 240: 22 against 19.5).
    const bool small = (nq == 1 || singles) && (m <= 128 || items4 <= n_cu || (nq >= 2 && items4 <= 2 * n_cu));
    if (!small) return singles ? kSingles : kPairs;
    // One for each: by eight waves, which take about as long for a key tile as four but share the first loads
    // and the output rows (1 x 32 x 167: 11.4 -> 8.7 us, x 1024: 28.1 -> 24.9).  More: these in rounds, or by
    // four waves with two workgroups on a compute unit, whichever the longest sequence of tiles in an XCD
    // says (us, fitted within a tenth: 1 x 32 x 1536: 32 and 36; 2 x 32 x 600: 18.4 and 21; 2 x 40 x 700:
    // 25.3 and 22.6; 1 x 32 x 2048: 48 and 47).  A group's tiles are all one XCD's, so one XCD may have far
    // more than two for each of its own compute units: there the tiles of 256 may win all the same (eight
    // waves, four, tiles of 256: 1 x 9117: 199, 190 and 211; 1 x 13000: 391, 342 and 309; 9 x 7000: 219, 194
    // and 161).
    const int n_tiles = (m + 127) / 128;
    const long long n_items = (long long)ng * n_tiles;
    if (n_items <= nwx) return kHalves;
    if (nq == 1) return kNarrow;
    const double halves = over_xcds(n_tiles, [&](const TileList& list) { return longest_sequence(list, nwx, 6.0, 2.2); });
    const double narrow = over_xcds(n_tiles, [&](const TileList& list) { return longest_of_two(list, nwx); });
    if (n_items > 2 * nwx && 1.47 * one_by_one < std::min(halves, narrow)) return kSingles;
    return halves <= narrow ? kHalves : kNarrow;
}

}  // namespace tf
