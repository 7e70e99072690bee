// Causal softmax attention over the kept tokens, bf16 inputs (Section 3.2: the tokens that
// are not skipped attend as usual and a skipped token's attention output is zero; here both
// queries and keys are the kept tokens, addressed through kept_idx, so "causal" means key rank
// <= query rank in the compacted order).
//
// Flash-style kernel for gfx950.  One work item covers 256 (eight waves of two blocks of 16: NW = 8, QB = 2)
// or 128 (QB = 1, or NW = 4) kept queries, two waves per SIMD with 256 registers each.  It walks the key
// tiles (64 kept keys) once, K and V rows gathered through kept_idx into LDS (two stages each).
//   S^T = K Q^T   v_mfma_f32_16x16x32_bf16, A = K rows from LDS, B = Q fragments held in
//                 registers for the whole item.  The transposed product puts one query per
//                 lane column, so P^T goes from the accumulators to the next product's operand
//                 without leaving the lane.
//   O^T += V^T P^T  A = V^T from LDS, written there already transposed (a pair of lanes swaps halves
//                 and permutes 16-bit words), so that a fragment is one 16-byte read: the
//                 transposing LDS read moves half as much per instruction.  The contraction
//                 order over keys is permuted the same way for both operands (k-slot 8 g + e of a
//                 32-key block is key 4 g + e, or 16 + 4 g + e - 4 for e >= 4).
//   LDS layout    K rows padded to 288 bytes, V^T slots XOR-ed: the 16 lanes that LDS serves together
//                 in a 16-byte read touch every bank once (4.7 cycles a read instead of 8 to 12); the
//                 writes of V^T meet in half of the banks.
//   MFMA shape    16x16x32 rather than 32x32x16: same rate, same operands from LDS, but on normally
//                 distributed data the card clocks down less (2.03 against 1.78 PFLOP/s in a loop
//                 of nothing else, 2.45 both on zeros).
//   softmax       fp32, base 2 (scale * log2 e folded into one FMA per score), against a reference
//                 that moves only when a row outgrows it (see neg_mc): no row maximum on the way.
//                 The denominators are summed on the matrix pipe from the weights as rounded
//                 (l_ones), so every output row is an exact convex combination of value rows;
//                 v_dot2_f32_bf16, which did it before, occupies that pipe for about 20 cycles each
//                 (0.66 against 0.60 us per 32 keys in a copy of the loop).
//   pipeline      Scores run one 32-key block ahead of the weights and the product with V one block
//                 behind them, so that in a block the MFMAs, the 16 exponentials and the 16 LDS reads
//                 do not depend on each other; they are interleaved chunk by chunk in program
//                 order.  The blocks that begin and end a wave's walk are instances of the same
//                 body with parts left out.
//   tile loads    A tile's rows are requested right after the registers they land in have been
//                 written to LDS, a whole iteration ahead of their use, and land in one register
//                 set (requested at the start of the iteration that delivers them the launch took
//                 0.299 instead of 0.282 ms at 8 x 32 heads x 2048 kept on all-zero inputs).
//   zero rows     The rows of the filtered positions between a query and the next kept token
//                 are written as zeros together with the query's row (kept_idx is ascending).
//   small calls   Eight waves of 16 queries take a key tile in about the time of four waves of 32 (1.1 us;
//                 they read twice the operands from LDS) and share an item's first loads and output rows,
//                 which is most of a short item: 1 x 32 heads x 167 kept 11.4 -> 8.7 us, x 512 18.2 -> 15.8,
//                 x 1024 28.1 -> 24.9.  (In 128 registers, two such workgroups on a CU, they spill: 70 us.)
//   scheduling    One persistent workgroup of eight waves per CU (or two of four) walks a static list of pairs
//                 of query tiles (tile p with tile n_qt - 1 - p: equal causal work) or, where there
//                 are too few pairs to go round, of single tiles; see the kernel and plan_attend().
// What bounds it: with real data the card runs at its power limit (1.4 kW) and clocks down; a
// library GEMM of 8192^3 reaches 1.2-1.36 PFLOP/s there, this kernel 1.25 at 32 heads x 16384 kept
// tokens (1.99 -> 1.76 ms; all-zero inputs 1.72 -> 1.54).  With short rows each item's start and
// end show: 8 x 32 heads x 2048 kept 0.341 -> 0.311 ms, of which about 8 x 11 us are the items'
// first loads, masked tiles and output rows.
#pragma once
#include "tf_kernels.h"

namespace tf {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));

constexpr int kBN = 64;                  // kept keys per tile
constexpr int kKStr = kHeadDim + 16;     // K tile row stride, elements (288 B)
constexpr int kVStr = kBN;               // V^T tile row stride (one row per column of V), elements (128 B)
constexpr int kKTile = kBN * kKStr;      // elements per K tile
constexpr int kVTile = kHeadDim * kVStr; // elements per V^T tile
constexpr int kOStr = kHeadDim + 8;      // output staging row stride, elements
constexpr float kSumLimit = 16777216.f;  // 2^24: largest softmax denominator in the tile loop, see below
constexpr float kMasked = -1e30f;

// Two floats rounded to bf16 and packed into one register (v_cvt_pk_bf16_f32).  The words are handled as plain
// unsigned values and only the assembled operand is reinterpreted as eight bf16 values:
// extracting words from a bf16 vector after element-wise stores made this compiler read the
// first word four times.
__device__ __forceinline__ unsigned pack_bf16x2(float a, float b)
{
    const f32x2 v = {a, b};
    return __builtin_bit_cast(unsigned, __builtin_convertvector(v, bf16x2));
}
// 16 bytes to global memory with the non-temporal hint (the line is not kept in the L2)
__device__ __forceinline__ void store_streaming(uint16_t* dst, uint4 v)
{
    __builtin_nontemporal_store(__builtin_bit_cast(u32x4, v), reinterpret_cast<u32x4*>(dst));
}

// Four keys x eight columns of V held by a pair of lanes 32 apart (the lower lane: keys k, k + 1
// in r0, r1; the upper lane: keys k + 2, k + 3) to the V^T tile: the half swap gives the lower
// lane columns 0-3 of all four keys and the upper lane columns 4-7, then 16-bit permutes put the
// four keys of a column side by side.  dst: this lane's first column at the keys' place.
__device__ __forceinline__ void store_v_transposed(u32x4 r0, u32x4 r1, uint16_t* tile, int off)
{
#pragma unroll
    for (int w = 0; w < 2; ++w) {
        const auto s0 = __builtin_amdgcn_permlane32_swap(r0[w], r0[w + 2], false, false);
        const auto s1 = __builtin_amdgcn_permlane32_swap(r1[w], r1[w + 2], false, false);
        // words of two columns: keys k, k + 1, k + 2, k + 3
        const unsigned k0 = s0[0], k2 = s0[1], k1 = s1[0], k3 = s1[1];
        const u32x2 even = {__builtin_amdgcn_perm(k1, k0, 0x05040100u), __builtin_amdgcn_perm(k3, k2, 0x05040100u)};
        const u32x2 odd = {__builtin_amdgcn_perm(k1, k0, 0x07060302u), __builtin_amdgcn_perm(k3, k2, 0x07060302u)};
        // column i of the lane's four is row i and carries i in its slot's XOR
        *reinterpret_cast<u32x2*>(tile + ((off ^ (8 * (2 * w))) + (2 * w) * kVStr)) = even;
        *reinterpret_cast<u32x2*>(tile + ((off ^ (8 * (2 * w + 1))) + (2 * w + 1) * kVStr)) = odd;
    }
}

// c += a b, and c = a b, as instructions of their own whose accumulator stays in one place: left to
// itself the compiler gives every such MFMA a destination of its own and spills.  It does not
// know their latency either, so what else reads a result, or takes over its registers, is tied to a place
// behind the MFMA where it has been written:
//   mfma_settle()  waits out the MFMAs issued before it; the two accumulators it names are read, and
//                  all their registers (l_acc: also the rows nobody reads) stay theirs, up to here;
//   mfma_result()  names a result where it is first read, in the tile loop two chunks, that is at least
//                  four MFMAs, after its last one (they leave the pipe in order).
// Neither moves against an MFMA.  tests/test_mfma_distances.py measures the distances in the assembly.
__device__ __forceinline__ void mfma_add(f32x4& c, bf16x8 a, bf16x8 b)
{
    asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+v"(c) : "v"(a), "v"(b));
}
__device__ __forceinline__ void mfma_first(f32x4& c, bf16x8 a, bf16x8 b)
{
    asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, 0" : "=&v"(c) : "v"(a), "v"(b));
}
__device__ __forceinline__ void mfma_settle(f32x4& c0, f32x4& c1)
{
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_nop 15\n\ts_nop 15" : "+v"(c0), "+v"(c1) : : "memory");
    __builtin_amdgcn_sched_barrier(0);
}
__device__ __forceinline__ void mfma_result(f32x4& c) { asm volatile("" : "+v"(c)); }

template <int NW, int QB, bool SINGLES>
__global__ __launch_bounds__(64 * NW, 2) void attend_bf16_kernel(
    Dims d, float scale_log2, int n_qt, int n_xcd, int n_cu, const uint16_t* __restrict__ Q,
    const uint16_t* __restrict__ K, const uint16_t* __restrict__ V,
    const int32_t* __restrict__ kept_idx, uint16_t* __restrict__ O,
    const int32_t* __restrict__ counts, long long idx_stride)
{
    constexpr int NT = 64 * NW;    // threads
    constexpr int NP = 8 / NW;     // passes of the workgroup over a tile when loading it
    constexpr int WQ = 16 * QB;    // queries per wave
    constexpr int kBM = WQ * NW;   // kept queries per work item
    // operand fragments in flight from LDS, per tensor (four waves, which hold two passes of rows: with three
    // 24 registers are spilled, 9 with two, all of them outside the tile loop; eight waves spill none in
    // pairs, 2 one by one; with QB = 1 four to eight are no faster than three)
    constexpr int kRing = NW == 8 ? 3 : 2;
    __shared__ __attribute__((aligned(16))) uint16_t smem[2 * kKTile + 2 * kVTile];
    uint16_t* const k_lds = smem;               // 2 stages of K
    uint16_t* const v_lds = smem + 2 * kKTile;  // 2 stages of V^T
    // Tiles of 256: output staging of its own (141 KB of LDS in all): a wave stages and writes its rows
    // without a workgroup barrier on either side, so the waves leave an item, and start on the next item's
    // first loads, as each gets there.  Tiles of 128: the rows are staged over the K tiles, behind the tile
    // loop's last barrier, and a barrier of its own keeps the next item's first K tile from them; four waves
    // so that two workgroups share a CU's LDS (70 KB each) and overlap each other's item ends.
    constexpr bool kOwnStage = NW == 8 && QB == 2;
    __shared__ __attribute__((aligned(16))) uint16_t own_stage[kOwnStage ? kBM * kOStr : 8];
    uint16_t* const ostage = kOwnStage ? own_stage : k_lds;
    static_assert(kOwnStage || kBM * kOStr <= 2 * kKTile, "staging fits the K stages");

    __shared__ int overflow;   // a row of the item at hand has outgrown its reference
    __shared__ unsigned lost_rows[NW];   // a wave's queries that have, bit 16 qb + c16 (no registers in the tile loop)

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // uniform: branches on it are scalar

    // Persistent workgroups, one per CU, with a static schedule.  (Left to the hardware
    // dispatcher, one workgroup per query tile, CUs sit idle for many microseconds whenever a
    // workgroup ends: it hands out workgroups in order, and the durations of causal query tiles
    // differ by a factor of n_qt.)  The (batch, head) groups are split into n_xcd contiguous
    // runs, one per XCD (the count is the device's, read by the host), so an XCD's L2 holds the
    // K and V of the few groups it is working on.  Correctness does not depend on where a
    // workgroup really runs, only the L2 hit rate does.
    const int n_groups = d.B * d.Hq;
    // Static schedule (SINGLES: an entry is one tile; uniform rows list the longest tiles of all groups
    // first): workgroup j of XCD x (x = id % n_xcd, as the dispatcher deals them) walks entries j, j + W, ...
    // of the XCD's list of (group, pair of query tiles); a pair joins query tile p with n_qt - 1 - p, so
    // every entry is the same amount of causal work, and the workgroups that share a group start on it
    // together and stream the same K / V tiles.
    const int x = blockIdx.x % n_xcd, j = blockIdx.x / n_xcd;
    const int nwx = (gridDim.x + n_xcd - 1 - x) / n_xcd;  // workgroups whose id % n_xcd is x
    const int g_lo = x * n_groups / n_xcd;
    const int ng = (x + 1) * n_groups / n_xcd - g_lo;
    const int n_pairs = SINGLES ? n_qt : (n_qt + 1) >> 1;
    const int n_entries = ng * n_pairs;

    // Ragged rows (counts != null: every batch row has its own number of kept tokens, read here
    // on the device; n_qt is only the bound for the longest possible row): the XCD's list holds,
    // group after group, as many pairs as the group's row needs (one entry for an empty row,
    // which only has zero rows to write), so that, as in the uniform case, workgroups with
    // neighbouring ids work on the same group.  (rb, row_e0): the batch row the current entry
    // lies in and the first entry of that row; entries only move forward.
    //
    // Uniform rows, last round: when the entries do not fill a whole number of rounds and the
    // rest (L entries) is at most half a round, those L entries are not dealt as pairs, which
    // would keep every other workgroup idle for a whole pair: they are the MIDDLE pairs of the
    // last L groups (the pair whose two tiles are closest in work), taken out of the list of
    // whole rounds, and their 2 L tiles go to workgroups 0 .. 2 L - 1, one tile each (two
    // neighbours share a group).  The last round then lasts one middle tile instead of a pair.
    const int full_rounds = n_entries / nwx;
    const int rest = n_entries - full_rounds * nwx;
    const bool split_rest = !SINGLES && !counts && rest > 0 && 2 * rest <= nwx && rest <= ng && n_pairs >= 2 && (n_qt & 1) == 0;
    const int n_main = split_rest ? n_entries - rest : n_entries;  // entries dealt as pairs
    const int whole_groups = split_rest ? ng - rest : ng;          // groups that keep all their pairs
    int rb = g_lo / d.Hq, row_e0 = 0;
    bool exact = false;  // the item is done again, see below
    for (int it = 0;; ++it) {
    // Tiles one by one, longest first: odd rounds backwards, and of two workgroups on a compute unit the
    // second half of them, so that a long tile goes with a short one (3 x 32 x 2048: 125 -> 115 us; four
    // waves, 1 x 32 x 2048: 49.6 -> 46.7).
    const int first = NW == 8 ? (it & 1 ? 0 : nwx) : n_cu / n_xcd;
    const int e = !SINGLES ? j + (it >> 1) * nwx : it * nwx + (j < first ? j : nwx - 1 - (j - min(first, nwx)));
    int pr, bh, m, nq;
    bool single = false;  // this entry is one tile of a split middle pair
    if (counts) {
        int P = 1;
        bool done = false;
        for (;;) {
            const int lo = max(g_lo, rb * d.Hq), hi = min(g_lo + ng, (rb + 1) * d.Hq);
            if (rb >= d.B || hi <= lo) { done = true; break; }
            m = __builtin_amdgcn_readfirstlane(counts[rb]);  // kept tokens of this row
            nq = (m + kBM - 1) / kBM;                        // its query tiles
            P = m == 0 ? 1 : (SINGLES ? nq : (nq + 1) >> 1);
            if (e < row_e0 + (hi - lo) * P) break;
            row_e0 += (hi - lo) * P;
            ++rb;
        }
        if (done) break;
        const int el = e - row_e0;
        const int row_g = max(g_lo, rb * d.Hq), row_n = min(g_lo + ng, (rb + 1) * d.Hq) - row_g;   // the row's groups here
        bh = row_g + (SINGLES ? el % row_n : el / P);
        pr = SINGLES ? el / row_n : el % P;
    } else {
        m = d.m;
        nq = n_qt;
        if (e < n_main) {
            const int e_whole = whole_groups * n_pairs;  // entries of the groups with all pairs
            if (SINGLES) {   // longest first
                pr = e / ng;
                bh = g_lo + e % ng;
            } else if (e < e_whole) {
                pr = e % n_pairs;
                bh = g_lo + e / n_pairs;
            } else {  // the last groups have given their middle pair away
                pr = (e - e_whole) % (n_pairs - 1);
                bh = g_lo + whole_groups + (e - e_whole) / (n_pairs - 1);
            }
        } else {
            // past the whole rounds: one tile of a middle pair, or nothing
            if (!split_rest || (it >> 1) != full_rounds || (it & 1) || j >= 2 * rest) break;
            single = true;
            pr = n_pairs - 1;
            bh = g_lo + whole_groups + (j >> 1);
        }
    }
    const int b = bh / d.Hq, hq = bh % d.Hq;
    const int hk = hq / (d.Hq / d.Hkv);
    if (m == 0) {
        // a row without kept tokens: nothing attends, every output row is zero
        if (pr == 0 && (SINGLES || !(it & 1))) {
            uint16_t* Oz = O + (long long)b * d.os[0] + (long long)hq * d.os[1] + 8 * (tid & 15);
            for (int g = tid >> 4; g < d.n; g += NT / 16)
                *reinterpret_cast<uint4*>(Oz + (long long)g * d.os[2]) = make_uint4(0, 0, 0, 0);
        }
        continue;
    }
    if (pr >= (SINGLES ? nq : (nq + 1) >> 1)) continue;
    const bool lower = single ? j & 1 : it & 1;
    const int qt = lower && !SINGLES ? pr : nq - 1 - pr;
    if (!SINGLES && !single && (it & 1) && pr == nq - 1 - pr) continue;  // the middle tile of an odd count is alone

    const int32_t* idx = kept_idx + (long long)b * idx_stride;
    const uint16_t* Qb = Q + (long long)b * d.qs[0] + (long long)hq * d.qs[1];
    const char* Kb = reinterpret_cast<const char*>(K + (long long)b * d.kvs[0] + (long long)hk * d.kvs[1]);
    const char* Vb = reinterpret_cast<const char*>(V + (long long)b * d.kvs[0] + (long long)hk * d.kvs[1]);
    uint16_t* Ob = O + (long long)b * d.os[0] + (long long)hq * d.os[1];
    const unsigned kv_row_bytes = (unsigned)d.kvs[2] * 2u;

    const int c16 = lane & 15, g4 = lane >> 4;  // row or column of a 16x16 operand, its group of 8 k-slots
    const int hh = lane >> 5;

    const int i0 = qt * kBM;
    // Waves w and w + NW / 2 share a SIMD.  Causal work grows with the row block, so the
    // second half of the waves takes the row blocks in reverse: every SIMD then carries one
    // early and one late block and the four SIMDs finish together.
    const int blk = wave < NW / 2 ? wave : NW + NW / 2 - 1 - wave;
    const int iw = i0 + WQ * blk;    // first query rank of this wave
    const int i_last = min(i0 + kBM, m) - 1;
    const int n_kt = i_last / kBN + 1;
    const int m_last = m - 1;
    // last key rank this lane's queries (c16 of the wave's two blocks of 16) may see
    int lim[QB];
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) lim[qb] = min(iw + 16 * qb + c16, m_last);
    const int q_last = iw > m_last ? 0 : iw / kBN;  // the last key tile the wave needs

    // tile-load roles: in pass p a thread moves columns 8 c .. + 7 of two neighbouring keys; the
    // lane 32 further holds the two keys after them, so that a pair of lanes can transpose four
    // keys of V, and the waves' keys are dealt so that a wave fills 16-byte slots of V^T.
    // Rows past the last kept token re-read the last kept row: finite values that the mask turns
    // into zero weights, so the loads need no branch.
    // A row's address is the uniform (batch, head) base plus a 32-bit byte offset formed by one 24-bit
    // multiply-add (the launcher checks that a slice spans less than 4 GiB and that positions
    // and row strides stay below 2^24).
    const int c8 = lane & 15;
    auto load_idx = [&](int j) -> int {
        return *reinterpret_cast<const int32_t*>(reinterpret_cast<const char*>(idx) + 4u * (unsigned)min(j, m_last));
    };
    int key0[NP];
#pragma unroll
    for (int p = 0; p < NP; ++p) {
        const int vw = wave + NW * p;
        key0[p] = 32 * (vw >> 2) + 4 * (vw & 3) + 16 * (g4 & 1) + 2 * hh;
    }
    u32x4 kreg[NP][2], vreg[NP][2];
    // byte offsets of the rows requested next (K and V share them), positions of those after
    unsigned off_k[NP][2], off_v[NP][2];
    int pos_n[NP][2];
#define TF_LOAD_IDX(P, J0)                                                                     \
    _Pragma("unroll") for (int p = 0; p < NP; ++p) {                                           \
        P[p][0] = load_idx((J0) + key0[p]);                                                    \
        P[p][1] = load_idx((J0) + key0[p] + 1);                                                \
    }
#define TF_OFFSETS(F, P)                                                                       \
    _Pragma("unroll") for (int p = 0; p < NP; ++p)                                             \
        _Pragma("unroll") for (int i = 0; i < 2; ++i)                                          \
            F[p][i] = __umul24((unsigned)P[p][i], kv_row_bytes) + 16u * c8
#define TF_LOAD_ROWS(R, BASE, F)                                                               \
    _Pragma("unroll") for (int p = 0; p < NP; ++p)                                             \
        _Pragma("unroll") for (int i = 0; i < 2; ++i)                                          \
            R[p][i] = *reinterpret_cast<const u32x4*>(BASE + F[p][i])
#define TF_STORE_K(STAGE)                                                                      \
    _Pragma("unroll") for (int p = 0; p < NP; ++p) {                                           \
        uint16_t* dst_ = k_wr + (STAGE) * kKTile + (key0[p] - key0[0]) * kKStr;                \
        *reinterpret_cast<u32x4*>(dst_) = kreg[p][0];                                          \
        *reinterpret_cast<u32x4*>(dst_ + kKStr) = kreg[p][1];                                  \
    }
#define TF_STORE_V(STAGE)                                                                      \
    _Pragma("unroll") for (int p = 0; p < NP; ++p)                                             \
        store_v_transposed(vreg[p][0], vreg[p][1], v_lds + (STAGE) * kVTile, v_wr[p])
    uint16_t* const k_wr = k_lds + key0[0] * kKStr + 8 * c8;
    // V^T: row = column of V; the 64 keys of a row are 8 slots of 16 bytes, slot 4 h + g holding the
    // eight keys 32 h + 4 g + {0..3, 16..19} that lane group g feeds to the MFMA of 32-key half h.
    // A row's slots are XOR-ed with (row % 8) ^ (row / 8 % 8): the 16 lanes that LDS serves together in a
    // 16-byte read then touch all 64 banks once (4.7 cycles a read; a padded row of 144 bytes
    // XOR-ed with row / 8 alone: 12.1).  A write's rows are 8 apart, which is one half of the banks: two lanes to
    // a bank, 8.4 cycles; the counted conflicts, a third of LDS's busy cycles, are these writes.
    int v_wr[NP];
#pragma unroll
    for (int p = 0; p < NP; ++p)
        v_wr[p] = (8 * c8 + 4 * hh) * kVStr + 8 * ((wave + NW * p) ^ (c8 & 7) ^ (4 * hh)) + 4 * (g4 & 1);

    // The weights are taken against a reference that stays where the first block of keys put it, the row
    // max of that block, as long as that will do: a running maximum cost 18 vector instructions and a
    // branch per block.  Later scores may exceed it: weights and sums have fp32's range.  Before
    // each inner tile the sums are looked at (their limit is out of the reach of 2^24 weights of at most
    // 1): a row that has outgrown it moves its reference by a power of two that brings its sum back
    // to 1 .. 2, and takes what it has summed along, exactly (keep_range).  Only where scores rise by
    // more than some 70 in natural logarithms within 192 keys is there no sum left to go on from: an
    // item where sums or numerators have overflowed is done again, those rows against their true maxima and
    // the others as before, so that no query's bits depend on later ones.
    // 8 x 32 heads x 2048 kept: level logits 322 us, rising by 136 or late by 23 or 45 302 to 319 (done again
    // as soon as a sum passed 2^40, as it was before: 670 to 735; a lazy running maximum 331 to 353).
    float neg_mc[QB] = {};   // minus the reference of a lane's queries, scaled to base 2
    if (tid == 0) overflow = 0;
    if (exact) {
        // scores only, tile by tile, for the row maxima (the others' over the first block, as above)
        float mx[QB];
        const unsigned lost = lost_rows[wave] >> c16;
        int top[QB];
        bf16x8 qm[QB][4];
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) {
            mx[qb] = kMasked;
            top[qb] = lost >> 16 * qb & 1 ? lim[qb] : min(lim[qb], 31);
#pragma unroll
            for (int s = 0; s < 4; ++s)
                qm[qb][s] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4*>(
                    Qb + (long long)idx[lim[qb]] * d.qs[2] + 32 * s + 8 * g4));
        }
        for (int j0 = 0; j0 <= i_last; j0 += kBN) {
            __syncthreads();
            TF_LOAD_IDX(pos_n, j0);
            TF_OFFSETS(off_k, pos_n);
            TF_LOAD_ROWS(kreg, Kb, off_k);
            TF_STORE_K(0);
            __syncthreads();
#pragma unroll 1
            for (int kb = 0; kb < kBN / 16; ++kb) {
                f32x4 sm[QB] = {};
#pragma unroll
                for (int s = 0; s < 4; ++s) {
                    const bf16x8 km = *reinterpret_cast<const bf16x8*>(k_lds + (16 * kb + c16) * kKStr + 32 * s + 8 * g4);
#pragma unroll
                    for (int qb = 0; qb < QB; ++qb) sm[qb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(km, qm[qb][s], sm[qb], 0, 0, 0);
                }
#pragma unroll
                for (int qb = 0; qb < QB; ++qb)
#pragma unroll
                    for (int v = 0; v < 4; ++v)
                        if (j0 + 16 * kb + 4 * g4 + v <= top[qb]) mx[qb] = fmaxf(mx[qb], sm[qb][v]);
            }
        }
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) {
            mx[qb] = fmaxf(mx[qb], __shfl_xor(mx[qb], 16));
            mx[qb] = fmaxf(mx[qb], __shfl_xor(mx[qb], 32));
            neg_mc[qb] = -mx[qb] * scale_log2;
        }
        __syncthreads();
    }

    // ---- prologue: every index first, then every row load, no wait in between -------------
    int qp[QB];
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) qp[qb] = idx[lim[qb]];
    const int qpos = (lane & 16) ? qp[QB - 1] : qp[0];   // position of query lane % WQ of the wave
    int pos_0[NP][2], pos_1[NP][2];
    TF_LOAD_IDX(pos_0, 0);
    TF_LOAD_IDX(pos_1, kBN);
    TF_LOAD_IDX(pos_n, 2 * kBN);
    // Q fragments (B operand of S^T = K Q^T): for query block qb and k-step s, the 8 elements
    // 32 s + 8 g4 .. +7 of query row iw + 16 qb + c16.
    bf16x8 qf[QB][4];
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
        const uint16_t* src = Qb + (long long)qp[qb] * d.qs[2] + 8 * g4;
#pragma unroll
        for (int s = 0; s < 4; ++s) qf[qb][s] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4*>(src + 32 * s));
    }
    TF_OFFSETS(off_k, pos_0);
    TF_LOAD_ROWS(kreg, Kb, off_k);
    TF_LOAD_ROWS(vreg, Vb, off_k);
    if (!kOwnStage) __syncthreads();   // the rows of the item before are staged where K goes
    TF_STORE_K(0);
    TF_OFFSETS(off_k, pos_1);
    TF_LOAD_ROWS(kreg, Kb, off_k);
    __syncthreads();

    // LDS offsets of this lane's operand fragments inside a K / V^T stage
    const int k_off = c16 * kKStr + 8 * g4;
    int v_off[4];
#pragma unroll
    for (int x4 = 0; x4 < 4; ++x4) v_off[x4] = c16 * kVStr + 8 * (g4 ^ (c16 & 7) ^ (c16 >> 3) ^ (2 * x4));

    const f32x4 zero4f = {0.f, 0.f, 0.f, 0.f};
    f32x4 oacc[8][QB];         // O^T: 16 columns of V x 16 queries
    f32x4 l_acc[QB];           // softmax denominators (row 0), see l_ones
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
        l_acc[qb] = zero4f;
#pragma unroll
        for (int db = 0; db < 8; ++db) oacc[db][qb] = zero4f;
    }
    f32x4 s_x[2][QB], s_y[2][QB];   // raw scores of an even / odd block of 32 keys: [16 keys][16 queries]
    u32x4 p_a[QB], p_b[QB];         // P^T of an even / odd block, per query block
    // A operand whose row 0 sums the weights of each query
    const unsigned one2 = c16 == 0 ? 0x3f803f80u : 0u;
    const bf16x8 l_ones = __builtin_bit_cast(bf16x8, u32x4{one2, one2, one2, one2});

    // fragment i (0..7) of half `half` of a stage: 16 keys i / 4 and k-step i % 4; 16 columns of V
    auto read_k = [&](const uint16_t* ks, int half, int i) -> bf16x8 {
        return *reinterpret_cast<const bf16x8*>(ks + k_off + (32 * half + 16 * (i >> 2)) * kKStr + 32 * (i & 3));
    };
    auto read_v = [&](const uint16_t* vs, int half, int i) -> bf16x8 {
        return *reinterpret_cast<const bf16x8*>(vs + v_off[(2 * half) ^ (i & 3)] + 16 * i * kVStr);
    };
    auto row_max = [&](const f32x4& a, const f32x4& b) -> float {
        float mx = fmaxf(fmaxf(fmaxf(a[0], a[1]), fmaxf(a[2], a[3])), fmaxf(fmaxf(b[0], b[1]), fmaxf(b[2], b[3])));
        // the other keys of this query sit 16, 32 and 48 lanes away
        mx = fmaxf(mx, __shfl_xor(mx, 16));
        return fmaxf(mx, __shfl_xor(mx, 32));
    };
    auto settle_sums = [&]() {
        if constexpr (QB == 2) mfma_settle(l_acc[0], l_acc[QB - 1]);
        else mfma_settle(l_acc[0], oacc[7][0]);
    };
    // Before an inner tile: rows whose weights so far sum to more than kSumLimit.  l_acc's last MFMAs are six
    // chunks back, oacc's are waited for; p_a holds the weights that are not summed yet.  (Asked before a
    // wave's last tiles as well it cost 7 spilled registers and 1 % of 8 x 32 x 4096.)
    auto keep_range = [&]() {
        mfma_result(l_acc[0]);
        if constexpr (QB == 2) mfma_result(l_acc[QB - 1]);
        if (!__any(fmaxf(l_acc[0][0], l_acc[QB - 1][0]) > kSumLimit)) return;
        settle_sums();
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) {
            const float sum = __shfl(l_acc[qb][0], c16);   // row 0 of the accumulator: lanes 0 - 15
            const int up = sum > kSumLimit ? min(__builtin_bit_cast(int, sum) >> 23, 253) - 127 : 0;
            const float down = __builtin_bit_cast(float, (127 - up) << 23);
            neg_mc[qb] -= (float)up;
            l_acc[qb] *= down;
#pragma unroll
            for (int db = 0; db < 8; ++db) {
                mfma_result(oacc[db][qb]);
                oacc[db][qb] *= down;
            }
#pragma unroll
            for (int w = 0; w < 4; ++w)
                p_a[qb][w] = pack_bf16x2(__builtin_bit_cast(float, p_a[qb][w] << 16) * down,
                                         __builtin_bit_cast(float, p_a[qb][w] & 0xffff0000u) * down);
        }
    };
    // Chunk i of a block's weights: query block i / 4, 16 keys (i / 2) % 2, accumulator registers
    // 2 (i % 2) and the next; register v is key J0 + 16 (i / 2 % 2) + 4 g4 + v.
#define TF_MASK(S, I, J0)                                                                      \
    do {                                                                                       \
        const int t_ = (J0) + 16 * (((I) >> 1) & 1) + 2 * ((I) & 1) + 4 * g4 - lim[(I) >> 2];  \
        f32x4& s_ = S[((I) >> 1) & 1][(I) >> 2];                                               \
        if (t_ > 0) s_[2 * ((I) & 1)] = kMasked;                                               \
        if (t_ + 1 > 0) s_[2 * ((I) & 1) + 1] = kMasked;                                       \
    } while (0)
    // One half of an iteration's chunk: fragment i against both query blocks.
#define TF_CHUNK(QK, EX, PV, S_NEW, S_OLD, P_NEW, P_OLD, J_OLD)                                \
    do {                                                                                       \
        const f32x4& s_ = S_OLD[(i >> 1) & 1][i >> 2];                                         \
        float e0_ = 0.f, e1_ = 0.f;                                                            \
        if (EX && (i & 1) == 0) mfma_result(S_OLD[(i >> 1) & 1][i >> 2]);                      \
        if (EX == 2) TF_MASK(S_OLD, i, J_OLD);                                                 \
        if (QK && (i & 3) == 0) mfma_first(S_NEW[i >> 2][0], kf[r], qf[0][0]);                 \
        if (QK && (i & 3) != 0) mfma_add(S_NEW[i >> 2][0], kf[r], qf[0][i & 3]);               \
        __builtin_amdgcn_sched_barrier(0);                                                     \
        if (EX) {                                                                              \
            e0_ = __builtin_amdgcn_exp2f(fmaf(s_[2 * (i & 1)], scale_log2, neg_mc[i >> 2]));   \
            e1_ = fmaf(s_[2 * (i & 1) + 1], scale_log2, neg_mc[i >> 2]);                       \
        }                                                                                      \
        if (PV) mfma_add(oacc[i][0], vf[r], __builtin_bit_cast(bf16x8, P_OLD[0]));             \
        __builtin_amdgcn_sched_barrier(0);                                                     \
        if (EX) e1_ = __builtin_amdgcn_exp2f(e1_);                                             \
        if (QK && (i & 3) == 0) mfma_first(S_NEW[i >> 2][1], kf[r], qf[1][0]);                 \
        if (QK && (i & 3) != 0) mfma_add(S_NEW[i >> 2][1], kf[r], qf[1][i & 3]);               \
        __builtin_amdgcn_sched_barrier(0);                                                     \
        if (EX) P_NEW[i >> 2][i & 3] = pack_bf16x2(e0_, e1_);                                  \
        if (PV) mfma_add(oacc[i][1], vf[r], __builtin_bit_cast(bf16x8, P_OLD[1]));             \
        if (PV && i < 2) mfma_add(l_acc[i], l_ones, __builtin_bit_cast(bf16x8, P_OLD[i]));     \
    } while (0)
    // The same where a wave has one query block: 16 keys i / 4, accumulator register i % 4.
#define TF_MASK1(S, I, J0)                                                                     \
    do {                                                                                       \
        if ((J0) + 16 * ((I) >> 2) + ((I) & 3) + 4 * g4 > lim[0]) S[(I) >> 2][0][(I) & 3] = kMasked; \
    } while (0)
#define TF_CHUNK1(QK, EX, PV, S_NEW, S_OLD, P_NEW, P_OLD, J_OLD)                               \
    do {                                                                                       \
        if (EX && (i & 3) == 0) mfma_result(S_OLD[i >> 2][0]);                                 \
        if (EX == 2) TF_MASK1(S_OLD, i, J_OLD);                                                \
        if (QK && (i & 3) == 0) mfma_first(S_NEW[i >> 2][0], kf[r], qf[0][0]);                 \
        if (QK && (i & 3) != 0) mfma_add(S_NEW[i >> 2][0], kf[r], qf[0][i & 3]);               \
        __builtin_amdgcn_sched_barrier(0);                                                     \
        if (EX) e_[i & 1] = __builtin_amdgcn_exp2f(fmaf(S_OLD[i >> 2][0][i & 3], scale_log2, neg_mc[0])); \
        if (PV) mfma_add(oacc[i][0], vf[r], __builtin_bit_cast(bf16x8, P_OLD[0]));             \
        if (PV && i == 0) mfma_add(l_acc[0], l_ones, __builtin_bit_cast(bf16x8, P_OLD[0]));    \
        __builtin_amdgcn_sched_barrier(0);                                                     \
        if (EX && (i & 1)) P_NEW[0][i >> 1] = pack_bf16x2(e_[0], e_[1]);                       \
    } while (0)
    // One iteration of the tile loop over two blocks of 32 keys (halves A and B of 8 chunks each); QK,
    // EX (1: weights, 2: with the causal mask) and PV say at compile time what a half has to do.
    // A chunk is two MFMAs of the scores, two weights and two MFMAs of the product; nothing moves
    // across chunk borders, so the two pipes always have each other's work next to theirs, and
    // operand fragments are read from LDS kRing - 1 chunks ahead.
#define TF_TILE(QK_A, EX_A, PV_A, QK_B, EX_B, PV_B, FIRST, MORE)                               \
    do {                                                                                       \
        bf16x8 kf[kRing], vf[kRing];                                                           \
        float e_[2] = {0.f, 0.f};                                                              \
        (void)e_;                                                                              \
        _Pragma("unroll") for (int j = 0; j < kRing - 1; ++j) {                                \
            if (QK_A) kf[j] = read_k(ks, 0, j);                                                \
            if (PV_A) vf[j] = read_v(vs, 0, j);                                                \
        }                                                                                      \
        __builtin_amdgcn_sched_barrier(0);                                                     \
        _Pragma("unroll") for (int j = 0; j < 16; ++j) {                                       \
            const int i = j & 7, n = j + kRing - 1, r = j % kRing;                             \
            if (n < 16 && (n < 8 ? QK_A : QK_B)) kf[n % kRing] = read_k(ks, n >> 3, n & 7);    \
            if (n < 16 && (n < 8 ? PV_A : PV_B)) vf[n % kRing] = read_v(vs, n >> 3, n & 7);    \
            if constexpr (QB == 2) {                                                           \
                if (j < 8) TF_CHUNK(QK_A, EX_A, PV_A, s_x, s_y, p_b, p_a, 64 * kt - 32);       \
                else TF_CHUNK(QK_B, EX_B, PV_B, s_y, s_x, p_a, p_b, 64 * kt);                  \
            } else {                                                                           \
                if (j < 8) TF_CHUNK1(QK_A, EX_A, PV_A, s_x, s_y, p_b, p_a, 64 * kt - 32);      \
                else TF_CHUNK1(QK_B, EX_B, PV_B, s_y, s_x, p_a, p_b, 64 * kt);                 \
            }                                                                                  \
            __builtin_amdgcn_sched_barrier(0);                                                 \
            if (j == 7) {                                                                      \
                if (FIRST) {                                                                   \
                    mfma_settle(s_x[0][0], s_x[1][0]);                                         \
                    if constexpr (QB == 2) {                                                   \
                        mfma_result(s_x[0][QB - 1]);                                           \
                        mfma_result(s_x[1][QB - 1]);                                           \
                        _Pragma("unroll") for (int v = 0; v < 8; ++v) TF_MASK(s_x, v, 0);      \
                    } else {                                                                   \
                        _Pragma("unroll") for (int v = 0; v < 8; ++v) TF_MASK1(s_x, v, 0);     \
                    }                                                                          \
                    if (!exact) {                                                              \
                        _Pragma("unroll") for (int qb = 0; qb < QB; ++qb)                       \
                            neg_mc[qb] = -row_max(s_x[0][qb], s_x[1][qb]) * scale_log2;            \
                    }                                                                          \
                }                                                                              \
            }                                                                                  \
            if (j == 11) TF_DELIVER_K(MORE);                                                   \
            if (j == 13) TF_DELIVER_V(MORE);                                                   \
        }                                                                                      \
    } while (0)

    // Iteration kt: scores of the two blocks of K tile kt, weights of blocks 2 kt - 1 and 2 kt, products of
    // blocks 2 kt - 2 and 2 kt - 1 with V tile kt - 1.  It writes K(kt + 1) and V(kt) to the stages that K(kt
    // - 1) and V(kt - 2) have left; iteration n_kt only finishes.  A wave runs n_kt + 1 iterations with a
    // barrier after each but the last, whatever it has to compute in them.  Delivering K(kt + 1) requests
    // K(kt + 2) into the same registers, V(kt) likewise V(kt + 1), with off_k and off_v; the positions of the
    // tile after (pos_n) are requested before the rows, because loads return in order and positions behind a
    // row that misses the L2 would hold up the next request.
#define TF_DELIVER_K(MORE)                                                                     \
    do {                                                                                       \
        if (MORE) {                                                                            \
            TF_STORE_K((kt & 1) ^ 1);                                                          \
            _Pragma("unroll") for (int p = 0; p < NP; ++p)                                     \
                _Pragma("unroll") for (int i = 0; i < 2; ++i) off_v[p][i] = off_k[p][i];       \
            TF_OFFSETS(off_k, pos_n);                                                          \
            TF_LOAD_IDX(pos_n, (kt + 3) * kBN);                                                \
            TF_LOAD_ROWS(kreg, Kb, off_k);                                                     \
        }                                                                                      \
    } while (0)
#define TF_DELIVER_V(MORE)                                                                     \
    do {                                                                                       \
        if (MORE) {                                                                            \
            TF_STORE_V(kt & 1);                                                                \
            TF_LOAD_ROWS(vreg, Vb, off_v);                                                     \
        }                                                                                      \
    } while (0)
#define TF_ADVANCE()                                                                           \
    do {                                                                                       \
        ++kt;                                                                                  \
        ks = k_lds + (kt & 1) * kKTile;                                                        \
        vs = v_lds + ((kt & 1) ^ 1) * kVTile;                                                  \
        __syncthreads();                                                                       \
    } while (0)
    int kt = 0;
    const uint16_t* ks = k_lds;
    const uint16_t* vs = v_lds + kVTile;
    TF_TILE(true, 0, false, true, 1, false, true, true);
    TF_ADVANCE();
    while (kt < q_last) {
        keep_range();
        TF_TILE(true, 1, true, true, 1, true, false, true);
        TF_ADVANCE();
    }
    // the wave's last tile, whose two blocks are masked
    if (q_last > 0) {
        TF_TILE(true, 1, true, true, 2, true, false, true);
        TF_ADVANCE();
    }
    TF_TILE(false, 2, true, false, 0, true, false, kt < n_kt);
    if (kt < n_kt) TF_ADVANCE();
    else ++kt;
    // nothing left to compute: only the tiles of the others
    while (kt < n_kt) {
        TF_DELIVER_K(true);
        TF_DELIVER_V(true);
        TF_ADVANCE();
    }
#undef TF_ADVANCE
#undef TF_DELIVER_V
#undef TF_DELIVER_K
#undef TF_TILE
#undef TF_CHUNK
#undef TF_MASK
#undef TF_CHUNK1
#undef TF_MASK1
#undef TF_STORE_V
#undef TF_STORE_K
#undef TF_LOAD_ROWS
#undef TF_OFFSETS
#undef TF_LOAD_IDX

    // (the output accumulators are first read in products with the reciprocals of these)
    settle_sums();
    unsigned lost = 0;
    if (!exact && __any(fmaxf(l_acc[0][0], l_acc[QB - 1][0]) > kSumLimit)) {
        // queries that have outgrown their reference and have an infinity or no number among their results
        auto gone = [](float x) { return (__builtin_bit_cast(unsigned, x) & 0x7f800000u) == 0x7f800000u; };
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) {
            const bool above = __shfl(l_acc[qb][0], c16) > kSumLimit;
            bool any = lane < 16 && gone(l_acc[qb][0]);
#pragma unroll
            for (int i = 0; i < 8; ++i)
#pragma unroll
                for (int e = 0; e < 4; ++e) any = any || gone(oacc[i][qb][e]);
            any = any && above;
            // (the other columns of this query are 16, 32 and 48 lanes away)
            const unsigned long long b = __ballot(any);
            lost |= (unsigned)((b | b >> 16 | b >> 32 | b >> 48) & 0xffff) << 16 * qb;
        }
        if (lost && lane == 0) overflow = 1;
    }
    __syncthreads();
    if (!exact && __builtin_amdgcn_readfirstlane(overflow)) {
        __syncthreads();   // everybody has read the flag before the item's second start clears it
        if (lane == 0) lost_rows[wave] = lost;
        exact = true;
        --it;
        continue;
    }
    exact = false;
    // normalise, transpose through LDS and write whole rows
    // (the lane number goes through an opaque move so that the addresses below are formed
    // here, per item, instead of being carried in registers across the tile loop)
    int ln = lane;
    asm volatile("" : "+v"(ln));
    uint16_t* os = ostage + wave * (WQ * kOStr);  // [WQ queries][kOStr], this wave's alone
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
        const float l_tot = __shfl(l_acc[qb][0], ln & 15);
        const float inv = l_tot > 0.f ? 1.0f / l_tot : 0.f;
#pragma unroll
        for (int db = 0; db < 8; ++db) {
            bf16x4 o4;
#pragma unroll
            for (int e = 0; e < 4; ++e) o4[e] = (__bf16)(oacc[db][qb][e] * inv);
            *reinterpret_cast<bf16x4*>(os + (16 * qb + (ln & 15)) * kOStr + 16 * db + 4 * (ln >> 4)) = o4;
        }
    }
    // the rows are read back by other lanes of this wave only: LDS operations of one wave
    // complete in order, the compiler must just not move them across this point
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    // Every 16-lane group writes one query's row: four rows per store instruction.
    const uint4 zero4 = make_uint4(0, 0, 0, 0);
    uint16_t* const Oc = Ob + 8 * (ln & 15);  // this lane's 16-byte column
#pragma unroll
        for (int it = 0; it < WQ / 4; ++it) {
            const int r = 4 * it + (ln >> 4);  // query row of the wave
            const int p = __shfl(qpos, r);    // its position, held by lane r
            if (iw + r < m) {
                const uint4 v = *reinterpret_cast<const uint4*>(os + r * kOStr + 8 * (ln & 15));
                store_streaming(Oc + (long long)p * d.os[2], v);
            }
        }
    // The zero rows this wave owns: the filtered positions after its first query and before the
    // first query of the next wave (n after the last kept token).  They are written densely, four
    // rows per store instruction whatever the gaps look like: with z_i = the zero rows before
    // query i (= position_i - position_0 - i, ascending), the k-th zero row sits at
    // position_0 + 1 + k + #{i >= 1 : z_i <= k}, and the count is a ballot over the queries.
    // All output stores are non-temporal: O is written once and never read here, and lines of O
    // allocated in the L2 push out K / V tiles that other query tiles of the group still need.
    {
        const int n_valid = min(max(m - iw, 0), WQ);  // queries of this wave that exist
        if (n_valid > 0) {
            const int p_first = __builtin_amdgcn_readfirstlane(qpos);
            const int last_rank = iw + n_valid - 1;
            const int p_end = last_rank < m_last ? idx[last_rank + 1] : d.n;  // uniform
            const int n_zero = __builtin_amdgcn_readfirstlane(p_end - p_first - n_valid);
            const int z_mine = qpos - p_first - ln;  // meaningful for lanes 1 .. n_valid - 1
            const bool counted = ln >= 1 && ln < n_valid;
            const int grp = ln >> 4;
            for (int k0 = 0; k0 < n_zero; k0 += 4) {
                const int c0 = __popcll(__ballot(counted && z_mine <= k0));
                const int c1 = __popcll(__ballot(counted && z_mine <= k0 + 1));
                const int c2 = __popcll(__ballot(counted && z_mine <= k0 + 2));
                const int c3 = __popcll(__ballot(counted && z_mine <= k0 + 3));
                const int cnt = grp == 0 ? c0 : (grp == 1 ? c1 : (grp == 2 ? c2 : c3));
                const int k = k0 + grp;
                if (k < n_zero)
                    store_streaming(Oc + (long long)(p_first + 1 + k + cnt) * d.os[2], zero4);
            }
        }
    }
    // positions before the first kept token
    if (qt == 0 && blk == 0) {
        const int ze = __shfl(qpos, 0);
        for (int g = ln >> 4; g < ze; g += 4) *reinterpret_cast<uint4*>(Oc + (long long)g * d.os[2]) = zero4;
    }
    // (no barrier here: after the one behind the tile loop nobody reads a tile stage; the staging area is not
    // shared, or, over the K tiles, protected by the barrier before the next item's first K tile)
    }  // items
}

}  // namespace
}  // namespace tf
