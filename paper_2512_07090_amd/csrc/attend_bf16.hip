// Causal softmax attention over the kept tokens, bf16 inputs (Section 3.2: the tokens that
// are not skipped attend as usual and a skipped token's attention output is zero; here both
// queries and keys are the kept tokens, addressed through kept_idx, so "causal" means key rank
// <= query rank in the compacted order).
//
// Flash-style kernel for gfx950.  One work item covers 256 kept queries: eight waves of 32, two
// per SIMD with 256 registers each.  It walks the key tiles (64 kept keys) once, K and V rows
// gathered through kept_idx into LDS (two stages each).
//   S^T = K Q^T   v_mfma_f32_32x32x16_bf16, A = K rows from LDS, B = Q fragments held in
//                 registers for the whole item.  The transposed product puts one query per
//                 lane column, so P^T goes from the accumulators to the next product's operand
//                 without leaving the lane.
//   O^T += V^T P^T  A = V^T from LDS, written there already transposed (a pair of lanes swaps halves
//                 and permutes 16-bit words), so that a fragment is one 16-byte read: the
//                 transposing LDS read moves half as much per instruction.  The contraction
//                 order over keys is permuted the same way for both operands (accumulator
//                 register v of a 32-key block is key 8 (v / 4) + 4 (lane / 32) + v % 4).
//   softmax       fp32, base 2 (scale * log2 e folded into one FMA per score), against a reference
//                 that moves only when a weight outgrows it (TF_RESCUE): no row maximum on the
//                 way.  The denominators are summed on the matrix pipe from the weights as
//                 rounded (l_ones), so every output row is an exact convex combination of value
//                 rows; v_dot2_f32_bf16, which did it before, occupies that pipe for about 20
//                 cycles each (0.66 against 0.60 us per 64 keys in a copy of the loop).
//   pipeline      Scores run one 32-key block ahead of the weights and the product with V one block
//                 behind them, so that in a block the 8 + 8 MFMAs, the 16 exponentials and the 16
//                 LDS reads do not depend on each other; they are interleaved chunk by chunk in
//                 program order.  The blocks that begin and end a wave's walk are instances of
//                 the same body with parts left out.
//   tile loads    A tile's rows are requested right after the registers they land in have been
//                 written to LDS, a whole iteration ahead of their use, and land in one register
//                 set (requested at the start of the iteration that delivers them the launch took
//                 0.299 instead of 0.282 ms at 8 x 32 heads x 2048 kept on all-zero inputs).
//   zero rows     The rows of the filtered positions between a query and the next kept token
//                 are written as zeros together with the query's row (kept_idx is ascending).
//   scheduling    One persistent workgroup per CU walks a static list of pairs of query tiles
//                 (tile p with tile n_qt - 1 - p: equal causal work); see the kernel.
// What bounds it: with real data the card runs at its power limit (1.4 kW) and clocks down; a
// library GEMM of 8192^3 reaches 1.2-1.36 PFLOP/s there, this kernel 1.1 at 16384 kept tokens.
// 8 x 32 heads x 2048 kept: 0.356 -> 0.346 ms (all-zero inputs, no power limit: 0.301 -> 0.282);
// 32 heads on 8 KV heads x 16384 kept: 2.06 -> 1.98 ms (1.72 -> 1.52).
#include "tf_kernels.h"
#include <algorithm>

namespace tf {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));

constexpr int kBN = 64;                  // kept keys per tile
constexpr int kKStr = kHeadDim + 8;      // K tile row stride, elements (272 B)
constexpr int kVStr = kBN + 8;           // V^T tile row stride (one row per column of V), elements (144 B)
constexpr int kKTile = kBN * kKStr;      // elements per K tile
constexpr int kVTile = kHeadDim * kVStr; // elements per V^T tile
constexpr int kOStr = kHeadDim + 8;      // output staging row stride, elements
constexpr float kRefBits = 16.f;         // headroom of the softmax reference, in powers of two
constexpr float kMasked = -1e30f;

// One 16-byte chunk of the row at position `pos`: `base` is uniform over the workgroup (the
// (batch, head) slice plus nothing else), the lane's part is a 32-bit byte offset
// pos * row_bytes + col_bytes formed by one 24-bit multiply-add (the launcher checks that a
// slice spans less than 4 GiB and that positions and row strides stay below 2^24).
__device__ __forceinline__ u32x4 load16(const char* base, int pos, unsigned row_bytes, unsigned col_bytes)
{
    const unsigned off = __umul24((unsigned)pos, row_bytes) + col_bytes;
    return *reinterpret_cast<const u32x4*>(base + off);
}
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
__device__ __forceinline__ void store_v_transposed(u32x4 r0, u32x4 r1, uint16_t* dst)
{
#pragma unroll
    for (int w = 0; w < 2; ++w) {
        const auto s0 = __builtin_amdgcn_permlane32_swap(r0[w], r0[w + 2], false, false);
        const auto s1 = __builtin_amdgcn_permlane32_swap(r1[w], r1[w + 2], false, false);
        // words of two columns: keys k, k + 1, k + 2, k + 3
        const unsigned k0 = s0[0], k2 = s0[1], k1 = s1[0], k3 = s1[1];
        const u32x2 even = {__builtin_amdgcn_perm(k1, k0, 0x05040100u), __builtin_amdgcn_perm(k3, k2, 0x05040100u)};
        const u32x2 odd = {__builtin_amdgcn_perm(k1, k0, 0x07060302u), __builtin_amdgcn_perm(k3, k2, 0x07060302u)};
        *reinterpret_cast<u32x2*>(dst + (2 * w) * kVStr) = even;
        *reinterpret_cast<u32x2*>(dst + (2 * w + 1) * kVStr) = odd;
    }
}

template <int NW>
__global__ __launch_bounds__(64 * NW, 2) void attend_bf16_kernel(
    Dims d, float scale_log2, int n_qt, int n_xcd, const uint16_t* __restrict__ Q,
    const uint16_t* __restrict__ K, const uint16_t* __restrict__ V,
    const int32_t* __restrict__ kept_idx, uint16_t* __restrict__ O,
    const int32_t* __restrict__ counts, long long idx_stride)
{
    constexpr int NT = 64 * NW;    // threads
    constexpr int NP = 8 / NW;     // passes of the workgroup over a tile when loading it
    constexpr int WQ = 32;         // queries per wave
    constexpr int kBM = WQ * NW;   // kept queries per work item
    constexpr int kRing = 3;       // operand fragments in flight from LDS, per tensor
    __shared__ __attribute__((aligned(16))) uint16_t smem[2 * kKTile + 2 * kVTile];
    uint16_t* const k_lds = smem;               // 2 stages of K
    uint16_t* const v_lds = smem + 2 * kKTile;  // 2 stages of V^T
    // Output staging of its own (141 KB of LDS in all): a wave stages and writes its rows without
    // a workgroup barrier on either side, so the waves leave an item, and start on the next
    // item's first loads, as each gets there.
    __shared__ __attribute__((aligned(16))) uint16_t ostage[kBM * kOStr];

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
    // Static schedule: workgroup j of XCD x (x = id % n_xcd, as the dispatcher deals them) walks
    // entries j, j + W, ... of the XCD's list of (group, pair of query tiles); a pair joins
    // query tile p with n_qt - 1 - p, so every entry is the same amount of causal work, and the
    // workgroups that share a group start on it together and stream the same K / V tiles.
    const int x = blockIdx.x % n_xcd, j = blockIdx.x / n_xcd;
    const int nwx = (gridDim.x + n_xcd - 1 - x) / n_xcd;  // workgroups whose id % n_xcd is x
    const int g_lo = x * n_groups / n_xcd;
    const int ng = (x + 1) * n_groups / n_xcd - g_lo;
    const int n_pairs = (n_qt + 1) >> 1;
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
    const bool split_rest = !counts && rest > 0 && 2 * rest <= nwx && rest <= ng && n_pairs >= 2 && (n_qt & 1) == 0;
    const int n_main = split_rest ? n_entries - rest : n_entries;  // entries dealt as pairs
    const int whole_groups = split_rest ? ng - rest : ng;          // groups that keep all their pairs
    int rb = g_lo / d.Hq, row_e0 = 0;
    for (int it = 0;; ++it) {
    const int e = j + (it >> 1) * nwx;
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
            P = m == 0 ? 1 : (nq + 1) >> 1;
            if (e < row_e0 + (hi - lo) * P) break;
            row_e0 += (hi - lo) * P;
            ++rb;
        }
        if (done) break;
        const int el = e - row_e0;
        bh = max(g_lo, rb * d.Hq) + el / P;
        pr = el % P;
    } else {
        m = d.m;
        nq = n_qt;
        if (e < n_main) {
            const int e_whole = whole_groups * n_pairs;  // entries of the groups with all pairs
            if (e < e_whole) {
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
        if (pr == 0 && !(it & 1)) {
            uint16_t* Oz = O + (long long)b * d.os[0] + (long long)hq * d.os[1] + 8 * (tid & 15);
            for (int g = tid >> 4; g < d.n; g += NT / 16)
                *reinterpret_cast<uint4*>(Oz + (long long)g * d.os[2]) = make_uint4(0, 0, 0, 0);
        }
        continue;
    }
    if (pr >= (nq + 1) >> 1) continue;
    const int qt = single ? ((j & 1) ? pr : nq - 1 - pr) : ((it & 1) ? pr : nq - 1 - pr);
    if (!single && (it & 1) && pr == nq - 1 - pr) continue;  // the middle tile of an odd count is alone

    const int32_t* idx = kept_idx + (long long)b * idx_stride;
    const uint16_t* Qb = Q + (long long)b * d.qs[0] + (long long)hq * d.qs[1];
    const char* Kb = reinterpret_cast<const char*>(K + (long long)b * d.kvs[0] + (long long)hk * d.kvs[1]);
    const char* Vb = reinterpret_cast<const char*>(V + (long long)b * d.kvs[0] + (long long)hk * d.kvs[1]);
    uint16_t* Ob = O + (long long)b * d.os[0] + (long long)hq * d.os[1];
    const unsigned kv_row_bytes = (unsigned)d.kvs[2] * 2u;

    const int col = lane & 31, hh = lane >> 5;

    const int i0 = qt * kBM;
    // Waves w and w + NW / 2 share a SIMD.  Causal work grows with the row block, so the
    // second half of the waves takes the row blocks in reverse: every SIMD then carries one
    // early and one late block and the four SIMDs finish together.
    const int blk = wave < NW / 2 ? wave : NW + NW / 2 - 1 - wave;
    const int iw = i0 + WQ * blk;    // first query rank of this wave
    const int i_last = min(i0 + kBM, m) - 1;
    const int n_kt = i_last / kBN + 1;
    const int m_last = m - 1;
    const int lim = min(iw + col, m_last);        // last key rank this lane's query may see
    const int h_diag = iw > m_last ? -1 : iw / 32;  // the wave's last block of 32 keys, the masked one

    // tile-load roles: in pass p a thread moves columns 8 c .. + 7 of two neighbouring keys; the
    // lane 32 further holds the two keys after them, so that a pair of lanes can transpose four
    // keys of V, and the waves' keys are dealt so that a wave fills 16-byte slots of V^T.
    // Rows past the last kept token re-read the last kept row: finite values that the mask turns
    // into zero weights, so the loads need no branch.
    const int c8 = lane & 15;
    // A operand that sums the weights of each query on the matrix pipe: the 64 lanes of a P^T operand
    // read as the B operand of a 16x16x32 MFMA are 16 columns x four groups of 8 keys, queries q
    // and q + 16 sharing column q; row 0 adds groups 0 and 2 (query q), row 1 groups 1 and 3.
    const unsigned one2 = (lane & 15) == ((lane >> 4) & 1) ? 0x3f803f80u : 0u;
    const bf16x8 l_ones = __builtin_bit_cast(bf16x8, u32x4{one2, one2, one2, one2});
    int key0[NP];
#pragma unroll
    for (int p = 0; p < NP; ++p) {
        const int vw = wave + NW * p;
        key0[p] = 16 * (vw >> 1) + 4 * (vw & 1) + 8 * ((lane >> 4) & 1) + 2 * hh;
    }
    u32x4 kreg[NP][2], vreg[NP][2];
    int pos_k[NP][2], pos_v[NP][2], pos_n[NP][2];
#define TF_LOAD_IDX(P, J0)                                                                     \
    _Pragma("unroll") for (int p = 0; p < NP; ++p) {                                           \
        P[p][0] = idx[min((J0) + key0[p], m_last)];                                            \
        P[p][1] = idx[min((J0) + key0[p] + 1, m_last)];                                        \
    }
#define TF_LOAD_ROWS(R, BASE, P)                                                               \
    _Pragma("unroll") for (int p = 0; p < NP; ++p) {                                           \
        R[p][0] = load16(BASE, P[p][0], kv_row_bytes, 16u * c8);                               \
        R[p][1] = load16(BASE, P[p][1], kv_row_bytes, 16u * c8);                               \
    }
#define TF_STORE_K(STAGE)                                                                      \
    _Pragma("unroll") for (int p = 0; p < NP; ++p) {                                           \
        uint16_t* dst_ = k_wr + (STAGE) * kKTile + (key0[p] - key0[0]) * kKStr;                \
        *reinterpret_cast<u32x4*>(dst_) = kreg[p][0];                                          \
        *reinterpret_cast<u32x4*>(dst_ + kKStr) = kreg[p][1];                                  \
    }
#define TF_STORE_V(STAGE)                                                                      \
    _Pragma("unroll") for (int p = 0; p < NP; ++p)                                             \
        store_v_transposed(vreg[p][0], vreg[p][1], v_lds + (STAGE) * kVTile + v_wr[p])
    uint16_t* const k_wr = k_lds + key0[0] * kKStr + 8 * c8;
    // V^T: row = column of V; the 64 keys of a row are 8 slots of 16 bytes, slot 2 ks + hh holding the
    // eight keys 16 ks + 4 hh + {0..3, 8..11} that lane half hh feeds to the MFMA of k-step ks.
    // Slots are XOR-ed with the row's number / 8: eight consecutive rows (a read) start at different
    // banks through the row stride, rows 8 apart (a write) through the XOR.
    int v_wr[NP];
#pragma unroll
    for (int p = 0; p < NP; ++p) {
        const int vw = wave + NW * p;
        v_wr[p] = (8 * c8 + 4 * hh) * kVStr + 8 * ((2 * (vw >> 1) + (vw & 1)) ^ (c8 & 7)) + 4 * ((lane >> 4) & 1);
    }

    // ---- prologue: every index first, then every row load, no wait in between -------------
    const int qpos = idx[lim];   // position of this lane's query
    int pos_0[NP][2];
    TF_LOAD_IDX(pos_0, 0);
    TF_LOAD_IDX(pos_v, kBN);
    TF_LOAD_IDX(pos_k, 2 * kBN);
    // Q fragments (B operand of S^T = K Q^T): lane (col, hh) holds, for k-step s, the 8 elements
    // 16 s + 8 hh .. +7 of query row iw + col.
    bf16x8 qf[8];
    {
        const uint16_t* src = Qb + (long long)qpos * d.qs[2];
#pragma unroll
        for (int s = 0; s < 8; ++s)
            qf[s] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4*>(src + 16 * s + 8 * hh));
    }
    TF_LOAD_ROWS(kreg, Kb, pos_0);
    TF_LOAD_ROWS(vreg, Vb, pos_0);
    TF_STORE_K(0);
    TF_LOAD_ROWS(kreg, Kb, pos_v);
    __syncthreads();

    // LDS offsets of this lane's operand fragments inside a K / V^T stage
    const int k_off = col * kKStr + 8 * hh;
    const int v_off0 = col * kVStr + 8 * (hh ^ (col >> 3));
    const int v_off1 = col * kVStr + 8 * ((2 + hh) ^ (col >> 3));

    f32x16 oacc[4];
#pragma unroll
    for (int dt = 0; dt < 4; ++dt)
#pragma unroll
        for (int v = 0; v < 16; ++v) oacc[dt][v] = 0.f;
    f32x4 l_acc = {0.f, 0.f, 0.f, 0.f};  // softmax denominators, see l_ones
    float neg_mc = 0.f;                  // minus the softmax reference, scaled to base 2
    const f32x16 zero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    f32x16 s_x = zero16, s_y = zero16;   // raw scores of an even / odd block of 32 keys
    u32x4 p_a[2], p_b[2];                // P^T of an even / odd block, per 16-key k-step

    // fragment i (0..7) of half `half` of a stage
    auto read_k = [&](const uint16_t* ks, int half, int i) -> bf16x8 {
        return *reinterpret_cast<const bf16x8*>(ks + k_off + half * (32 * kKStr) + 16 * i);
    };
    auto read_v = [&](const uint16_t* vs, int half, int i) -> bf16x8 {
        const int ks2 = i >> 2, dt = i & 3;   // k-step 2 half + ks2 of the tile, 32 columns
        return *reinterpret_cast<const bf16x8*>(vs + (ks2 ? v_off1 : v_off0) + 32 * dt * kVStr + 32 * (half ^ (dt & 1)));
    };
    auto row_max = [&](const f32x16& s) -> float {
        float mx = fmaxf(s[0], s[1]), my = fmaxf(s[2], s[3]);
#pragma unroll
        for (int v = 4; v < 16; v += 4) {
            mx = fmaxf(fmaxf(mx, s[v]), s[v + 1]);
            my = fmaxf(fmaxf(my, s[v + 2]), s[v + 3]);
        }
        mx = fmaxf(mx, my);
        // the other half of this query's keys sits 32 lanes away: swap halves in the VALU
        const FloatPair sw = swap32(mx, mx);
        return fmaxf(sw.first, sw.second);
    };
    // causal mask of accumulator registers 2 i, 2 i + 1 of the block that starts at key rank J0:
    // register v is key J0 + 8 (v / 4) + 4 hh + v % 4
#define TF_MASK(S, I, J0)                                                                      \
    do {                                                                                       \
        const int t_ = (J0) + 4 * hh - lim + 8 * ((I) >> 1) + ((2 * (I)) & 3);                 \
        if (t_ > 0) S[2 * (I)] = kMasked;                                                      \
        if (t_ + 1 > 0) S[2 * (I) + 1] = kMasked;                                              \
    } while (0)
    // weights of accumulator registers 2 i, 2 i + 1, rounded and packed; their bits to ANY
#define TF_WEIGHTS(S, P, I, ANY)                                                               \
    do {                                                                                       \
        const float e0_ = __builtin_amdgcn_exp2f(fmaf(S[2 * (I)], scale_log2, neg_mc));        \
        const float e1_ = __builtin_amdgcn_exp2f(fmaf(S[2 * (I) + 1], scale_log2, neg_mc));    \
        const unsigned w_ = pack_bf16x2(e0_, e1_);                                             \
        P[(I) >> 2][(I) & 3] = w_;                                                             \
        if (((I) & 1) == 0) w_even = w_; else ANY |= w_ | w_even;                              \
    } while (0)
    // The weights of a block are taken against a reference that only moves when it has to: the row
    // max of the first block plus kRefBits, until a weight reaches 2 (a weight that overflowed
    // included): a score more than kRefBits + 1 bits above the reference's max.  Then that
    // query's reference becomes this block's max, what has been accumulated is rescaled and the
    // block's weights are taken again.  Nothing is lost on the way: the sums stay far inside
    // fp32's range, and the test is an OR over the packed weights instead of a row maximum per
    // block (18 fewer vector instructions on the way from the scores to the weights).
#define TF_RESCUE(S, P, ANY)                                                                   \
    do {                                                                                       \
        if (__any(ANY & 0x40004000u)) {                                                        \
            const bool move_ = ((ANY | (unsigned)__shfl_xor((int)(ANY), 32)) & 0x40004000u) != 0; \
            const float new_mc_ = move_ ? -row_max(S) * scale_log2 - kRefBits : neg_mc;        \
            const float corr_ = __builtin_amdgcn_exp2f(new_mc_ - neg_mc);                      \
            neg_mc = new_mc_;                                                                  \
            l_acc[0] *= corr_;                                                                 \
            l_acc[1] *= __shfl(corr_, (lane & 15) + 16);                                       \
            _Pragma("unroll") for (int dt = 0; dt < 4; ++dt)                                   \
                _Pragma("unroll") for (int v = 0; v < 16; ++v) oacc[dt][v] *= corr_;           \
            _Pragma("unroll") for (int i = 0; i < 8; ++i) TF_WEIGHTS(S, P, i, ANY);            \
        }                                                                                      \
        ANY = 0;                                                                               \
    } while (0)
    // One iteration of the tile loop over two blocks of 32 keys (halves A and B of 8 chunks each); QK,
    // EX (1: weights, 2: with the causal mask) and PV say at compile time what a half has to do.
    // A chunk is one MFMA of the scores, two weights and one MFMA of the product; nothing moves
    // across chunk borders, so the two pipes always have each other's work next to theirs, and
    // operand fragments are read from LDS kRing - 1 chunks ahead.
#define TF_TILE(QK_A, EX_A, PV_A, QK_B, EX_B, PV_B, FIRST, MORE)                                   \
    do {                                                                                       \
        bf16x8 kf[kRing], vf[kRing];                                                           \
        unsigned any = 0, w_even = 0;                                                          \
        _Pragma("unroll") for (int j = 0; j < kRing - 1; ++j) {                                \
            if (QK_A) kf[j] = read_k(ks, 0, j);                                                \
            if (PV_A) vf[j] = read_v(vs, 0, j);                                                \
        }                                                                                      \
        TF_REQUEST(MORE);                                                                      \
        __builtin_amdgcn_sched_barrier(0);                                                     \
        _Pragma("unroll") for (int j = 0; j < 16; ++j) {                                       \
            const int i = j & 7, n = j + kRing - 1, r = j % kRing;                             \
            if (n < 16 && (n < 8 ? QK_A : QK_B)) kf[n % kRing] = read_k(ks, n >> 3, n & 7);    \
            if (n < 16 && (n < 8 ? PV_A : PV_B)) vf[n % kRing] = read_v(vs, n >> 3, n & 7);    \
            if (j < 8) {                                                                       \
                if (QK_A) s_x = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[r], qf[i], i ? s_x : zero16, 0, 0, 0); \
                if (EX_A == 2) TF_MASK(s_y, i, 64 * kt - 32);                                  \
                if (EX_A) TF_WEIGHTS(s_y, p_b, i, any);                                        \
                if (PV_A) {                                                                    \
                    if ((i & 3) == 0)                                                          \
                        l_acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(l_ones, __builtin_bit_cast(bf16x8, p_a[i >> 2]), l_acc, 0, 0, 0); \
                    oacc[i & 3] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(                     \
                        vf[r], __builtin_bit_cast(bf16x8, p_a[i >> 2]), oacc[i & 3], 0, 0, 0); \
                }                                                                              \
            } else {                                                                           \
                if (QK_B) s_y = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[r], qf[i], i ? s_y : zero16, 0, 0, 0); \
                if (EX_B == 2) TF_MASK(s_x, i, 64 * kt);                                       \
                if (EX_B) TF_WEIGHTS(s_x, p_a, i, any);                                        \
                if (PV_B) {                                                                    \
                    if ((i & 3) == 0)                                                          \
                        l_acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(l_ones, __builtin_bit_cast(bf16x8, p_b[i >> 2]), l_acc, 0, 0, 0); \
                    oacc[i & 3] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(                     \
                        vf[r], __builtin_bit_cast(bf16x8, p_b[i >> 2]), oacc[i & 3], 0, 0, 0); \
                }                                                                              \
            }                                                                                  \
            __builtin_amdgcn_sched_barrier(0);                                                 \
            if (j == 7) {                                                                      \
                if (EX_A) TF_RESCUE(s_y, p_b, any);                                            \
                if (FIRST) {                                                                   \
                    if (FIRST == 2) { _Pragma("unroll") for (int v = 0; v < 8; ++v) TF_MASK(s_x, v, 0); } \
                    neg_mc = -row_max(s_x) * scale_log2 - kRefBits;                            \
                }                                                                              \
            }                                                                                  \
            if (j == 11) TF_DELIVER_K(MORE);                                                   \
            if (j == 13) TF_DELIVER_V(MORE);                                                   \
        }                                                                                      \
        if (EX_B) TF_RESCUE(s_x, p_a, any);                                                    \
    } while (0)

    // Iteration kt: scores of the two blocks of K tile kt, weights of blocks 2 kt - 1 and 2 kt, products
    // of blocks 2 kt - 2 and 2 kt - 1 with V tile kt - 1.  It requests K(kt + 1) and V(kt) at its
    // start and writes them to the stages that K(kt - 1) and V(kt - 2) have left; iteration
    // n_kt only finishes.  A wave runs n_kt + 1 iterations with a barrier after each but the
    // last, whatever it has to compute in them.
    // (pos_k: rows of K tile kt + 2, pos_v: of V tile kt + 1, requested in iteration kt)
#define TF_REQUEST(MORE)                                                                       \
    do {                                                                                       \
        if (MORE) TF_LOAD_IDX(pos_n, (kt + 3) * kBN);                                          \
    } while (0)
#define TF_DELIVER_K(MORE)                                                                     \
    do {                                                                                       \
        if (MORE) {                                                                            \
            TF_STORE_K((kt & 1) ^ 1);                                                          \
            TF_LOAD_ROWS(kreg, Kb, pos_k);                                                     \
        }                                                                                      \
    } while (0)
#define TF_DELIVER_V(MORE)                                                                     \
    do {                                                                                       \
        if (MORE) {                                                                            \
            TF_STORE_V(kt & 1);                                                                \
            TF_LOAD_ROWS(vreg, Vb, pos_v);                                                     \
        }                                                                                      \
    } while (0)
#define TF_ADVANCE()                                                                           \
    do {                                                                                       \
        _Pragma("unroll") for (int p = 0; p < NP; ++p)                                         \
            _Pragma("unroll") for (int i = 0; i < 2; ++i) { pos_v[p][i] = pos_k[p][i]; pos_k[p][i] = pos_n[p][i]; } \
        ++kt;                                                                                  \
        ks = k_lds + (kt & 1) * kKTile;                                                        \
        vs = v_lds + ((kt & 1) ^ 1) * kVTile;                                                  \
        __syncthreads();                                                                       \
    } while (0)
    int kt = 0;
    const uint16_t* ks = k_lds;
    const uint16_t* vs = v_lds + kVTile;
    if (h_diag > 0) {
        TF_TILE(true, 0, false, true, 1, false, 1, true);
    } else if (h_diag == 0) {
        TF_TILE(true, 0, false, false, 1, false, 2, true);
    } else {
        TF_REQUEST(true);
        TF_DELIVER_K(true);
        TF_DELIVER_V(true);
    }
    TF_ADVANCE();
    while (2 * kt + 1 <= h_diag) {
        TF_TILE(true, 1, true, true, 1, true, 0, true);
        TF_ADVANCE();
    }
    // the wave's masked block: the first half of K tile kt, or the second half of the one before
    if (h_diag >= 0) {
        bool last_even = h_diag == 0;
        if (h_diag > 0 && (h_diag & 1) == 0) {
            TF_TILE(true, 1, true, false, 2, true, 0, true);
            TF_ADVANCE();
            last_even = true;
        }
        if (last_even) {
            TF_TILE(false, 0, true, false, 0, false, 0, kt < n_kt);
        } else {
            TF_TILE(false, 2, true, false, 0, true, 0, kt < n_kt);
        }
        if (kt < n_kt) TF_ADVANCE();
        else ++kt;
    }
    // nothing left to compute: only the tiles of the others
    while (kt <= n_kt) {
        if (kt == n_kt) break;
        TF_REQUEST(true);
        TF_DELIVER_K(true);
        TF_DELIVER_V(true);
        TF_ADVANCE();
    }
#undef TF_ADVANCE
#undef TF_DELIVER_V
#undef TF_DELIVER_K
#undef TF_REQUEST
#undef TF_TILE
#undef TF_RESCUE
#undef TF_WEIGHTS
#undef TF_MASK
#undef TF_STORE_V
#undef TF_STORE_K
#undef TF_LOAD_ROWS
#undef TF_LOAD_IDX

    // normalise, transpose through LDS and write whole rows
    // (the lane number goes through an opaque move so that the addresses below are formed
    // here, per item, instead of being carried in registers across the tile loop)
    int ln = lane;
    asm volatile("" : "+v"(ln));
    uint16_t* os = ostage + wave * (WQ * kOStr);  // [WQ queries][kOStr], this wave's alone
    {
        const float l_lo = __shfl(l_acc[0], ln & 15), l_hi = __shfl(l_acc[1], ln & 15);
        const float l_tot = (ln & 16) ? l_hi : l_lo;
        const float inv = l_tot > 0.f ? 1.0f / l_tot : 0.f;
#pragma unroll
        for (int dt = 0; dt < 4; ++dt)
#pragma unroll
            for (int v4 = 0; v4 < 4; ++v4) {
                bf16x4 o4;
#pragma unroll
                for (int e = 0; e < 4; ++e) o4[e] = (__bf16)(oacc[dt][4 * v4 + e] * inv);
                *reinterpret_cast<bf16x4*>(os + (ln & 31) * kOStr + 32 * dt + 8 * v4 + 4 * (ln >> 5)) = o4;
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
        for (int it = 0; it < 8; ++it) {
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
    // (no barrier here: the last tile-loop iteration ended with one, after which nobody reads a
    // tile stage, and the staging area is not shared)
    }  // items
}

}  // namespace

hipError_t launch_attend_bf16(const Dims& d, float scale, const void* Q, const void* K,
                              const void* V, const int32_t* kept_idx, void* O, int n_cu, int n_xcd,
                              const int32_t* counts, long long idx_stride, hipStream_t s)
{
    // the tile gathers address a row as a 32-bit byte offset from its (batch, head) slice
    if (d.n > (1 << 24) || d.kvs[2] * 2 >= (1 << 24) || (long long)d.n * d.kvs[2] * 2 >= (1ll << 32))
        return hipErrorInvalidValue;
    n_xcd = std::max(n_xcd, 1);
    // with per-row counts d.m is the bound (the longest possible row)
    constexpr int NW = 8;
    constexpr int kBM = 32 * NW, wg_per_cu = 8 / NW;
    const int n_qt = (d.m + kBM - 1) / kBM;
    const long long items = (long long)d.B * d.Hq * n_qt;
    // persistent workgroups: as many as are resident at once; at least one per XCD, so that every
    // residue of id % n_xcd owns a share of the groups
    const int grid = (int)std::max<long long>(n_xcd, std::min<long long>(items, (long long)wg_per_cu * std::max(n_cu, 1)));
    attend_bf16_kernel<NW><<<dim3(grid), dim3(64 * NW), 0, s>>>(
        d, scale * 1.44269504088896340736f, n_qt, n_xcd, (const uint16_t*)Q,
        (const uint16_t*)K, (const uint16_t*)V, kept_idx, (uint16_t*)O, counts,
        counts ? idx_stride : (long long)d.m);
    return hipGetLastError();
}

}  // namespace tf
