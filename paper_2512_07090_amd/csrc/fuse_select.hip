// Head statistics and variance-aware fusion (Algorithm 1 mean/var/alpha/s_KV lines; Eq. 2),
// the exact-count keep decision (Algorithm 1 "skip if s_KV > tau" with tau placed so that
// exactly m tokens stay), and stream compaction of the kept positions.
#include "tf_kernels.h"

namespace tf {

namespace {

// ------------------------------------------------------------------------------ fusion
// 64 tokens per workgroup.  All 256 threads stage the tokens' per-head cosines in LDS
// ([head][token]: global reads and LDS accesses are unit-stride across a wave), eight heads a
// thread under way at once (one by one, 32 heads are eight round trips to memory in a row: 8 x
// 4096 tokens 6.3 -> 5.2 us); then one thread per token takes the mean and the two-pass variance
// over the heads (the head count is a run-time value).
constexpr int kFuseTokens = 64;
constexpr int kFuseThreads = 256;

// One token's score from its per-head cosines, `stride` apart.
__device__ __forceinline__ float fuse_token(const float* ck, const float* cv, int stride, int H, int mode)
{
    float sk = 0.f, sv = 0.f;
#pragma unroll 8
    for (int h = 0; h < H; ++h) {
        sk += ck[h * stride];
        sv += cv[h * stride];
    }
    const float inv_h = 1.0f / (float)H;
    sk *= inv_h;
    sv *= inv_h;
    float vk = 0.f, vv = 0.f;
#pragma unroll 8
    for (int h = 0; h < H; ++h) {
        const float dk = ck[h * stride] - sk;
        const float dv = cv[h * stride] - sv;
        vk = fmaf(dk, dk, vk);
        vv = fmaf(dv, dv, vv);
    }
    const float ek = vk * inv_h + 1e-12f, ev = vv * inv_h + 1e-12f;
    float alpha;
    if (mode == 0)
        alpha = ek / (ek + ev);  // = (1/ev) / (1/ek + 1/ev), the printed form of Eq. 2
    else if (mode == 1)
        alpha = ev / (ek + ev);  // = (1/ek) / (1/ek + 1/ev)
    else
        alpha = mode == 2 ? 1.f : 0.f;
    return alpha * sk + (1.f - alpha) * sv;
}

__global__ __launch_bounds__(kFuseThreads) void fuse_kernel(const float* __restrict__ sim_k,
                                                            const float* __restrict__ sim_v,
                                                            int H, int n, int mode,
                                                            float* __restrict__ fused)
{
    extern __shared__ float stage[];  // [2][H][kFuseTokens]
    float* ck = stage;
    float* cv = stage + (size_t)H * kFuseTokens;
    const int b = blockIdx.y;
    const int tok = threadIdx.x & (kFuseTokens - 1);
    const int hg = __builtin_amdgcn_readfirstlane(threadIdx.x / kFuseTokens);   // a wave each
    const int t = blockIdx.x * kFuseTokens + tok;
    if (t < n) {
        // key-only / value-only scores read one tensor's cosines (the other was not computed)
        const float* pk = (mode == 3 ? sim_v : sim_k) + (long long)b * H * n + t;
        const float* pv = (mode == 2 ? sim_k : sim_v) + (long long)b * H * n + t;
        // eight heads of each tensor under way at a time
        constexpr int kStep = kFuseThreads / kFuseTokens, kBatch = 8;
        for (int h0 = hg; h0 < H; h0 += kStep * kBatch) {
            float k[kBatch], v[kBatch];
#pragma unroll
            for (int u = 0; u < kBatch; ++u)
                if (const int h = h0 + u * kStep; h < H) { k[u] = pk[(long long)h * n]; v[u] = pv[(long long)h * n]; }
#pragma unroll
            for (int u = 0; u < kBatch; ++u)
                if (const int h = h0 + u * kStep; h < H) { ck[h * kFuseTokens + tok] = k[u]; cv[h * kFuseTokens + tok] = v[u]; }
        }
    }
    __syncthreads();
    if (hg != 0 || t >= n) return;
    fused[(long long)b * n + t] = fuse_token(ck + tok, cv + tok, kFuseTokens, H, mode);
}

// ------------------------------------------------------------------------------ block scan
constexpr int kSelThreads = 1024;
constexpr int kSelWaves = kSelThreads / 64;

// Exclusive prefix sum of one int per thread over the 1024-thread block; *total gets the
// block sum.  `lds` must hold kSelWaves + 1 ints.  Ends with a barrier, so `lds` may be
// reused immediately.
__device__ __forceinline__ int block_excl_scan(int v, int* lds, int* total)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    // inclusive over the wave, in the VALU: shifts by 1, 2, 4, 8 within rows of 16 lanes, then the rows before
    int inc = v;
    inc += __builtin_amdgcn_update_dpp(0, inc, 0x111, 0xf, 0xf, true);   // row_shr
    inc += __builtin_amdgcn_update_dpp(0, inc, 0x112, 0xf, 0xf, true);
    inc += __builtin_amdgcn_update_dpp(0, inc, 0x114, 0xf, 0xf, true);
    inc += __builtin_amdgcn_update_dpp(0, inc, 0x118, 0xf, 0xf, true);
    inc += __builtin_amdgcn_update_dpp(0, inc, 0x142, 0xa, 0xf, true);   // row_bcast 15: rows 1 and 3
    inc += __builtin_amdgcn_update_dpp(0, inc, 0x143, 0xc, 0xf, true);   // row_bcast 31: rows 2 and 3
    if (lane == 63) lds[wave] = inc;
    __syncthreads();
    int base = 0, tot = 0;
#pragma unroll
    for (int w = 0; w < kSelWaves; ++w) {
        const int x = lds[w];
        if (w < wave) base += x;
        tot += x;
    }
    __syncthreads();
    *total = tot;
    return base + inc - v;
}

// Order-preserving map from float to unsigned; -0 is folded onto +0 so that the two compare
// equal, as they do as floats (ties then go by index).
__device__ __forceinline__ unsigned f2key(float f)
{
    unsigned u = __builtin_bit_cast(unsigned, f);
    if (u == 0x80000000u) u = 0u;
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
__device__ __forceinline__ float key2f(unsigned k)
{
    const unsigned u = (k & 0x80000000u) ? (k & 0x7fffffffu) : ~k;
    return __builtin_bit_cast(float, u);
}

// ------------------------------------------------------------------------------ decision
// One workgroup per batch row.  The `want`-th smallest score among the non-forced tokens is
// found by a most-significant-digit-first radix select on the order-preserving keys (four
// passes of 8 bits, a 256-bin LDS histogram each); tokens strictly below it are kept, tokens
// equal to it are kept in index order until the count is met.
__global__ __launch_bounds__(kSelThreads) void select_kernel(const float* __restrict__ fused,
                                                             int n, int m, int warmup,
                                                             uint8_t* __restrict__ keep,
                                                             float* __restrict__ tau)
{
    __shared__ int hist[256];
    __shared__ int scan_lds[kSelWaves + 1];
    __shared__ unsigned sel_prefix;
    __shared__ int sel_k;

    const int b = blockIdx.x;
    const float* S = fused + (long long)b * n;
    uint8_t* kp = keep + (long long)b * n;
    const int tid = threadIdx.x;
    const int forced = min(max(warmup, 0), m);
    const int want = m - forced;

    if (m >= n || want <= 0) {
        for (int t = tid; t < n; t += kSelThreads) kp[t] = (m >= n || t < forced) ? 1 : 0;
        if (tid == 0 && tau) tau[b] = m >= n ? INFINITY : -INFINITY;
        return;
    }

    unsigned prefix = 0;
    int k = want;  // 1-based rank still to find inside the current prefix bucket
    for (int pass = 0; pass < 4; ++pass) {
        const int shift = 24 - 8 * pass;
        const unsigned himask = pass == 0 ? 0u : (0xffffffffu << (shift + 8));
        if (tid < 256) hist[tid] = 0;
        __syncthreads();
        for (int t = forced + tid; t < n; t += kSelThreads) {
            const unsigned key = f2key(S[t]);
            if ((key & himask) == prefix) atomicAdd(&hist[(key >> shift) & 255u], 1);
        }
        __syncthreads();
        const int cnt = tid < 256 ? hist[tid] : 0;
        int total;
        const int before = block_excl_scan(cnt, scan_lds, &total);
        if (tid < 256 && before < k && k <= before + cnt) {
            sel_prefix = prefix | ((unsigned)tid << shift);
            sel_k = k - before;
        }
        __syncthreads();
        prefix = sel_prefix;
        k = sel_k;
        __syncthreads();
    }
    const unsigned tkey = prefix;  // key of the want-th smallest score
    const int k_eq = k;            // how many tokens equal to it are kept (>= 1)
    if (tid == 0 && tau) tau[b] = key2f(tkey);

    int eq_base = 0;
    for (int t0 = forced; t0 < n; t0 += kSelThreads) {
        const int t = t0 + tid;
        unsigned key = 0xffffffffu;
        if (t < n) key = f2key(S[t]);
        const int is_eq = (t < n && key == tkey) ? 1 : 0;
        int total;
        const int rank = eq_base + block_excl_scan(is_eq, scan_lds, &total);
        eq_base += total;
        if (t < n) kp[t] = (key < tkey || (is_eq && rank < k_eq)) ? 1 : 0;
    }
    for (int t = tid; t < forced; t += kSelThreads) kp[t] = 1;
}

// ------------------------------------------------------------------------------ compaction
// One workgroup per batch row: ordered exclusive prefix count of the keep flags, kept
// positions written ascending.
__global__ __launch_bounds__(kSelThreads) void compact_kernel(const uint8_t* __restrict__ keep,
                                                              int n, int m,
                                                              int32_t* __restrict__ kept_idx)
{
    __shared__ int scan_lds[kSelWaves + 1];
    const int b = blockIdx.x;
    const uint8_t* kp = keep + (long long)b * n;
    int32_t* out = kept_idx + (long long)b * m;
    int base = 0;
    for (int t0 = 0; t0 < n; t0 += kSelThreads) {
        const int t = t0 + threadIdx.x;
        const int flag = (t < n && kp[t]) ? 1 : 0;
        int total;
        const int pos = base + block_excl_scan(flag, scan_lds, &total);
        base += total;
        if (flag && pos < m) out[pos] = t;
    }
}

// ------------------------------------------------------------------------------ decision + compaction
// Same decision as select_kernel followed by compact_kernel, in one launch, for rows of up to
// 1024 * IPT tokens.  Thread i holds tokens i, i + 1024, ... as keys in registers (loads and
// stores are then contiguous over a wave).  The want-th smallest (score, index) is found by
//   1. a histogram over kBins equal steps between the smallest and the largest score (scores are
//      spread over that range, while their bit patterns share a handful of exponents, so that a
//      histogram of bit patterns is 1024 threads adding to a few bins), and again between the
//      smallest and the largest score of the bin that holds the wanted rank, until that bin
//      holds at most kMaxCand tokens (once or twice; after kLevels times, as when an outlier
//      stretches the range over and over, or at once when a score is infinite or no number, four
//      radix passes over the bit patterns take over);
//   2. those tokens compared with each other.  Where the bin holds equal scores only, the
//      wanted one is picked by its rank in token order.
// Everything at or below the token found is kept.  What bounds it: short rows a chain of some 15
// barriers and LDS round trips, long rows the passes over 32 scores a thread on the one compute unit
// that works on a row.  One row of 32768 tokens: 55 -> 24 us against four radix passes in thread
// order, 2 x 8192: 16 -> 9.3, 8 x 4096: 11.4 -> 7.4, 333: 8.1 -> 4.9.  Reductions and scans of a
// wave are made in the VALU (through LDS, a chain of twelve accesses for the range alone, in another
// timing: 8 x 4096 9.4 -> 8.2, 1 x 2048 6.6 -> 5.8).
constexpr int kBins = 2048;
constexpr int kMaxCand = 256;
constexpr int kLevels = 4;

// Positions of flagged tokens in token order: base[i * kSelWaves + wave] + the lane's rank in its
// ballot.  `base` holds IPT * kSelWaves ints; returns the number of flagged tokens; ends with a
// barrier.
template <int IPT>
__device__ __forceinline__ int ordered_bases(const unsigned long long* ballots, int* base, int* scan_lds)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (lane == 0) {
#pragma unroll
        for (int i = 0; i < IPT; ++i) base[i * kSelWaves + wave] = __popcll(ballots[i]);
    }
    __syncthreads();
    const int v = threadIdx.x < IPT * kSelWaves ? base[threadIdx.x] : 0;
    int total;
    const int before = block_excl_scan(v, scan_lds, &total);
    if (threadIdx.x < IPT * kSelWaves) base[threadIdx.x] = before;
    __syncthreads();
    return total;
}
__device__ __forceinline__ int rank_below(unsigned long long ballot)
{
    return __builtin_amdgcn_mbcnt_hi((unsigned)(ballot >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)ballot, 0));
}

//
// FUSE: the scores are not there yet; the workgroup makes them from the row's cosines (at most
// kFuseFloats a tensor, staged in LDS) with the arithmetic of fuse_kernel and writes them to `fused`.
// That takes about 2 us here and 4 in a launch of its own; a longer row, or one with more heads,
// would keep one compute unit loading what fuse_kernel spreads over many.  Whole calls: 32 heads x
// 333 tokens 29.4 -> 27.3 us, fp32 32 x 512 36.9 -> 35.5 (the kernel 9.5 -> 7.6 with all loads under
// way at once); 8 heads x 2048 tokens (four a thread) 0.5 us slower a call.
constexpr int kFuseFloats = 16384;

template <int IPT, bool FUSE>
__global__ __launch_bounds__(kSelThreads) void select_compact_kernel(
    float* __restrict__ fused, int n, int m, int warmup, uint8_t* __restrict__ keep,
    int32_t* __restrict__ kept_idx, float* __restrict__ tau, const float* __restrict__ sim_k,
    const float* __restrict__ sim_v, int H, int mode)
{
    // copies of the histogram, one per lane residue: a wave's tokens fall into few bins at times
    // (runs of like tokens), and lanes adding to one word take turns
    constexpr int kCopies = IPT >= 8 ? 8 : 2;
    __shared__ __attribute__((aligned(16))) int hist[kBins * kCopies];
    __shared__ float cand[kMaxCand];
    __shared__ int cand_idx[kMaxCand];
    __shared__ int base[IPT * kSelWaves];
    __shared__ int scan_lds[kSelWaves + 1];
    __shared__ float lo_lds[kSelWaves], hi_lds[kSelWaves];
    __shared__ unsigned sel_u;
    __shared__ float sel_f;
    __shared__ int sel_k, sel_cnt, n_cand;

    const int b = blockIdx.x;
    float* S = fused + (long long)b * n;
    uint8_t* kp = keep + (long long)b * n;
    int32_t* out = kept_idx + (long long)b * m;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int forced = min(max(warmup, 0), m);
    const int want = m - forced;
    const bool all = m >= n;            // nothing is filtered
    const bool none = want <= 0;        // no non-forced token is kept

    // (every load is issued whatever the token, so that none waits for the one before; forced tokens
    // and the tail past n take no part in the selection: they stay above every score)
    float sc[IPT];
    if constexpr (FUSE) {
        __shared__ float cos_k[kFuseFloats], cos_v[kFuseFloats];   // [head][token], as in memory
        // (key-only / value-only scores read one tensor's cosines, the other was not computed)
        const float* pk = (mode == 3 ? sim_v : sim_k) + (long long)b * H * n;
        const float* pv = (mode == 2 ? sim_k : sim_v) + (long long)b * H * n;
        constexpr int kEach = kFuseFloats / kSelThreads;   // all of a thread's loads under way at once
        float k[kEach], v[kEach];
#pragma unroll
        for (int u = 0; u < kEach; ++u)
            if (u * kSelThreads < H * n) {   // (uniform)
                const int i = min(u * kSelThreads + tid, H * n - 1);
                k[u] = pk[i];
                v[u] = pv[i];
            }
#pragma unroll
        for (int u = 0; u < kEach; ++u)
            if (const int i = u * kSelThreads + tid; i < H * n) { cos_k[i] = k[u]; cos_v[i] = v[u]; }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < IPT; ++i) {
            const int t = i * kSelThreads + tid;
            sc[i] = 0.f;
            if (t < n) S[t] = sc[i] = fuse_token(cos_k + t, cos_v + t, n, H, mode);
        }
    } else {
#pragma unroll
        for (int i = 0; i < IPT; ++i) sc[i] = S[min(i * kSelThreads + tid, n - 1)];
    }
    auto takes_part = [&](int i) { return i * kSelThreads + tid >= forced && i * kSelThreads + tid < n; };
    bool finite = true;
#pragma unroll
    for (int i = 0; i < IPT; ++i)
        if (!takes_part(i)) sc[i] = INFINITY;
        else finite = finite && fabsf(sc[i]) < INFINITY;

    // smallest and largest score over the workgroup; one barrier before the result, none after
    auto min_max = [&](float& lo, float& hi) {
        lo = fminf(lo, dpp_mov<0xB1>(lo));    hi = fmaxf(hi, dpp_mov<0xB1>(hi));    // as in row16_sum
        lo = fminf(lo, dpp_mov<0x4E>(lo));    hi = fmaxf(hi, dpp_mov<0x4E>(hi));
        lo = fminf(lo, dpp_mov<0x141>(lo));   hi = fmaxf(hi, dpp_mov<0x141>(hi));
        lo = fminf(lo, dpp_mov<0x140>(lo));   hi = fmaxf(hi, dpp_mov<0x140>(hi));
        const FloatPair lo16 = swap16(lo, lo), hi16 = swap16(hi, hi);
        lo = fminf(lo16.first, lo16.second);  hi = fmaxf(hi16.first, hi16.second);
        const FloatPair lo32 = swap32(lo, lo), hi32 = swap32(hi, hi);
        lo = fminf(lo32.first, lo32.second);  hi = fmaxf(hi32.first, hi32.second);
        if (lane == 0) { lo_lds[wave] = lo; hi_lds[wave] = hi; }
        __syncthreads();
#pragma unroll
        for (int w = 0; w < kSelWaves; ++w) { lo = fminf(lo, lo_lds[w]); hi = fmaxf(hi, hi_lds[w]); }
    };

    float tf_ = 0.f, tau_ = 0.f;   // tau_: the score itself where tf_ stands for its key
    bool by_key = false;
    int tidx = -1;   // kept: forced, or (score, index) <= (tf_, tidx)
    if (!all && !none) {
        // the wanted token is the k-th smallest of those with scores lo .. hi (in bin `bin` of that range)
        float lo = INFINITY, hi = -INFINITY, to_bin = 0.f;
        int k = want, cnt = n - forced, bin = 0;
        // monotone in the score: a rounded difference times a constant, truncated
        auto bin_of = [&](float x) -> int { return (int)fminf((x - lo) * to_bin, (float)(kBins - 1)); };
#pragma unroll
        for (int i = 0; i < IPT; ++i) {
            lo = fminf(lo, sc[i]);
            hi = fmaxf(hi, sc[i] == INFINITY ? -INFINITY : sc[i]);
        }
        if (!finite) hi = INFINITY;
        bool few = false;
        for (int level = 0;; ++level) {
            for (int i = 4 * tid; i < kBins * kCopies; i += 4 * kSelThreads) *reinterpret_cast<int4*>(&hist[i]) = make_int4(0, 0, 0, 0);
            if (tid == 0) n_cand = 0;
            min_max(lo, hi);
            if (lo == hi || level == kLevels || hi == INFINITY) break;
            to_bin = fminf((float)kBins / (hi - lo), 3e38f);
#pragma unroll
            for (int i = 0; i < IPT; ++i)
                if (sc[i] >= lo && sc[i] <= hi) atomicAdd(&hist[bin_of(sc[i]) * kCopies + (lane & (kCopies - 1))], 1);
            __syncthreads();
            int c0 = 0, c1 = 0;
#pragma unroll
            for (int c = 0; c < kCopies; ++c) { c0 += hist[2 * tid * kCopies + c]; c1 += hist[(2 * tid + 1) * kCopies + c]; }
            int total;
            const int before = block_excl_scan(c0 + c1, scan_lds, &total);
            if (before < k && k <= before + c0) { sel_u = 2 * tid; sel_k = k - before; sel_cnt = c0; }
            else if (before + c0 < k && k <= before + c0 + c1) { sel_u = 2 * tid + 1; sel_k = k - before - c0; sel_cnt = c1; }
            __syncthreads();
            bin = (int)sel_u;
            k = sel_k;
            cnt = sel_cnt;
            few = cnt <= kMaxCand;
            if (few) break;
            float lo2 = INFINITY, hi2 = -INFINITY;
#pragma unroll
            for (int i = 0; i < IPT; ++i)
                if (sc[i] >= lo && sc[i] <= hi && bin_of(sc[i]) == bin) { lo2 = fminf(lo2, sc[i]); hi2 = fmaxf(hi2, sc[i]); }
            lo = lo2;
            hi = hi2;
        }
        bool tie = false;   // the wanted token is the k-th of those with score tf_, in token order
        if (few) {
#pragma unroll
            for (int i = 0; i < IPT; ++i)
                if (sc[i] >= lo && sc[i] <= hi && bin_of(sc[i]) == bin) {
                    const int c = atomicAdd(&n_cand, 1);
                    cand[c] = sc[i];
                    cand_idx[c] = i * kSelThreads + tid;
                }
            __syncthreads();
            if (tid < cnt) {
                const float mine = cand[tid];
                const int my_idx = cand_idx[tid];
                int rank = 0;
                for (int c = 0; c < cnt; ++c) {
                    const float other = cand[c];
                    rank += (other < mine || (other == mine && cand_idx[c] < my_idx)) ? 1 : 0;
                }
                if (rank == k - 1) { sel_f = mine; sel_k = my_idx; }
            }
            __syncthreads();
            tf_ = sel_f;
            tidx = sel_k;
        } else if (lo == hi && hi != INFINITY) {
            tf_ = lo;
            tie = true;
        } else {
            unsigned prefix = 0;
            k = want;  // 1-based rank still to find inside the current prefix bucket
            for (int pass = 0; pass < 4; ++pass) {
                const int shift = 24 - 8 * pass;
                const unsigned himask = pass == 0 ? 0u : (0xffffffffu << (shift + 8));
                if (tid < 256) hist[tid] = 0;
                __syncthreads();
                for (int i = 0; i < IPT; ++i) {
                    const unsigned key = f2key(sc[i]);
                    if (takes_part(i) && (key & himask) == prefix) atomicAdd(&hist[(key >> shift) & 255u], 1);
                }
                __syncthreads();
                const int c = tid < 256 ? hist[tid] : 0;
                int total;
                const int before = block_excl_scan(c, scan_lds, &total);
                if (tid < 256 && before < k && k <= before + c) {
                    sel_u = prefix | ((unsigned)tid << shift);
                    sel_k = k - before;
                }
                __syncthreads();
                prefix = sel_u;
                k = sel_k;
                __syncthreads();
            }
            // from here on only the order of the keys matters (a NaN compares with nothing)
#pragma unroll
            for (int i = 0; i < IPT; ++i) {
                const unsigned key = f2key(sc[i]);
                sc[i] = !takes_part(i) || key > prefix ? 1.f : (key == prefix ? 0.f : -1.f);
            }
            tau_ = key2f(prefix);
            by_key = true;
            tie = true;
        }
        if (tie) {
            unsigned long long eq[IPT];
#pragma unroll
            for (int i = 0; i < IPT; ++i) eq[i] = __ballot(sc[i] == tf_);
            ordered_bases<IPT>(eq, base, scan_lds);
#pragma unroll
            for (int i = 0; i < IPT; ++i)
                if (((eq[i] >> lane) & 1) && base[i * kSelWaves + wave] + rank_below(eq[i]) == k - 1)
                    sel_k = i * kSelThreads + tid;
            __syncthreads();
            tidx = sel_k;
        }
    }
    // (-0 counts as +0 and is given as that, as the radix passes do)
    if (tid == 0 && tau) tau[b] = all ? INFINITY : (none ? -INFINITY : (by_key ? tau_ : tf_ + 0.f));

    unsigned long long kept[IPT];
#pragma unroll
    for (int i = 0; i < IPT; ++i) {
        const int t = i * kSelThreads + tid;
        const bool chosen = !none && (sc[i] < tf_ || (sc[i] == tf_ && t <= tidx));
        const bool mine = t < n && (all || t < forced || chosen);
        kept[i] = __ballot(mine);
        if (t < n) kp[t] = mine ? 1 : 0;
    }
    ordered_bases<IPT>(kept, base, scan_lds);
#pragma unroll
    for (int i = 0; i < IPT; ++i)
        if ((kept[i] >> lane) & 1) {
            const int pos = base[i * kSelWaves + wave] + rank_below(kept[i]);
            if (pos < m) out[pos] = i * kSelThreads + tid;
        }
}

// ------------------------------------------------------------------------------ online decision
// Adaptive threshold (Algorithm 1 threshold / skip lines, warm-up of Section 3.2, Eq. 4): a
// sequential recurrence over a row's tokens,
//   skip iff t >= W and S_t > tau;  tau <- fma(eta, (float)skipped * (1 / (t + 1)) - target, tau),
// all in float so that the result is reproducible bit for bit.  One workgroup per batch row
// walks the row in chunks of kOnChunk tokens: all threads stage the chunk's scores and the
// reciprocals in LDS, wave 0 decides 64 tokens at a time, then all threads compact the decisions.
//
// 64 tokens at once: the decisions are guessed, the thresholds that follow from them are computed
// for all 64 tokens together, and the decisions that follow from those replace the guess, until
// they agree.  The first wrong guess is right the next time (all before it were), so this ends
// after at most 64 rounds; it mostly takes one or two, because the threshold moves little over 64 tokens.
// The thresholds of given decisions: the skipped counts are a prefix sum of bits, so every
// product and difference is formed as the recurrence forms it; what is left, a chain of 64 fma
// roundings, is a prefix sum as well as long as the threshold stays inside one binade: it is then
// a multiple of one ulp g, and rounding tau + eta * diff to a multiple of g rounds the exact
// product eta * diff (formed in double) to a multiple of g, ties apart.  Where the threshold leaves
// its binade or a tie occurs, the tokens before are taken, that one step is made with the fma
// itself, and the next 64 tokens begin after it.
// What bounds it is a lone wave's chain: it waits about 10 cycles for every dependent result, which is 26 ns a
// token one by one, and 0.34 us for a step of one round.  Scores spread about a threshold away
// from zero take 1.0 to 1.3 steps per 64 tokens (8 rows of 4096: 32 us; all of it token by token 119).  A
// threshold near zero leaves its binade often (4 to 5 steps per 64 tokens), one that rests on a power of
// two ends every step at its first token, and an eta of few bits ties often (15 to 20 steps per 64 tokens
// at 0.25 to 1): in such steps alone 8 rows of 4096 took 75 to 153, 1385, and 380 to 440 us.  So every kOnSteps
// steps are looked at together: where they took fewer tokens than one by one in the same time, the row
// goes on one by one, for longer and longer stretches while the kOnProbe steps tried in between do not pay
// either: 79 to 119 us for all of these.
constexpr int kOnStep = 13;                  // a step's cost, in tokens taken one by one
constexpr int kOnSteps = 4, kOnProbe = 2;    // (16: 3 us more in a row before it changes its pace)
constexpr int kOnRun = 64;                   // tokens of the first stretch
constexpr int kOnShort = 256;                // rows up to here are taken one by one: 7 us, 4 to 11 in steps
constexpr int kOnChunk = 4096;

// inclusive prefix sum over the wave (row_shr 1, 2, 4, 8, then row_bcast 15 and 31)
__device__ __forceinline__ int wave_incl_scan(int v)
{
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);
    return v;
}

// Up to `many` tokens from token i0 of the chunk on, one after the other, with the decisions left as the
// steps of 64 leave them; called by a whole wave, s_u and inv hold its next 64 tokens.  A function of its own:
// inlined it costs the steps of 64 another 1.5 % (registers and branches in their loop).
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) float lds_float;
typedef __attribute__((address_space(3))) f32x4 lds_f32x4;
struct OneByOne { float tau, tau_judged; int skipped, i0; };
__device__ __attribute__((noinline)) OneByOne take_one_by_one(
    lds_float* s_lds, const lds_float* inv_lds, float s_u, float inv, float tau, float tau_judged,
    int skipped, int i0, int len, int many, float eta, float target)
{
    const int lane = threadIdx.x & 63;
    // 16 at a time from registers; a row may end inside such a block (what follows its last token is
    // read by nobody).  The running count of skipped tokens replaces the scores.
    const int i_first = i0, i_block = min((i0 + 15) & ~15, len);
    const int stop_at = min((i0 + many + 15) & ~15, (len + 15) & ~15);
    const float before = (float)skipped;
    float cnt = before;
    auto step = [&](float s, float iv) {
#pragma clang fp contract(off)
        const float s1 = cnt + 1.f;
        cnt = s > tau ? s1 : cnt;
        const float p_next = cnt * iv;
        const float d = p_next - target;
        tau = fmaf(eta, d, tau);
    };
    auto lane_of = [](float x, int l) { return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, x), l)); };
    // (up to the first block: from the 64 at hand)
    for (; i0 < i_block; ++i0) {
        tau_judged = tau;
        step(lane_of(s_u, i0 - i_first), lane_of(inv, i0 - i_first));
        if (lane == 0) s_lds[i0] = cnt;
    }
    if (i0 < min(stop_at, len) && lane == 0) {   // i0 is a multiple of 16 then
        struct Eight { f32x4 s[2], iv[2]; } a, c;   // one in use, the next requested
        auto request = [&](Eight& e, int at) {
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                e.s[h] = *(const lds_f32x4*)(s_lds + at + 4 * h);
                e.iv[h] = *(const lds_f32x4*)(inv_lds + at + 4 * h);
            }
        };
        float tau_in[16];
        auto eight = [&](const Eight& e, int at, float* in) {
            f32x4 counts[2];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                in[u] = tau;
                step(e.s[u >> 2][u & 3], e.iv[u >> 2][u & 3]);
                counts[u >> 2][u & 3] = cnt;
            }
            *(lds_f32x4*)(s_lds + at) = counts[0];
            *(lds_f32x4*)(s_lds + at + 4) = counts[1];
        };
        request(a, i0 & ~15);
        for (int i = i0 & ~15; i < stop_at; i += 16) {
            request(c, i + 8);
            eight(a, i, tau_in);
            request(a, i + 16);   // (64 entries of padding behind the chunk)
            eight(c, i + 8, tau_in + 8);
        }
#pragma unroll
        for (int u = 0; u < 16; ++u)
            if (stop_at - 16 + u < len) tau_judged = tau_in[u];
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");   // lane 0's counts, read by the others
    __builtin_amdgcn_wave_barrier();
    // skipped where the count moved; from the back, because a token's count is its neighbour's too
    i0 = max(i0, min(stop_at, len));
    for (int i = i_first + ((i0 - 1 - i_first) & ~63); i >= i_first; i -= 64) {
        const int t = i + lane;
        const float mine = t < i0 ? s_lds[t] : 0.f;
        const float prev = t == i_first ? before : (t < i0 ? s_lds[t - 1] : 0.f);
        if (t < i0) s_lds[t] = mine != prev ? 1.f : 0.f;
    }
    return OneByOne{lane_of(tau, 0), lane_of(tau_judged, 0), (int)lane_of(cnt, 0), i0};
}

__global__ __launch_bounds__(kSelThreads) void select_online_kernel(
    const float* __restrict__ fused, int n, int warmup, float target, float eta, float tau0,
    uint8_t* __restrict__ keep, int32_t* __restrict__ kept_idx, int32_t* __restrict__ count,
    float* __restrict__ tau_out)
{
    // every product and difference below is rounded on its own (the only fused operations are
    // the fmaf calls): the recurrence is defined operation by operation
#pragma clang fp contract(off)
    __shared__ __attribute__((aligned(16))) float s_lds[kOnChunk + 64];    // scores, then decisions (1 = skipped)
    __shared__ __attribute__((aligned(16))) float inv_lds[kOnChunk + 64];
    __shared__ int base_lds[kOnChunk / kSelThreads * kSelWaves];
    __shared__ int scan_lds[kSelWaves + 1];

    const int b = blockIdx.x;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const float* S = fused + (long long)b * n;
    uint8_t* kp = keep + (long long)b * n;
    int32_t* out = kept_idx + (long long)b * n;

    // state of the recurrence (meaningful in wave 0, the same in all its lanes): tau is the threshold
    // the next token will be judged with, already updated for it
    int skipped = 0;  // exact in float up to 2^24 tokens
    float tau = fmaf(eta, 0.f - target, tau0);
    float drift = eta * (0.f - target);   // its latest movement (only the guess depends on it)
    float tau_judged = tau;  // the threshold the latest token was judged with
    int base = 0;            // kept tokens so far
    // steps still to make before they are looked at, of so many that began at token `mark` of the chunk;
    // the next stretch of tokens one by one, what is left of this one
    int left = kOnSteps, steps = kOnSteps, mark = 0, run = kOnRun, one_by_one = n <= kOnShort ? n : 0;
    for (int t0 = 0; t0 < n; t0 += kOnChunk) {
        const int len = min(kOnChunk, n - t0);
        // (warm-up tokens and the padding get a score that is never above the threshold, so the
        // rule below needs no test for them)
        for (int i = tid; i < len + 64; i += kSelThreads) {
            s_lds[i] = (i < len && t0 + i >= warmup) ? S[t0 + i] : -INFINITY;
            inv_lds[i] = 1.0f / (float)(t0 + i + 1);   // reciprocal of the NEXT token's index
        }
        __syncthreads();
        if (wave == 0) {
            float s_u = s_lds[lane], inv = inv_lds[lane];
            for (int i0 = 0;;) {
                while (one_by_one == 0) {
                    const int ahead = min(i0 + 64, len) + lane;   // the next 64, if all of these are taken
                    const float s_next = s_lds[ahead], inv_next = inv_lds[ahead];
                    // tau as a multiple of its ulp
                    const unsigned tau_bits = __builtin_bit_cast(unsigned, tau);
                    const int ex = (int)((tau_bits >> 23) & 255u) - 127;
                    const bool grid = ex > -100 && ex < 127;   // an ordinary number
                    const int mant = (int)((tau_bits & 0x7fffffu) | 0x800000u);
                    const float ulp = __builtin_bit_cast(float, (unsigned)max(ex - 23 + 127, 1) << 23);
                    // eta in ulps; its sign makes up for tau's, so that magnitudes are added
                    const double per_ulp = __builtin_bit_cast(double, (unsigned long long)(1023 + 23 - ex) << 52);
                    const double eta_ulp = (tau_bits >> 31) ? -(double)eta * per_ulp : (double)eta * per_ulp;
                    unsigned long long d = __ballot(s_u > fmaf((float)lane, drift, tau));
                    float tau_u, diff;
                    int taken;   // tokens 0 .. taken - 1 of the 64 are decided
                    for (;;) {
                        const int cnt = skipped + rank_below(d) + (int)((d >> lane) & 1);
                        const float p_next = (float)cnt * inv;
                        diff = p_next - target;
                        const double in_ulps = eta_ulp * (double)diff;   // exact
                        const double whole = rint(in_ulps);
                        const bool odd = !(fabs(in_ulps) < 8388608.0) || fabs(in_ulps - whole) == 0.5;
                        const int mag = mant + wave_incl_scan(odd ? 0 : (int)whole);   // at most 65 * 2^23
                        // the first token whose step is not a plain sum
                        const unsigned long long stop = __ballot(!grid || odd || mag <= 0x800000 || mag >= 0x1000000);
                        const int j = stop ? __builtin_ctzll(stop) : 64;
                        const float mag_f = (float)mag * ulp;
                        const float after = (tau_bits >> 31) ? -mag_f : mag_f;
                        // wave_shr 1: the threshold after the token before
                        tau_u = __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(
                            __builtin_bit_cast(int, tau), __builtin_bit_cast(int, after), 0x138, 0xf, 0xf, false));
                        const unsigned long long seen = __ballot(s_u > tau_u);
                        const unsigned long long known = j >= 63 ? ~0ull : (2ull << j) - 1;   // thresholds 0 .. j
                        taken = min(j + 1, 64);
                        if (((seen ^ d) & known) == 0) break;
                        d = (seen & known) | (d & ~known);
                    }
                    taken = min(taken, len - i0);
                    if (lane < taken) s_lds[i0 + lane] = (d >> lane) & 1 ? 1.f : 0.f;
                    tau_judged = __shfl(tau_u, taken - 1);
                    tau = __shfl(fmaf(eta, diff, tau_u), taken - 1);
                    drift = tau - tau_judged;
                    skipped += __popcll(d & (taken == 64 ? ~0ull : (1ull << taken) - 1));
                    i0 += taken;
                    s_u = s_next;
                    inv = inv_next;
                    if (i0 >= len) break;
                    if (taken < 64) { s_u = s_lds[i0 + lane]; inv = inv_lds[i0 + lane]; }
                    if (--left == 0) {
                        const bool pays = i0 - mark >= steps * kOnStep;
                        if (pays && steps == kOnSteps) run = kOnRun;
                        steps = left = pays ? kOnSteps : kOnProbe;
                        mark = i0;
                        if (!pays) {
                            one_by_one = run;
                            run = min(2 * run, kOnChunk);
                            break;
                        }
                    }
                }
                if (i0 >= len) break;
                const OneByOne r = take_one_by_one((lds_float*)s_lds, (const lds_float*)inv_lds, s_u, inv, tau,
                                                   tau_judged, skipped, i0, len, one_by_one, eta, target);
                tau = r.tau;
                tau_judged = r.tau_judged;
                drift = tau - tau_judged;
                skipped = __builtin_amdgcn_readfirstlane(r.skipped);
                mark = __builtin_amdgcn_readfirstlane(r.i0);
                one_by_one = max(0, one_by_one - (mark - i0));
                i0 = mark;
                if (i0 >= len) break;
                s_u = s_lds[i0 + lane];
                inv = inv_lds[i0 + lane];
            }
            mark -= kOnChunk;
        }
        __syncthreads();
        unsigned long long kept[kOnChunk / kSelThreads];
#pragma unroll
        for (int i = 0; i < kOnChunk / kSelThreads; ++i) {
            const int t = i * kSelThreads + tid;
            const bool mine = t < len && s_lds[t] == 0.f;
            kept[i] = __ballot(mine);
            if (t < len) kp[t0 + t] = mine ? 1 : 0;
        }
        const int chunk_kept = ordered_bases<kOnChunk / kSelThreads>(kept, base_lds, scan_lds);
#pragma unroll
        for (int i = 0; i < kOnChunk / kSelThreads; ++i)
            if ((kept[i] >> lane) & 1) out[base + base_lds[i * kSelWaves + wave] + rank_below(kept[i])] = t0 + i * kSelThreads + tid;
        base += chunk_kept;
        __syncthreads();
    }
    for (int i = base + tid; i < n; i += kSelThreads) out[i] = -1;
    if (tid == 0) {
        count[b] = base;
        if (tau_out) tau_out[b] = tau_judged;
    }
}

}  // namespace

hipError_t launch_fuse(const Dims& d, int fusion, const float* sim_k, const float* sim_v,
                       float* fused, hipStream_t s)
{
    const size_t lds = (size_t)2 * d.Hkv * kFuseTokens * sizeof(float);
    dim3 grid((d.n + kFuseTokens - 1) / kFuseTokens, d.B);
    fuse_kernel<<<grid, dim3(kFuseThreads), lds, s>>>(sim_k, sim_v, d.Hkv, d.n, fusion, fused);
    return hipGetLastError();
}

hipError_t launch_select_compact(const Dims& d, int warmup, const float* fused, uint8_t* keep,
                                 int32_t* kept_idx, float* tau, hipStream_t s)
{
    const int ipt = (d.n + kSelThreads - 1) / kSelThreads;
    // (the kernel only reads the scores here)
    float* S = const_cast<float*>(fused);
#define TF_SELECT(IPT) \
    select_compact_kernel<IPT, false><<<dim3(d.B), dim3(kSelThreads), 0, s>>>(S, d.n, d.m, warmup, keep, kept_idx, tau, nullptr, nullptr, 0, 0)
    if (ipt <= 1) TF_SELECT(1);
    else if (ipt <= 4) TF_SELECT(4);
    else if (ipt <= 8) TF_SELECT(8);
    else if (ipt <= 32) TF_SELECT(32);
#undef TF_SELECT
    else {
        // longer rows: scores stay in global memory, decision and compaction in two launches
        select_kernel<<<dim3(d.B), dim3(kSelThreads), 0, s>>>(fused, d.n, d.m, warmup, keep, tau);
        compact_kernel<<<dim3(d.B), dim3(kSelThreads), 0, s>>>(keep, d.n, d.m, kept_idx);
    }
    return hipGetLastError();
}

bool fuse_select_fits(const Dims& d) { return d.n <= kSelThreads && (long long)d.Hkv * d.n <= kFuseFloats; }

hipError_t launch_fuse_select(const Dims& d, int fusion, const float* sim_k, const float* sim_v,
                              int warmup, float* fused, uint8_t* keep, int32_t* kept_idx, float* tau, hipStream_t s)
{
    if (!fuse_select_fits(d)) return hipErrorInvalidValue;
    select_compact_kernel<1, true><<<dim3(d.B), dim3(kSelThreads), 0, s>>>(fused, d.n, d.m, warmup, keep, kept_idx, tau, sim_k,
                                                                           sim_v, d.Hkv, fusion);
    return hipGetLastError();
}

hipError_t launch_select_online(const Dims& d, int warmup, float target, float eta, float tau0,
                                const float* fused, uint8_t* keep, int32_t* kept_idx,
                                int32_t* count, float* tau, hipStream_t s)
{
    select_online_kernel<<<dim3(d.B), dim3(kSelThreads), 0, s>>>(fused, d.n, warmup, target, eta,
                                                                 tau0, keep, kept_idx, count, tau);
    return hipGetLastError();
}

__global__ void keep_all_kernel(int n, uint8_t* __restrict__ keep, int32_t* __restrict__ kept_idx,
                                float* __restrict__ tau)
{
    const int b = blockIdx.y;
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) {
        keep[(long long)b * n + i] = 1;
        kept_idx[(long long)b * n + i] = i;
    }
    if (tau && i == 0) tau[b] = INFINITY;
}

hipError_t launch_keep_all(const Dims& d, uint8_t* keep, int32_t* kept_idx, float* tau,
                           hipStream_t s)
{
    keep_all_kernel<<<dim3((d.n + 255) / 256, d.B), dim3(256), 0, s>>>(d.n, keep, kept_idx, tau);
    return hipGetLastError();
}

__global__ void keep_none_kernel(int n, uint8_t* __restrict__ keep, float* __restrict__ tau)
{
    const int b = blockIdx.y;
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) keep[(long long)b * n + i] = 0;
    if (tau && i == 0) tau[b] = -INFINITY;
}

hipError_t launch_keep_none(const Dims& d, uint8_t* keep, float* tau, hipStream_t s)
{
    keep_none_kernel<<<dim3((d.n + 255) / 256, d.B), dim3(256), 0, s>>>(d.n, keep, tau);
    return hipGetLastError();
}

}  // namespace tf
