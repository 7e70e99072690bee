// Per-token form of the layer (Algorithm 1 called once per new token): score the new key and
// value against the caller-held anchors, move the threshold, decide, absorb the token into the
// anchors, append a kept token to the cache of kept keys / values and attend over that cache.
// Two launches per step: decode_score_kernel (one workgroup per batch row) and the attention over
// the cache, split over workgroups of which the last to end merges the slices.
#include <algorithm>
#include <type_traits>

#include "tf_kernels.h"

namespace tf {

namespace {

constexpr double kEpsCos = 1e-8;
constexpr double kEpsVar = 1e-12;
constexpr float kLowest = -1e30f;  // "no key yet": finite, so differences of two of them are 0
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
constexpr int kPartStride = kDecodePartFloats;  // partial result: 128 numerators, running max, sum

// eight consecutive elements of a row as floats
__device__ __forceinline__ void load8(const uint16_t* p, float* x)
{
    const uint4 r = *reinterpret_cast<const uint4*>(p);
    const unsigned w[4] = {r.x, r.y, r.z, r.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        x[2 * i] = __uint_as_float(w[i] << 16);
        x[2 * i + 1] = __uint_as_float(w[i] & 0xffff0000u);
    }
}
__device__ __forceinline__ void load8(const float* p, float* x)
{
    const float4 a = *reinterpret_cast<const float4*>(p), b = *reinterpret_cast<const float4*>(p + 4);
    x[0] = a.x; x[1] = a.y; x[2] = a.z; x[3] = a.w;
    x[4] = b.x; x[5] = b.y; x[6] = b.z; x[7] = b.w;
}
// the same in two steps: the bytes, and the floats they hold
struct Raw8 { float4 lo, hi; };
__device__ __forceinline__ void unpack8(const Raw8& r, float* x)
{
    x[0] = r.lo.x; x[1] = r.lo.y; x[2] = r.lo.z; x[3] = r.lo.w;
    x[4] = r.hi.x; x[5] = r.hi.y; x[6] = r.hi.z; x[7] = r.hi.w;
}
__device__ __forceinline__ void copy8(uint16_t* dst, const uint16_t* src)
{
    *reinterpret_cast<uint4*>(dst) = *reinterpret_cast<const uint4*>(src);
}
__device__ __forceinline__ void copy8(float* dst, const float* src)
{
    reinterpret_cast<float4*>(dst)[0] = reinterpret_cast<const float4*>(src)[0];
    reinterpret_cast<float4*>(dst)[1] = reinterpret_cast<const float4*>(src)[1];
}
__device__ __forceinline__ void store_out(uint16_t* p, float v)
{
    const unsigned u = __float_as_uint(v);
    *p = (uint16_t)((u + 0x7fffu + ((u >> 16) & 1u)) >> 16);  // round to nearest even
}
__device__ __forceinline__ void store_out(float* p, float v) { *p = v; }

// two consecutive elements
template <typename T> struct Raw2;
template <> struct Raw2<uint16_t> { typedef unsigned type; };
template <> struct Raw2<float> { typedef unsigned long long type; };
__device__ __forceinline__ void unpack2(unsigned r, float* x)
{
    x[0] = __uint_as_float(r << 16);
    x[1] = __uint_as_float(r & 0xffff0000u);
}
__device__ __forceinline__ void unpack2(unsigned long long r, float* x)
{
    x[0] = __uint_as_float((unsigned)r);
    x[1] = __uint_as_float((unsigned)(r >> 32));
}

// A double moved between lanes of its 16-lane row in the VALU (two 32-bit DPP moves): the shuffles
// that go through LDS were most of the scoring kernel's latency.
template <int CTRL, int ROW_MASK = 0xf>
__device__ __forceinline__ double dpp_mov_f64(double v)
{
    const unsigned long long u = __builtin_bit_cast(unsigned long long, v);
    const unsigned lo = __builtin_amdgcn_update_dpp(0, (int)(unsigned)u, CTRL, ROW_MASK, 0xf, false);
    const unsigned hi = __builtin_amdgcn_update_dpp(0, (int)(unsigned)(u >> 32), CTRL, ROW_MASK, 0xf, false);
    return __builtin_bit_cast(double, (unsigned long long)hi << 32 | lo);
}
// sum over each aligned group of 16 lanes; every lane ends with the total
__device__ __forceinline__ double group16_sum(double v)
{
    v += dpp_mov_f64<0xB1>(v);   // quad_perm [1,0,3,2]
    v += dpp_mov_f64<0x4E>(v);   // quad_perm [2,3,0,1]
    v += dpp_mov_f64<0x141>(v);  // row_half_mirror
    v += dpp_mov_f64<0x140>(v);  // row_mirror
    return v;
}

__global__ void decode_init_kernel(double* anchor_k, double* anchor_v, long long n_anchor,
                                   int32_t* seen, int32_t* skipped, float* tau, int32_t* cache_len,
                                   int32_t* overflow, int B, float tau0)
{
    const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n_anchor) { anchor_k[i] = 0.0; anchor_v[i] = 0.0; }
    if (i < B) { seen[i] = 0; skipped[i] = 0; tau[i] = tau0; cache_len[i] = 0; overflow[i] = 0; }
}

// One workgroup per batch row; a 16-lane group per (tensor, KV head) pair, columns 32 i + 2 l and the next of
// lane l, so that its accesses to an anchor are 256 bytes side by side (with eight columns in a row a lane,
// four accesses a lane went to each 64 bytes: a skipped token of 8 x 32 KV heads 10.4 us, 7.6 like this; of
// 128 24.3 and 12.0).  The float operations of the threshold rule are the ones of the batched online
// decision, in the same order, with contraction switched off, so both forms agree bit for bit.  Latency is
// what this kernel costs, so the row's scalars are fetched up front by the lane that needs them, the head
// statistics are reduced by one wave rather than one lane, the anchors are stored before the decision, which
// they do not depend on, and the first row of a group stays in registers for the cache.
#pragma clang fp contract(off)
__device__ __forceinline__ double wave_sum(double v)
{
    v = group16_sum(v);
    v += dpp_mov_f64<0x142, 0xa>(v);   // row_bcast 15: rows 1 and 3 add the row before them
    v += dpp_mov_f64<0x143, 0xc>(v);   // row_bcast 31: rows 2 and 3 add rows 0 and 1
    const unsigned long long u = __builtin_bit_cast(unsigned long long, v);   // lane 63 holds the sum
    const unsigned lo = __builtin_amdgcn_readlane((int)(unsigned)u, 63), hi = __builtin_amdgcn_readlane((int)(unsigned)(u >> 32), 63);
    return __builtin_bit_cast(double, (unsigned long long)hi << 32 | lo);
}

template <typename T>
__device__ __forceinline__ void score_row(
    const T* __restrict__ k, const T* __restrict__ v, double* __restrict__ anchor_k,
    double* __restrict__ anchor_v, int32_t* __restrict__ seen, int32_t* __restrict__ skipped,
    float* __restrict__ tau, int32_t* __restrict__ cache_len, int32_t* __restrict__ overflow,
    T* __restrict__ k_cache, T* __restrict__ v_cache, int capacity, int Hkv, int ema, double gamma,
    int inclusive, int fusion, int warmup, float target, float eta,
    uint8_t* __restrict__ skip_out, float* __restrict__ fused_out, int32_t* __restrict__ tickets,
    int n_tickets)
{
    __shared__ double cosb[2][128];
    __shared__ int slot_s;
    const int b = blockIdx.x;
    const int grp = threadIdx.x >> 4, l16 = threadIdx.x & 15, n_grp = blockDim.x >> 4;
    const int t = seen[b];
    for (int i = threadIdx.x; i < n_tickets; i += blockDim.x) tickets[b * n_tickets + i] = 0;
    int n_skipped = 0, len = 0;
    float th_old = 0.f;
    if (threadIdx.x == 0) { n_skipped = skipped[b]; len = cache_len[b]; th_old = tau[b]; }
    // the anchor a row is compared with is f_a * state + f_x * row
    const int rows_in = inclusive ? t + 1 : t;
    const double f_a = ema ? (inclusive ? gamma : 1.0) : (rows_in > 0 ? 1.0 / (double)rows_in : 0.0);
    const double f_x = inclusive ? (ema ? 1.0 - gamma : f_a) : 0.0;

    typedef typename Raw2<T>::type Pair;
    Pair first[4] = {};   // the group's first row, kept for the cache
    for (int pr = grp; pr < 2 * Hkv; pr += n_grp) {
        const int w = pr >= Hkv, h = pr - w * Hkv;
        const long long off = ((long long)b * Hkv + h) * kHeadDim + 2 * l16;
        Pair row[4];
        double2 old[4];
        double2* const a = reinterpret_cast<double2*>((w ? anchor_v : anchor_k) + off);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            row[i] = *reinterpret_cast<const Pair*>((w ? v : k) + off + 32 * i);
            old[i] = a[16 * i];
        }
        double av[8];
        float x[8];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if (pr == grp) first[i] = row[i];
            av[2 * i] = old[i].x; av[2 * i + 1] = old[i].y;
            unpack2(row[i], x + 2 * i);
        }
        // the token is absorbed whatever is decided about it, and nobody else reads these columns
        auto absorbed = [&](int c) { return ema ? gamma * av[c] + (1.0 - gamma) * (double)x[c] : av[c] + (double)x[c]; };
#pragma unroll
        for (int i = 0; i < 4; ++i) a[16 * i] = make_double2(absorbed(2 * i), absorbed(2 * i + 1));
        double dot = 0.0, na = 0.0, nx = 0.0;
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            const double xc = (double)x[c], ac = fma(av[c], f_a, xc * f_x);
            dot = fma(ac, xc, dot);
            na = fma(ac, ac, na);
            nx = fma(xc, xc, nx);
        }
        dot = group16_sum(dot); na = group16_sum(na); nx = group16_sum(nx);
        double den = sqrt(na) * sqrt(nx);
        den = den < kEpsCos ? kEpsCos : den;
        double cs = dot / den;
        cs = cs > 1.0 ? 1.0 : (cs < -1.0 ? -1.0 : cs);
        if (l16 == 0) cosb[w][h] = cs;
    }
    __syncthreads();  // every read of seen[b] above precedes lane 0's update below

    if (threadIdx.x < 64) {
        // mean and population variance over the heads (two passes), one wave
        const int l = threadIdx.x;
        const double ck0 = l < Hkv ? cosb[0][l] : 0.0, cv0 = l < Hkv ? cosb[1][l] : 0.0;
        const double ck1 = l + 64 < Hkv ? cosb[0][l + 64] : 0.0, cv1 = l + 64 < Hkv ? cosb[1][l + 64] : 0.0;
        const double sk = wave_sum(ck0 + ck1) / (double)Hkv, sv = wave_sum(cv0 + cv1) / (double)Hkv;
        double dk = 0.0, dv = 0.0;
        if (l < Hkv) { dk = (ck0 - sk) * (ck0 - sk); dv = (cv0 - sv) * (cv0 - sv); }
        if (l + 64 < Hkv) { dk += (ck1 - sk) * (ck1 - sk); dv += (cv1 - sv) * (cv1 - sv); }
        const double ek = wave_sum(dk) / (double)Hkv + kEpsVar, ev = wave_sum(dv) / (double)Hkv + kEpsVar;
        if (l == 0) {
            const double alpha = fusion == 0 ? (1.0 / ev) / (1.0 / ek + 1.0 / ev)
                               : fusion == 1 ? (1.0 / ek) / (1.0 / ek + 1.0 / ev)
                               : fusion == 2 ? 1.0 : 0.0;
            const float S = (float)(alpha * sk + (1.0 - alpha) * sv);

            const float inv = t == 0 ? 0.0f : 1.0f / (float)t;
            const float p_current = (float)n_skipped * inv;
            const float diff = p_current - target;
            const float th = fmaf(eta, diff, th_old);
            int skip = (t >= warmup) && (S > th);
            int slot = -1;
            if (!skip) {
                if (len >= capacity) { overflow[b] = 1; skip = 1; }  // handled as skipped
                else { slot = len; cache_len[b] = len + 1; }
            }
            tau[b] = th;
            seen[b] = t + 1;
            skipped[b] = n_skipped + skip;
            skip_out[b] = (uint8_t)skip;
            fused_out[b] = S;
            slot_s = slot;
        }
    }
    __syncthreads();
    const int slot = slot_s;

    if (slot < 0) return;
    for (int pr = grp; pr < 2 * Hkv; pr += n_grp) {
        const int w = pr >= Hkv, h = pr - w * Hkv;
        const T* src = (w ? v : k) + ((long long)b * Hkv + h) * kHeadDim + 2 * l16;
        T* dst = (w ? v_cache : k_cache) + (((long long)b * Hkv + h) * capacity + slot) * kHeadDim + 2 * l16;
#pragma unroll
        for (int i = 0; i < 4; ++i)
            *reinterpret_cast<Pair*>(dst + 32 * i) = pr == grp ? first[i] : *reinterpret_cast<const Pair*>(src + 32 * i);
    }
}
#pragma clang fp contract(fast)

// The kernels of a step take their arguments as one block: a launch handles each argument by itself, and 40
// of them were 0.6 of a call's 6.5 us on the host.  (The bodies are functions of their own for the pointers'
// sake, which are known not to overlap as arguments only.)
template <typename T> struct ScoreArgs {
    const T *k, *v;
    double *anchor_k, *anchor_v;
    int32_t *seen, *skipped;
    float* tau;
    int32_t *cache_len, *overflow;
    T *k_cache, *v_cache;
    int capacity, Hkv, ema;
    double gamma;
    int inclusive, fusion, warmup;
    float target, eta;
    uint8_t* skip_out;
    float* fused_out;
    int32_t* tickets;
    int n_tickets;
};
template <typename T>
__global__ __launch_bounds__(1024) void decode_score_kernel(const ScoreArgs<T> a)
{
    score_row<T>(a.k, a.v, a.anchor_k, a.anchor_v, a.seen, a.skipped, a.tau, a.cache_len, a.overflow, a.k_cache, a.v_cache,
                 a.capacity, a.Hkv, a.ema, a.gamma, a.inclusive, a.fusion, a.warmup, a.target, a.eta, a.skip_out,
                 a.fused_out, a.tickets, a.n_tickets);
}

// sum over the four lanes that share lane % 16
__device__ __forceinline__ float wave_group_sum(float v)
{
    const FloatPair a = swap16(v, v);
    v = a.first + a.second;
    const FloatPair b = swap32(v, v);
    return b.first + b.second;
}
__device__ __forceinline__ float wave_group_max(float v)
{
    const FloatPair a = swap16(v, v);
    v = fmaxf(a.first, a.second);
    const FloatPair b = swap32(v, v);
    return fmaxf(b.first, b.second);
}

// Two floats to or from memory past the caches that are not shared between the dies (relaxed, device
// scope): written and read this way, a partial result needs no cache to be written back or
// invalidated on its way from one workgroup to another.
struct Float2 { float x, y; };
__device__ __forceinline__ void put_shared(float* p, Float2 v)
{
    __hip_atomic_store(reinterpret_cast<unsigned long long*>(p), __builtin_bit_cast(unsigned long long, v), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ Float2 get_shared(const float* p)
{
    return __builtin_bit_cast(Float2, __hip_atomic_load(reinterpret_cast<const unsigned long long*>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
}

// Behind a slice's partial result, which the workgroup has just written: the workgroup that draws the last
// ticket merges the `used` slices of its heads into the output rows.
template <typename T>
__device__ __forceinline__ void merge_slices(float* part0, T* out, float (*weight)[kDecodeMaxSplit + 1], int* drawn,
                                             int32_t* ticket, int heads, int used, int n_split)
{
    // every partial result of this workgroup is in memory before its ticket is drawn
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (threadIdx.x == 0) *drawn = __hip_atomic_fetch_add(ticket, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    if (*drawn != used - 1) return;

    // Numerators of the first kBatch slices of this thread's two columns, requested before their weights are
    // known (16 slices at a time, one column a thread: eight round trips to memory in a row with 64 slices of
    // four heads).  The last ones of a batch repeat a slice with weight 0, so few slices go in a small one (1
    // x 32 / 8 heads x 500 keys, four slices: 12.2 us a step in a batch of 32, 11.5 in one of eight).
    const int pairs = heads * kHeadDim / 2;
    auto merge = [&](auto batch) {
        constexpr int kBatch = decltype(batch)::value;
        Float2 x[kBatch];
        auto fetch = [&](int i, int l) {
            const float* pr = part0 + (long long)(i / (kHeadDim / 2)) * n_split * kPartStride + 2 * (i % (kHeadDim / 2));
#pragma unroll
            for (int u = 0; u < kBatch; ++u) x[u] = get_shared(pr + min(l + u, used - 1) * kPartStride);
        };
        if ((int)threadIdx.x < pairs) fetch(threadIdx.x, 0);
        // weights of the slices, per head, and their weighted sum behind them
        for (int g = threadIdx.x >> 6; g < heads; g += 4) {
            const int l = threadIdx.x & 63;
            Float2 own = {kLowest, 0.f};
            if (l < used) own = get_shared(part0 + ((long long)g * n_split + l) * kPartStride + kHeadDim);
            float m_all = own.x;
#pragma unroll
            for (int step = 1; step < 64; step *= 2) m_all = fmaxf(m_all, __shfl_xor(m_all, step));
            const float wt = __builtin_amdgcn_exp2f(own.x - m_all);
            float den = own.y * wt;
#pragma unroll
            for (int step = 1; step < 64; step *= 2) den += __shfl_xor(den, step);
            weight[g][l] = wt;   // 0 from `used` on
            if (l == 0) weight[g][kDecodeMaxSplit] = den;
        }
        __syncthreads();
        for (int i = threadIdx.x; i < pairs; i += 256) {
            const int g = i / (kHeadDim / 2), c = 2 * (i % (kHeadDim / 2));
            Float2 num = {0.f, 0.f};
            for (int l = 0; l < used; l += kBatch) {
                if (l > 0 || i >= 256) fetch(i, l);
#pragma unroll
                for (int u = 0; u < kBatch; ++u) {
                    num.x = fmaf(x[u].x, weight[g][l + u], num.x);
                    num.y = fmaf(x[u].y, weight[g][l + u], num.y);
                }
            }
            const float den = weight[g][kDecodeMaxSplit];
            store_out(out + g * kHeadDim + c, num.x / den);
            store_out(out + g * kHeadDim + c + 1, num.y / den);
        }
    };
    if (used <= 8) merge(std::integral_constant<int, 8>());
    else merge(std::integral_constant<int, 32>());
}

// Attention of the new token over one slice of its row's cache in fp32, for the G query heads that
// share a KV head.  A 16-lane group owns every 16th key of the slice and keeps its own running
// (max, sum, numerators), four keys at a time with the next four already requested; groups are
// merged through shuffles and LDS.  With one slice in use the result is final; with more, each slice
// leaves a partial result of kPartStride floats per query head, and the workgroup that draws the
// last ticket of its heads merges them (no order among the slices is assumed, and nobody
// waits).  A skipped row's first slice writes the zero row.
template <int G>
__global__ __launch_bounds__(256, G == 8 ? 2 : 1) void decode_attend_f32_kernel(
    const float* __restrict__ q, const float* __restrict__ k_cache, const float* __restrict__ v_cache,
    const int32_t* __restrict__ cache_len, const uint8_t* __restrict__ skip,
    float* __restrict__ part, int32_t* __restrict__ tickets, float* __restrict__ o, int Hq, int Hkv,
    int capacity, int n_split, float scale_log2e)
{
    __shared__ float merge[4][G][kPartStride];
    __shared__ float weight[G][kDecodeMaxSplit + 1];
    __shared__ int drawn;
    const int sp = blockIdx.x % n_split;
    const int hg = (blockIdx.x / n_split) % (Hq / G);  // group of G query heads
    const int b = blockIdx.x / n_split / (Hq / G);
    const int hq0 = hg * G, hk = hq0 / (Hq / Hkv);
    const int len = cache_len[b];
    const bool skipped = skip[b] != 0;
    const int grp = threadIdx.x >> 4, c8 = threadIdx.x & 15, wave = threadIdx.x >> 6;
    float* const out = o + ((long long)b * Hq + hq0) * kHeadDim;
    const long long row0 = ((long long)b * Hkv + hk) * capacity;
    const float* kb = k_cache + row0 * kHeadDim + c8 * 8;
    const float* vb = v_cache + row0 * kHeadDim + c8 * 8;
    // Slices are of at least kDecodeSlice keys, whatever the cache has room for, and the workgroups of those
    // without a key have nothing to do.  One row of 8 groups in a cache of 32768: 4 keys 20.8 -> 10.3 us a
    // step, 300 21.1 -> 13.8, 2000 22.7 -> 16.9, against 64 slices of which the most were empty.
    const int chunk = max(kDecodeSlice, ((len + n_split - 1) / n_split + 15) & ~15);
    const int lo = sp * chunk, hi = min(len, lo + chunk);
    if (skipped | (lo >= len)) {
        if (skipped && sp == 0)
            for (int i = threadIdx.x; i < G * kHeadDim; i += 256) store_out(out + i, 0.f);
        return;
    }

    float qf[G][8], acc[G][8], mx[G], sum[G];
#pragma unroll
    for (int g = 0; g < G; ++g) load8(q + ((long long)b * Hq + hq0 + g) * kHeadDim + c8 * 8, qf[g]);
#pragma unroll
    for (int g = 0; g < G; ++g) {
#pragma unroll
        for (int c = 0; c < 8; ++c) { qf[g][c] *= scale_log2e; acc[g][c] = 0.f; }
        mx[g] = kLowest; sum[g] = 0.f;
    }
    Raw8 k_raw[4], v_raw[4];
    auto request = [&](int j) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int ju = min(j + 16 * u, hi - 1);  // a valid row; its score is discarded below
            k_raw[u] = *reinterpret_cast<const Raw8*>(kb + (long long)ju * kHeadDim);
            v_raw[u] = *reinterpret_cast<const Raw8*>(vb + (long long)ju * kHeadDim);
        }
    };
    // (eight heads leave no registers for keys ahead: with them one workgroup is left on a compute unit)
    constexpr bool kAhead = G < 8;
    if (kAhead && lo + grp < hi) request(lo + grp);
    for (int j = lo + grp; j < hi; j += 64) {
        float kk[4][8], vv[4][8];
        if (!kAhead) request(j);
#pragma unroll
        for (int u = 0; u < 4; ++u) { unpack8(k_raw[u], kk[u]); unpack8(v_raw[u], vv[u]); }
        if (kAhead && j + 64 < hi) request(j + 64);
#pragma unroll
        for (int g = 0; g < G; ++g) {
            float s[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                float d = 0.f;
#pragma unroll
                for (int c = 0; c < 8; ++c) d = fmaf(qf[g][c], kk[u][c], d);
                d = row16_sum(d);
                s[u] = (j + 16 * u < hi) ? d : kLowest;
            }
            const float m_new = fmaxf(fmaxf(mx[g], fmaxf(s[0], s[1])), fmaxf(s[2], s[3]));
            const float scale_old = __builtin_amdgcn_exp2f(mx[g] - m_new);
            float p[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) p[u] = __builtin_amdgcn_exp2f(s[u] - m_new);
            sum[g] = fmaf(sum[g], scale_old, (p[0] + p[1]) + (p[2] + p[3]));
#pragma unroll
            for (int c = 0; c < 8; ++c) {
                float a = acc[g][c] * scale_old;
#pragma unroll
                for (int u = 0; u < 4; ++u) a = fmaf(p[u], vv[u][c], a);
                acc[g][c] = a;
            }
            mx[g] = m_new;
        }
    }

    // merge the four groups of a wave (lanes 16 and 32 apart), then the four waves through LDS
#pragma unroll
    for (int g = 0; g < G; ++g) {
        // (half swaps in the VALU; the exponent is at most 0)
        const float m_wave = wave_group_max(mx[g]);
        const float w_me = __builtin_amdgcn_exp2f(mx[g] - m_wave);
        mx[g] = m_wave;
        sum[g] = wave_group_sum(sum[g] * w_me);
#pragma unroll
        for (int c = 0; c < 8; ++c) acc[g][c] = wave_group_sum(acc[g][c] * w_me);
        if ((threadIdx.x & 63) < 16) {
#pragma unroll
            for (int c = 0; c < 8; ++c) merge[wave][g][c8 * 8 + c] = acc[g][c];
            if (c8 == 0) { merge[wave][g][kHeadDim] = mx[g]; merge[wave][g][kHeadDim + 1] = sum[g]; }
        }
    }
    __syncthreads();
    float* const part0 = part + ((long long)b * Hq + hq0) * n_split * kPartStride;   // [head][slice]
    constexpr int kPairs = kPartStride / 2;   // the last one: running max, sum
    for (int i = threadIdx.x; i < G * kPairs; i += 256) {
        const int g = i / kPairs, c = 2 * (i - g * kPairs);
        float m_all = kLowest;
#pragma unroll
        for (int w = 0; w < 4; ++w) m_all = fmaxf(m_all, merge[w][g][kHeadDim]);
        Float2 v = {0.f, 0.f};
        float den = 0.f;
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            const float wt = __builtin_amdgcn_exp2f(merge[w][g][kHeadDim] - m_all);
            v.x = fmaf(merge[w][g][c], wt, v.x);
            v.y = fmaf(merge[w][g][c + 1], wt, v.y);
            den = fmaf(merge[w][g][kHeadDim + 1], wt, den);
        }
        if (c == kHeadDim) v.x = m_all;
        if (len > chunk) put_shared(part0 + ((long long)g * n_split + sp) * kPartStride + c, v);
        else if (c < kHeadDim) { store_out(out + g * kHeadDim + c, v.x / den); store_out(out + g * kHeadDim + c + 1, v.y / den); }
    }
    if (len > chunk)
        merge_slices<float>(part0, out, weight, &drawn, &tickets[b * (Hq / G) + hg], G, (len + chunk - 1) / chunk, n_split);
}

// The same for bf16 rows, on the matrix pipe; a wave takes blocks of 32 keys.
//   S^T = K Q^T   v_mfma_f32_16x16x32_bf16, A = 16 rows of K as they lie in memory, B = the queries (column c:
//                 head c % G of the group, the last one again where it has fewer than G), so a lane has the
//                 scores of one head for eight keys.
//   O^T += V^T P^T  A: a lane loads 8 columns of the eight keys whose weights it holds (the contraction order
//                 over keys is the one in which they come out of the first product) and transposes them
//                 within its own registers; the 16 columns of product i are 8 c + i.
//   weights       stay fp32: a weight is the exact sum of three bf16 parts (8 bits of the mantissa each), and
//                 the parts of a head's weight are columns of their own of P^T (column c: part c / G), which
//                 with one to five heads are there anyway.  Their products with V are added up in fp32 at the
//                 end.  (An infinite value meets parts that are zero: where the products of whole weights
//                 gave an infinity, these give no number.  Non-finite inputs are outside the contract.)
// What bounds it is the way of the keys from memory, and for short rows the first loads (2 to 4 us) and the
// merge (6 us).  In fp32 on the vector pipe, as above, 480 instructions a wave went into 16 keys of four
// heads, 2 us for 64 keys with two workgroups on a compute unit.  A step with a kept token, scoring included
// (half of the tokens to be skipped): 1 x 32 / 8 heads x 2000, 16384 and 32768 keys 16.0, 29.7, 36.7 -> 12.9,
// 21.6, 29.9 us; 8 x 32 / 8 x 2048 26.1 -> 21.2; 1 x 32 / 32 x 2048 22.6 -> 14.7; 8 x 32 / 32 x 2048 52.7 ->
// 49.6, 47.2 if all rows are known to attend.  Distance from 64 bits as before (1.65e-3, the rounding of the
// output).
template <int G, bool FULL>
__device__ __forceinline__ void attend_bf16(
    const uint16_t* __restrict__ q, const uint16_t* __restrict__ k_cache, const uint16_t* __restrict__ v_cache,
    const int32_t* __restrict__ cache_len, const uint8_t* __restrict__ skip,
    float* __restrict__ part, int32_t* __restrict__ tickets, uint16_t* __restrict__ o, int B, int Hq, int Hkv,
    int parts, int per, int capacity, int n_few, int n_split, float scale_log2e)
{
    constexpr bool kTwice = 3 * G > 16;              // the third parts get a product of their own
    constexpr int kCols = kTwice ? 2 * G : 3 * G;    // columns of O^T in use
    constexpr int kRow = kHeadDim + 4;
    __shared__ __attribute__((aligned(16))) float o_part[4][kCols][kRow];
    __shared__ float stat[4][G][2];                  // a wave's running max and sum
    __shared__ float weight[G][kDecodeMaxSplit + 1];
    __shared__ int drawn;
    const int lane = threadIdx.x & 63, c16 = lane & 15, g4 = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // Groups of query heads: G of them (FULL), or at most G, the heads of a KV head in `parts` groups of `per`
    // and the last one of what is left.
    const int groups = FULL ? Hq / G : Hkv * parts, ratio = Hq / Hkv;
    auto first_head = [&](int hg) { return FULL ? hg * G : hg / parts * ratio + hg % parts * per; };
    auto heads_of = [&](int hg) { return FULL ? G : min(per, ratio - hg % parts * per); };
    // The workgroups are dealt out to the rows that attend: where skipped rows have a share of the grid,
    // their places on the compute units stay empty (16 steps of 8 x 32 / 32 heads x 2048 keys with about half
    // of the rows skipped: 533 us, 506 dealt out; of 8 x 32 / 8 280 and 275).
    const bool dealt = B <= kDecodeDealt;
    const int lane_row = min(lane, B - 1), lane_len = dealt ? cache_len[lane_row] : 0;
    const bool attends = dealt && lane < B && skip[lane_row] == 0;
    const unsigned long long rows = __ballot(attends);
    // zero rows, by the first workgroups of the grid
    if (blockIdx.x < B * groups) {
        const int zb = blockIdx.x / groups, zg = blockIdx.x % groups;
        if (dealt ? !(rows >> zb & 1) : skip[zb] != 0)
            for (int i = threadIdx.x; i < heads_of(zg) * kHeadDim; i += 256)
                o[((long long)zb * Hq + first_head(zg)) * kHeadDim + i] = 0;
    }
    // first the n_few slices that every row has, then those that only long rows have
    int at = blockIdx.x, slices = n_few, sp = 0;
    if (const int of_all = (dealt ? __popcll(rows) : B) * groups * n_few; at >= of_all) {
        if (n_split == n_few) return;
        at -= of_all;
        slices = n_split - n_few;
        sp = n_few;
    }
    sp += at % slices;
    const int hg = at / slices % groups;
    int b = at / slices / groups, len;
    if (dealt) {   // the b-th row that attends
        const unsigned long long here = __ballot(attends && __popcll(rows & ((1ull << lane) - 1)) == b);
        if (here == 0) return;
        b = __builtin_ctzll(here);
        len = __shfl(lane_len, b);
    } else {
        if (b >= B || skip[b] != 0) return;
        len = cache_len[b];
    }
    len = __builtin_amdgcn_readfirstlane(len);
    const int hq0 = first_head(hg), hk = hq0 / ratio, heads = heads_of(hg);
    uint16_t* const out = o + ((long long)b * Hq + hq0) * kHeadDim;
    const long long row0 = ((long long)b * Hkv + hk) * capacity;
    const uint16_t* kb = k_cache + row0 * kHeadDim + 8 * g4;
    const uint16_t* vb = v_cache + row0 * kHeadDim + 8 * c16;
    // How a row is sliced follows from its own length, not from the other rows, and so do its bits.
    const int n_row = len >= n_split * kDecodeLongSlice ? n_split : n_few;
    const int chunk = max(kDecodeSliceBf16, ((len + n_row - 1) / n_row + 31) & ~31);
    const int lo = sp * chunk, hi = min(len, lo + chunk);
    if (lo >= len) return;

    u32x4 k_raw[2][4], v_raw[8];
    auto request_k = [&](int j) {   // (past the end: the last row again, its scores are masked)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const uint16_t* row = kb + (long long)min(j + 16 * h + c16, hi - 1) * kHeadDim;
#pragma unroll
            for (int s = 0; s < 4; ++s) k_raw[h][s] = *reinterpret_cast<const u32x4*>(row + 32 * s);
        }
    };
    auto request_v = [&](int j) {
#pragma unroll
        for (int e = 0; e < 8; ++e)
            v_raw[e] = *reinterpret_cast<const u32x4*>(vb + (long long)min(j + 16 * (e >> 2) + 4 * g4 + (e & 3), hi - 1) * kHeadDim);
    };
    // A wave's blocks in turn, each KV head from another one on: workgroups that walk caches side by side in
    // step meet in the same memory channels at some distances of the caches (8 x 32 / 32 heads x 2048 keys
    // from memory: 70 us a step in caches of 2064 rows, 58 to 62 in others; like this 62 in all of them).
    const int first = lo + 32 * wave, blocks = max(0, (hi - first + 127) / 128);
    int j = blocks ? first + 128 * (hk % blocks) : hi;
    if (blocks) { request_k(j); request_v(j); }
    bf16x8 qf[4];
#pragma unroll
    for (int s = 0; s < 4; ++s)
        qf[s] = *reinterpret_cast<const bf16x8*>(q + ((long long)b * Hq + hq0 + (FULL ? c16 % G : min(c16 % G, heads - 1))) * kHeadDim + 32 * s + 8 * g4);
    f32x4 acc[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) acc[i] = f32x4{0.f, 0.f, 0.f, 0.f};
    float mx = kLowest, sum = 0.f;
    for (int left = blocks; left > 0; --left) {
        const int next = j + 128 < hi ? j + 128 : first;
        float s[8];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            f32x4 d = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int t = 0; t < 4; ++t)
                d = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, k_raw[h][t]), qf[t], d, 0, 0, 0);
#pragma unroll
            for (int v = 0; v < 4; ++v) s[4 * h + v] = j + 16 * h + 4 * g4 + v < hi ? d[v] * scale_log2e : kLowest;
        }
        if (left > 1) request_k(next);
        const float top = wave_group_max(fmaxf(fmaxf(fmaxf(s[0], s[1]), fmaxf(s[2], s[3])), fmaxf(fmaxf(s[4], s[5]), fmaxf(s[6], s[7]))));
        if (__any(top > mx)) {
            const float m_new = fmaxf(mx, top), down = __builtin_amdgcn_exp2f(mx - m_new);
            mx = m_new;
            sum *= down;
#pragma unroll
            for (int i = 0; i < 8; ++i) acc[i] *= down;
        }
        u32x4 p1, p2;   // weights: the parts of this lane's column, and the third parts if they go by themselves
#pragma unroll
        for (int e = 0; e < 8; e += 2) {
            unsigned x[2], y[2];
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const float p = __builtin_amdgcn_exp2f(s[e + i] - mx);
                sum += p;
                const float r1 = p - __uint_as_float(__float_as_uint(p) & 0xffff0000u);    // without the first part
                const float r2 = r1 - __uint_as_float(__float_as_uint(r1) & 0xffff0000u);  // without the second
                x[i] = __float_as_uint(c16 < G ? p : c16 < 2 * G ? r1 : kTwice || c16 >= 3 * G ? 0.f : r2);
                y[i] = __float_as_uint(c16 < G ? r2 : 0.f);
            }
            p1[e / 2] = __builtin_amdgcn_perm(x[1], x[0], 0x07060302u);
            if (kTwice) p2[e / 2] = __builtin_amdgcn_perm(y[1], y[0], 0x07060302u);
        }
        bf16x8 vt[8];   // column 8 c16 + i of the lane's eight keys
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            u32x4 t;
#pragma unroll
            for (int e = 0; e < 4; ++e)
                t[e] = __builtin_amdgcn_perm(v_raw[2 * e + 1][i / 2], v_raw[2 * e][i / 2], i & 1 ? 0x07060302u : 0x05040100u);
            vt[i] = __builtin_bit_cast(bf16x8, t);
        }
        if (left > 1) request_v(next);
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            acc[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vt[i], __builtin_bit_cast(bf16x8, p1), acc[i], 0, 0, 0);
            if (kTwice) acc[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vt[i], __builtin_bit_cast(bf16x8, p2), acc[i], 0, 0, 0);
        }
        j = next;
    }

    // the four waves' results through LDS (register v of product i is column 8 (4 g4 + v) + i)
    sum = wave_group_sum(sum);
    if (c16 < kCols)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            float* dst = &o_part[wave][c16][8 * (4 * g4 + v)];
            *reinterpret_cast<f32x4*>(dst) = f32x4{acc[0][v], acc[1][v], acc[2][v], acc[3][v]};
            *reinterpret_cast<f32x4*>(dst + 4) = f32x4{acc[4][v], acc[5][v], acc[6][v], acc[7][v]};
        }
    if (lane < G) { stat[wave][lane][0] = mx; stat[wave][lane][1] = sum; }
    __syncthreads();
    float* const part0 = part + ((long long)b * Hq + hq0) * n_split * kPartStride;   // [head][slice]
    constexpr int kPairs = kPartStride / 2;   // the last one: running max, sum
    auto combine = [&](auto n_waves) {
        for (int i = threadIdx.x; i < heads * kPairs; i += 256) {
            const int g = i / kPairs, c = 2 * (i - g * kPairs);
            float m_all = kLowest;
#pragma unroll
            for (int w = 0; w < n_waves; ++w) m_all = fmaxf(m_all, stat[w][g][0]);
            Float2 v = {0.f, 0.f};
            float den = 0.f;
#pragma unroll
            for (int w = 0; w < n_waves; ++w) {
                const float wt = __builtin_amdgcn_exp2f(stat[w][g][0] - m_all);
                den = fmaf(stat[w][g][1], wt, den);
                if (c == kHeadDim) continue;
                Float2 n = {o_part[w][G + g][c], o_part[w][G + g][c + 1]};
                if (!kTwice) {
                    constexpr int third = kTwice ? 0 : 2 * G;
                    n.x += o_part[w][third + g][c];
                    n.y += o_part[w][third + g][c + 1];
                }
                v.x = fmaf(n.x + o_part[w][g][c], wt, v.x);
                v.y = fmaf(n.y + o_part[w][g][c + 1], wt, v.y);
            }
            if (c == kHeadDim) v = {m_all, den};
            if (len > chunk) put_shared(part0 + ((long long)g * n_split + sp) * kPartStride + c, v);
            else if (c < kHeadDim) { store_out(out + g * kHeadDim + c, v.x / den); store_out(out + g * kHeadDim + c + 1, v.y / den); }
        }
    };
    // (up to 32 keys are one wave's)
    if (hi - lo <= 32) combine(std::integral_constant<int, 1>());
    else combine(std::integral_constant<int, 4>());
    if (len > chunk)
        merge_slices<uint16_t>(part0, out, weight, &drawn, &tickets[b * groups + hg], heads, (len + chunk - 1) / chunk, n_split);
}

struct AttendArgs {
    const uint16_t *q, *k_cache, *v_cache;
    const int32_t* cache_len;
    const uint8_t* skip;
    float* part;
    int32_t* tickets;
    uint16_t* o;
    int B, Hq, Hkv, parts, per, capacity, n_few, n_split;
    float scale_log2e;
};
template <int G, bool FULL>
__global__ __launch_bounds__(256, 2) void decode_attend_bf16_kernel(const AttendArgs a)
{
    attend_bf16<G, FULL>(a.q, a.k_cache, a.v_cache, a.cache_len, a.skip, a.part, a.tickets, a.o, a.B, a.Hq, a.Hkv, a.parts,
                   a.per, a.capacity, a.n_few, a.n_split, a.scale_log2e);
}

// Hand-off from the batched path: the anchors as they stand after all n rows of a prompt.
// One workgroup per (tensor, batch row, KV head) and 8 * LANES columns: a group of LANES lanes folds
// every (1024 / LANES)-th row in Horner form, A <- g^stride A + x (g = 1 for the exact mean, whose
// state is the plain sum), brings its partial to the end of the prompt with g^(rows after its last
// one), and the partials are added through shuffles and LDS.  All in double.  Rows further back
// than `window` from the end are skipped (the incremental anchor forgets them: g^window is far
// below double resolution).
// What bounds it is the latency of a thread's loads, one row after the other, so the rows are spread
// over many groups and four are in flight per group; with few chains (LANES = 4: a quarter of the
// columns each) there are four times the workgroups.  16 chains x 3001 rows: 62 -> 9 us against
// 16 groups of 16 lanes.
// The workgroups behind those `anchors` copy 64 kept rows of K and V each, in order, into the caches and
// set the controller's counters (5 us when they were a launch of their own; neither part fills the chip).
template <typename T, int LANES>
__global__ __launch_bounds__(1024) void decode_seed_kernel(
    const T* __restrict__ K, const T* __restrict__ V, double* __restrict__ anchor_k,
    double* __restrict__ anchor_v, int Hkv, int n, long long s_b, long long s_h, long long s_t,
    double g, double weight, int window, int anchors, const int32_t* __restrict__ kept_idx,
    const int32_t* __restrict__ count, T* __restrict__ k_cache, T* __restrict__ v_cache,
    int32_t* __restrict__ seen, int32_t* __restrict__ skipped, int32_t* __restrict__ cache_len,
    int32_t* __restrict__ overflow, int capacity)
{
    if ((int)blockIdx.x >= anchors) {
        const int row_blocks = (n + 63) / 64, rb = (blockIdx.x - anchors) % row_blocks;
        const int bh = (blockIdx.x - anchors) / row_blocks, b = bh / Hkv, h = bh % Hkv;
        const int m = count[b];
        if (rb == 0 && h == 0 && threadIdx.x == 0) {
            seen[b] = n; skipped[b] = n - m; cache_len[b] = m; overflow[b] = 0;
        }
        const int i = rb * 64 + (threadIdx.x >> 4), c8 = threadIdx.x & 15;
        if (i >= m) return;
        const long long src = b * s_b + h * s_h + (long long)kept_idx[(long long)b * n + i] * s_t + c8 * 8;
        const long long dst = ((long long)bh * capacity + i) * kHeadDim + c8 * 8;
        copy8(k_cache + dst, K + src);
        copy8(v_cache + dst, V + src);
        return;
    }
    constexpr int kGroups = 1024 / LANES, kParts = 16 / LANES;   // row groups; workgroups per chain
    __shared__ double part[16][8 * LANES];
    const int q = blockIdx.x % kParts, chain = blockIdx.x / kParts;
    const int w = chain & 1, bh = chain >> 1;
    const int b = bh / Hkv, h = bh % Hkv;
    const int grp = threadIdx.x / LANES, c8 = threadIdx.x % LANES;
    const T* X = (w ? V : K) + b * s_b + h * s_h + (q * LANES + c8) * 8;
    double g_step = g;
    for (int i = 1; i < kGroups; i *= 2) g_step *= g_step;
    double a[8];
#pragma unroll
    for (int c = 0; c < 8; ++c) a[c] = 0.0;
    const int j0 = (n - window > 0 ? n - window : 0);
    int last = -1;
    for (int j = j0 + grp; j < n; j += 4 * kGroups) {
        float x[4][8];
#pragma unroll
        for (int u = 0; u < 4; ++u) load8(X + (long long)min(j + u * kGroups, n - 1) * s_t, x[u]);
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (j + u * kGroups < n) {
#pragma unroll
                for (int c = 0; c < 8; ++c) a[c] = g_step * a[c] + (double)x[u][c];
                last = j + u * kGroups;
            }
    }
    double tail = last >= 0 ? weight : 0.0;  // weight * g^(n - 1 - last)
    double pw = g;
    for (int e = last >= 0 ? n - 1 - last : 0; e > 0; e >>= 1) {
        if (e & 1) tail *= pw;
        pw *= pw;
    }
#pragma unroll
    for (int c = 0; c < 8; ++c) {
        double v = a[c] * tail;
#pragma unroll
        for (int step = LANES; step < 64; step *= 2) v += __shfl_xor(v, step);
        if ((threadIdx.x & 63) < LANES) part[threadIdx.x >> 6][c8 * 8 + c] = v;
    }
    __syncthreads();
    if (threadIdx.x < 8 * LANES) {
        double sum = 0.0;
#pragma unroll
        for (int i = 0; i < 16; ++i) sum += part[i][threadIdx.x];
        (w ? anchor_v : anchor_k)[(long long)bh * kHeadDim + q * 8 * LANES + threadIdx.x] = sum;
    }
}

template <typename T>
hipError_t launch_decode_seed_t(const DecodeArgs& a, const T* K, const T* V, const int32_t* kept_idx,
                                const int32_t* count, int n, const long long* kvs, hipStream_t s)
{
    const double g = a.ema ? a.gamma : 1.0;
    // rows that still matter to the incremental anchor: g^window <= 1e-40
    int window = n;
    if (a.ema) {
        const double rows = g > 0.0 ? ceil(-92.2 / log(g)) : 1.0;
        window = rows < (double)n ? (int)rows : n;
    }
    const double wt = a.ema ? 1.0 - a.gamma : 1.0;
    const int chains = 2 * a.B * a.Hkv;
    // below one workgroup per two compute units a chain's columns are shared out
    const int anchors = chains < 128 ? 4 * chains : chains;
    const unsigned grid = (unsigned)anchors + (unsigned)((n + 63) / 64) * a.B * a.Hkv;
#define TF_DECODE_SEED(LANES)                                                                     \
    decode_seed_kernel<T, LANES><<<dim3(grid), dim3(1024), 0, s>>>(                               \
        K, V, a.anchor_k, a.anchor_v, a.Hkv, n, kvs[0], kvs[1], kvs[2], g, wt, window, anchors, kept_idx, \
        count, (T*)a.k_cache, (T*)a.v_cache, a.seen, a.skipped, a.cache_len, a.overflow, a.capacity)
    if (chains < 128) TF_DECODE_SEED(4);
    else TF_DECODE_SEED(16);
#undef TF_DECODE_SEED
    return hipGetLastError();
}

template <typename T>
hipError_t launch_decode_step_t(const DecodeArgs& a, const T* q, const T* k, const T* v, T* o,
                                hipStream_t s)
{
    const int threads = std::min(1024, (32 * a.Hkv + 63) / 64 * 64);  // 16 lanes per (tensor, head)
    const int g = decode_heads_per_wg(sizeof(T) == 2, a.B, a.Hq, a.Hkv);
    const int ratio = a.Hq / a.Hkv, parts = (ratio + g - 1) / g, groups = a.Hkv * parts;
    // tickets of the attention's workgroups behind the partial results
    int32_t* const tickets = (int32_t*)(a.part + (size_t)a.B * a.Hq * a.n_split * kDecodePartFloats);
    decode_score_kernel<T><<<dim3(a.B), dim3(threads), 0, s>>>(ScoreArgs<T>{
        k, v, a.anchor_k, a.anchor_v, a.seen, a.skipped, a.tau, a.cache_len, a.overflow,
        (T*)a.k_cache, (T*)a.v_cache, a.capacity, a.Hkv, a.ema, a.gamma, a.inclusive, a.fusion, a.warmup,
        a.target, a.eta, a.skip, a.fused, tickets, a.n_split > 1 ? groups : 0});
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const float sl2 = a.scale * 1.4426950408889634f;
#define TF_DECODE_ATTEND(G, FULL)                                                                 \
    do {                                                                                          \
        if constexpr (sizeof(T) == 2)                                                             \
            decode_attend_bf16_kernel<G, FULL><<<dim3(grid), dim3(256), 0, s>>>(                  \
                AttendArgs{q, k_cache, v_cache, a.cache_len, a.skip, a.part, tickets, o, a.B, a.Hq, a.Hkv, parts,     \
                           (ratio + parts - 1) / parts, a.capacity, a.n_few, a.n_split, sl2});    \
        else                                                                                      \
            decode_attend_f32_kernel<G><<<dim3(grid), dim3(256), 0, s>>>(                         \
                q, k_cache, v_cache, a.cache_len, a.skip, a.part, tickets, o, a.Hq, a.Hkv,        \
                a.capacity, a.n_split, sl2);                                                      \
    } while (0)
    const T *k_cache = (const T*)a.k_cache, *v_cache = (const T*)a.v_cache;
    const int grid = a.B * groups * a.n_split;
    if (ratio % g != 0) {   // bf16: some workgroups have fewer heads
        if (g == 8) TF_DECODE_ATTEND(8, false);
        else TF_DECODE_ATTEND(4, false);
    } else if (g == 8) TF_DECODE_ATTEND(8, true);
    else if (g == 4) TF_DECODE_ATTEND(4, true);
    else if (g == 2) TF_DECODE_ATTEND(2, true);
    else TF_DECODE_ATTEND(1, true);
#undef TF_DECODE_ATTEND
    return hipGetLastError();
}

}  // namespace

int decode_heads_per_wg(bool bf16, int B, int Hq, int Hkv)
{
    const int ratio = Hq / Hkv;
    // Heads that share a KV head share workgroups, whatever their number: one by one each reads the cache for
    // itself (a step of 1 x 128 / 8 heads x 5000 keys: 33.6 us, 16.8 by fours; 8 x 40 / 8 x 2000: 55 and 23;
    // 4 x 71 / 1 x 2000: 37 and 20; below some 500 keys one by one is up to 0.5 us faster).  More than four
    // go by eights, but by fours where few caches are read: the slices of four are merged in half the time (1
    // x 16 / 2 x 16384: 20.2 by eights, 17.7 by fours; 1 x 64 / 8 x 4000: 17.6 and 15.9; 8 x 28 / 4 x 2000:
    // 20.0 and 18.4; but 8 x 64 / 8 x 4000: 33.8 and 48.5; 16 x 48 / 8 x 2000: 32.6 and 48; fp32 16 x 64 / 8
    // x 4000: 108 and 159).
    if (bf16 && ratio > 2) return ratio <= 4 || B * Hkv < 48 ? 4 : 8;
    if (ratio == 8) return B * Hkv < 48 ? 4 : 8;
    return ratio == 2 || ratio == 4 ? ratio : 1;   // (fp32, other ratios: one by one)
}

// Slices of each of `rows` caches that a step reads.
static int decode_slices(int rows, int n_cu)
{
    // One workgroup on a compute unit has enough keys under way, and a merge of more slices costs more than
    // more workgroups bring (a step of 1 x 32 / 8 heads x 16384 keys: 24.9 us with 512, 21.5 with 256; 1 x 32
    // / 32 x 2048: 18.9, 16.0 and 15.2 with 1024, 512 and 256; 8 x 32 / 32 x 256: 19.0, 15.1 and 13.0).
    // Where rows do not fill whole rounds of the compute units, the fewest slices that come within a tenth of
    // even shares, in up to four rounds (8 x 40 / 40 x 2048, 320 rows: 73.7 us with 320 workgroups, 68.1 with
    // 640, 65.1 with 960).
    const int most = std::min(kDecodeMaxSplit, 4 * n_cu / rows);
    int split = std::min(kDecodeMaxSplit, std::max(1, n_cu / rows));
    int busiest = (rows * split + n_cu - 1) / n_cu;   // workgroups of the busiest compute unit
    for (int n = split + 1; n <= most && 10 * busiest * n_cu > 11 * rows * split; ++n) {
        const int of_n = (rows * n + n_cu - 1) / n_cu;
        if (of_n * split < busiest * n) { split = n; busiest = of_n; }
    }
    return split;
}

DecodeSplit decode_split(bool bf16, int B, int Hq, int Hkv, double target, int n_cu)
{
    const int g = decode_heads_per_wg(bf16, B, Hq, Hkv), groups = Hkv * ((Hq / Hkv + g - 1) / g), rows = B * groups;
    if (bf16) {
        // By the batch rows that attend on average: by those that do attend in a step, a row's rounding would
        // depend on its neighbours.  Where the number varies from step to step whole rounds are not worth
        // more slices (16 steps of 8 x 40 / 40 x 2048, half of the rows skipped: 586 us with one slice, 618
        // with three; 8 x 32 / 32 x 2048, a quarter: 600 with one, 687 with four; 16 x 32 / 32 x 1024, a
        // quarter: 628 with one, 681 with two), but they are where only one row now and then leaves a second
        // round (8 x 40 / 40 x 2048, a tenth: 1052 and 961).
        const int attending = std::max(1, (int)lround(B * (1.0 - target))), caches = attending * groups;
        const bool steady = attending == B || (attending == B - 1 && caches > n_cu);
        const int few = steady ? decode_slices(caches, n_cu) : std::min(kDecodeMaxSplit, std::max(1, n_cu / caches));
        // Long rows, where merging costs little beside the keys, get a round of the compute units for each batch
        // row if they can, so that whole rounds are walked whatever attends (16 steps, 8 x 32 / 32 x 8000, half
        // of the rows skipped: 1732 us with two slices, 1656 with eight; 2 x 40 / 40 x 20000, a quarter: 1967
        // with three, 1881 with six; at 704 keys a slice they are even: 3 x 32 / 32 x 5000 565 with four and
        // 572 with eight slices, x 6000 677 and 659; 8 x 32 / 8 x 8000 491 with 8 and 579 with 32).
        const bool varies = B > 1 && target > 0.0;
        return {few, varies ? std::max(few, std::min(4 * few, decode_slices(groups, n_cu))) : few};
    }
    // fp32: two workgroups a compute unit where they take four or eight heads, as many as are resident at
    // once (224 and 249 registers); four where they take one or two, which is more than the three and two
    // that are (164 and 186): many rows gain from it what they lose in rounds, few do not (16 steps with half
    // of the rows skipped, one / two / three / four a compute unit: 8 x 40 / 40 heads x 2000 keys 1270, 1215,
    // 1134, 1120 us; 8 x 32 / 32 x 1000 451, 489, 502, 482; 1 x 32 / 32 x 4000 296, 299, 303, 319; 1 x 32 /
    // 16 x 6000 249, 253, 294, 315; 4 x 32 / 8 x 2000 with one and two 274, 283).
    const int n = std::min(kDecodeMaxSplit, std::max(1, ((g >= 4 ? 2 : 4) * n_cu + rows - 1) / rows));
    return {n, n};
}

size_t decode_scratch_bytes(bool bf16, int B, int Hq, int Hkv, double target)
{
    const size_t rows = (size_t)B * Hq;
    return (rows * decode_split(bf16, B, Hq, Hkv, target).most * kDecodePartFloats + rows) * sizeof(float);
}

hipError_t launch_decode_init(const DecodeArgs& a, float tau0, hipStream_t s)
{
    const long long n_anchor = (long long)a.B * a.Hkv * kHeadDim;
    const long long n = std::max<long long>(n_anchor, a.B);
    decode_init_kernel<<<dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s>>>(
        a.anchor_k, a.anchor_v, n_anchor, a.seen, a.skipped, a.tau, a.cache_len, a.overflow, a.B, tau0);
    return hipGetLastError();
}

hipError_t launch_decode_seed(const DecodeArgs& a, int dtype, const void* K, const void* V,
                              const int32_t* kept_idx, const int32_t* count, int n,
                              const long long* kvs, hipStream_t s)
{
    if (dtype == 0) return launch_decode_seed_t<float>(a, (const float*)K, (const float*)V, kept_idx, count, n, kvs, s);
    return launch_decode_seed_t<uint16_t>(a, (const uint16_t*)K, (const uint16_t*)V, kept_idx, count, n, kvs, s);
}

hipError_t launch_decode_step(const DecodeArgs& a, int dtype, const void* q, const void* k,
                              const void* v, void* o, hipStream_t s)
{
    if (dtype == 0)
        return launch_decode_step_t<float>(a, (const float*)q, (const float*)k, (const float*)v, (float*)o, s);
    return launch_decode_step_t<uint16_t>(a, (const uint16_t*)q, (const uint16_t*)k,
                                          (const uint16_t*)v, (uint16_t*)o, s);
}

}  // namespace tf
