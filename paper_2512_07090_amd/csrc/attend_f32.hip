// Causal softmax attention over the kept tokens (Section 3.2: filtered tokens get a zero
// attention output; the rest attend as usual, here to kept tokens only).  Queries and keys are
// addressed through kept_idx, so "causal" is "key rank <= query rank" in the compacted order.
//
//   zero_filtered_kernel  writes zero rows of O from a mask (a layer that filters every token);
//   attend_f32_kernel     fp32 on the matrix cores' fp32 form, zero rows included.
// The bf16 MFMA kernel lives in attend_bf16.hip.
#include "tf_kernels.h"
#include <algorithm>

namespace tf {

namespace {

// ------------------------------------------------------------------------------ zero rows
// 16 lanes per row (16 B each for bf16, 32 B for fp32), 16 rows per workgroup.
template <int ELEM_BYTES>
__global__ __launch_bounds__(256) void zero_filtered_kernel(Dims d, const uint8_t* __restrict__ keep,
                                                            char* __restrict__ O)
{
    const int pos = blockIdx.x * 16 + (threadIdx.x >> 4);
    const int hq = blockIdx.y, b = blockIdx.z;
    if (pos >= d.n || keep[(long long)b * d.n + pos]) return;
    char* row = O + ((long long)b * d.os[0] + (long long)hq * d.os[1] + (long long)pos * d.os[2]) * ELEM_BYTES;
    const int l = threadIdx.x & 15;
    const uint4 z = make_uint4(0, 0, 0, 0);
    if (ELEM_BYTES == 2) {
        reinterpret_cast<uint4*>(row)[l] = z;
    } else {
        reinterpret_cast<uint4*>(row)[l] = z;
        reinterpret_cast<uint4*>(row)[16 + l] = z;
    }
}

// ------------------------------------------------------------------------------ fp32 path
// One workgroup per 16 kept queries of a head: its four waves hold the same queries and take the
// 16-key blocks in turns, each with its own softmax state, and are merged through LDS at the end.
//   S^T = K Q^T       v_mfma_f32_16x16x4_f32, fp32 products and sums; lane group g = lane / 16 feeds
//                     k-slot g of step 4 j + e with column 16 j + 4 g + e, so a lane's operands are
//                     16-byte loads
//   O^T += V^T P^T    the accumulator of S^T (key 4 g + r of the block in register r, query lane % 16) is
//                     the B operand of step r as it stands; row i of the A operand's block db is
//                     column 8 i + db, so a lane reads 32 contiguous bytes of a V row and a
//                     16-lane group the whole row
// Keys and values go from the caches straight to registers (no two waves of a workgroup need the
// same ones): the next block's K is requested when the products have consumed this one's, V one
// block's scores ahead of its use.
// What bounds it: a block is 64 MFMAs of 32 cycles (1.7 times that in all at long rows: three waves a SIMD,
// limited by their registers, do not hide all of the softmax), at short rows one wave's latency chain. Plain FMAs on 32 x 32
// tiles in LDS with the zero rows in a launch of their own against this: 32 heads x 256 kept
// tokens of 512 75 -> 18 us, 40 x 1350 of 1500 856 -> 215 us, distance from 64 bits 3.0e-7 -> 2.0e-7 (fewer
// roundings in a row). 32 queries a workgroup halve the loads but take 346 us there (two waves a SIMD).
typedef float f32x4 __attribute__((ext_vector_type(4)));
constexpr float kNone = -1e30f;   // masked score, and the maximum of a row without keys

// Workgroups of a tile: where few tokens are kept its zero rows are more than one should write.
__host__ __device__ __forceinline__ int zero_parts(int n, int m)
{
    const int parts = n / (32 * m);
    return parts < 1 ? 1 : (parts > 64 ? 64 : parts);
}

__device__ __forceinline__ float across_groups_max(float v)
{
    const FloatPair a = swap16(v, v);
    v = fmaxf(a.first, a.second);
    const FloatPair b = swap32(v, v);
    return fmaxf(b.first, b.second);
}
__device__ __forceinline__ float across_groups_sum(float v)
{
    const FloatPair a = swap16(v, v);
    v = a.first + a.second;
    const FloatPair b = swap32(v, v);
    return b.first + b.second;
}

__global__ __launch_bounds__(256, 3) void attend_f32_kernel(Dims d, float scale,
                                                         const float* __restrict__ Q,
                                                         const float* __restrict__ K,
                                                         const float* __restrict__ V,
                                                         const int32_t* __restrict__ kept_idx,
                                                         float* __restrict__ O,
                                                         const int32_t* __restrict__ counts,
                                                         long long idx_stride, int parts, int ranks, unsigned line)
{
    constexpr int kRows = 16, kStride = kHeadDim + 4;
    __shared__ __attribute__((aligned(16))) float part[4][kRows][kStride];
    __shared__ float part_m[4][kRows], part_l[4][kRows];
    __shared__ int tile_pos[kRows + 1];

    // The longest tiles of all heads first, so that they spread over the dies and the short ones fill in behind
    // them (head by head, 32 heads x 256 kept tokens took 21.3 instead of 17.6 us, 8 x 32 x 125 45 instead of 35); of the `parts` workgroups of
    // a tile the others only help with its zero rows.
    // Workgroups lie in lines of `line`, `ranks` of them per head.
    const unsigned id = blockIdx.y * line + blockIdx.x, groups = d.B * d.Hq;
    const int bh = id % groups, rank = id / groups;
    if (rank >= ranks) return;   // behind the last one in the last line
    int qt = (ranks - 1 - rank) / parts, zp = rank % parts;
    const int hq = bh % d.Hq, b = bh / d.Hq;
    const int hk = hq / (d.Hq / d.Hkv);
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int c16 = lane & 15, g = lane >> 4;
    // kept tokens of this batch row (per row when counts is given: d.m is then the bound)
    const int m = counts ? counts[b] : d.m;
    float* Ob = O + (long long)b * d.os[0] + (long long)hq * d.os[1];
    const float4 zero = make_float4(0.f, 0.f, 0.f, 0.f);
    if (m == 0) {
        // a row without kept tokens (its grid is the one of a full row): every output row is zero
        for (int r = qt * kRows + (tid >> 5); r < min(qt * kRows + kRows, d.n); r += 8)
            reinterpret_cast<float4*>(Ob + (long long)r * d.os[2])[tid & 31] = zero;
        return;
    }
    if (counts) {
        // the workgroups that the row's tiles leave over (its grid is the one of a full row) help with their zero rows:
        // with one workgroup a tile, 32 heads x 16384 with 16 kept took 191 us, 70 with them (a mask and a launch of its own: 78)
        const int tiles = (m + kRows - 1) / kRows;
        parts = min(zero_parts(d.n, m), ranks / tiles);
        if (rank >= tiles * parts) return;
        qt = tiles - 1 - rank % tiles;
        zp = rank / tiles;
    }
    const int i0 = qt * kRows;
    const int32_t* idx = kept_idx + (long long)b * idx_stride;
    const float* Qb = Q + (long long)b * d.qs[0] + (long long)hq * d.qs[1];
    const float* Kb = K + (long long)b * d.kvs[0] + (long long)hk * d.kvs[1];
    const float* Vb = V + (long long)b * d.kvs[0] + (long long)hk * d.kvs[1];
    const int i_last = min(i0 + kRows, m) - 1;
    const int n_blocks = i_last / 16 + 1;
    // positions of the tile's queries and of the kept token after them (or the row's end)
    if (tid <= kRows) tile_pos[tid] = i0 + tid < m ? idx[i0 + tid] : d.n;
    // The filtered positions behind each query of the tile (and before the first one) are zero rows, written
    // without a look at the gaps one by one: with z_i = the zero rows before query i of the tile, the k-th one
    // sits at position_0 + 1 + k + #{i >= 1 : z_i <= k}, and the count is a ballot.  (After a barrier.)
    const int col = 4 * (tid & 31);   // 32 threads a row, four columns each
    auto zero_rows = [&]() {
        const int n_q = i_last - i0 + 1, half = lane >> 5, qi = lane & 31;
        const int first = tile_pos[0], n_zero = tile_pos[n_q] - first - n_q;
        const int z_mine = qi >= 1 && qi < n_q ? tile_pos[qi] - first - qi : 0x7fffffff;
        for (int k0 = 8 * zp + 2 * wave; k0 < n_zero; k0 += 8 * parts) {
            const int k = k0 + half;
            const unsigned long long below = __ballot(z_mine <= k);
            const int p = first + 1 + k + __popc((unsigned)(below >> (32 * half)));
            if (k < n_zero) *reinterpret_cast<float4*>(Ob + (long long)p * d.os[2] + col) = zero;
        }
        if (i0 == 0)
            for (int z = 8 * zp + (tid >> 5); z < first; z += 8 * parts)
                *reinterpret_cast<float4*>(Ob + (long long)z * d.os[2] + col) = zero;
    };
    if (zp > 0) {
        __syncthreads();
        zero_rows();
        return;
    }

    // positions of the block's keys as the K and the V operand need them (keys past the last
    // kept one repeat it: finite values whose weights are zero)
    int pos_k, pos_v[4];
    auto request_pos = [&](int kb) {
        pos_k = idx[min(16 * kb + c16, m - 1)];
#pragma unroll
        for (int r = 0; r < 4; ++r) pos_v[r] = idx[min(16 * kb + 4 * g + r, m - 1)];
    };
    f32x4 kr[8], vr[4][2];
    auto request_k = [&]() {
        const float* src = Kb + (long long)pos_k * d.kvs[2] + 4 * g;
#pragma unroll
        for (int j = 0; j < 8; ++j) kr[j] = *reinterpret_cast<const f32x4*>(src + 16 * j);
    };

    const int i = min(i0 + c16, m - 1);   // rank of this lane's query: the last key it may see
    const float* q_src = Qb + (long long)idx[i] * d.qs[2] + 4 * g;
    request_pos(wave);
    f32x4 qf[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) qf[j] = *reinterpret_cast<const f32x4*>(q_src + 16 * j);
    request_k();

    f32x4 acc[8];                         // O^T: column 8 (4 g + r) + db in register r, query c16
    float m_run = kNone, l_run = 0.f;     // l_run: this lane's keys only
#pragma unroll
    for (int db = 0; db < 8; ++db) acc[db] = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int kb = wave; kb < n_blocks; kb += 4) {
        // this block's V, behind the positions of the wave's next block: loads return in order
        const float* v_src[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) v_src[r] = Vb + (long long)pos_v[r] * d.kvs[2] + 8 * c16;
        request_pos(kb + 4);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            vr[r][0] = *reinterpret_cast<const f32x4*>(v_src[r]);
            vr[r][1] = *reinterpret_cast<const f32x4*>(v_src[r] + 4);
        }
        f32x4 s[2];   // two chains of dependent MFMAs
        s[0] = s[1] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int j = 0; j < 8; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) s[e & 1] = __builtin_amdgcn_mfma_f32_16x16x4f32(kr[j][e], qf[j][e], s[e & 1], 0, 0, 0);
        request_k();
        float sc[4], p[4], mx = kNone;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            sc[r] = 16 * kb + 4 * g + r <= i ? (s[0][r] + s[1][r]) * scale : kNone;
            mx = fmaxf(mx, sc[r]);
        }
        const float m_new = fmaxf(m_run, across_groups_max(mx));
        const float corr = expf(m_run - m_new);
        m_run = m_new;
#pragma unroll
        for (int r = 0; r < 4; ++r) p[r] = sc[r] > -1e29f ? expf(sc[r] - m_new) : 0.f;
        l_run = l_run * corr + ((p[0] + p[1]) + (p[2] + p[3]));
#pragma unroll
        for (int db = 0; db < 8; ++db) acc[db] *= corr;
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int db = 0; db < 8; ++db) acc[db] = __builtin_amdgcn_mfma_f32_16x16x4f32(vr[r][db >> 2][db & 3], p[r], acc[db], 0, 0, 0);
    }

    l_run = across_groups_sum(l_run);
    float* mine = part[wave][c16] + 32 * g;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        *reinterpret_cast<float4*>(mine + 8 * r) = make_float4(acc[0][r], acc[1][r], acc[2][r], acc[3][r]);
        *reinterpret_cast<float4*>(mine + 8 * r + 4) = make_float4(acc[4][r], acc[5][r], acc[6][r], acc[7][r]);
    }
    if (g == 0) { part_m[wave][c16] = m_run; part_l[wave][c16] = l_run; }
    __syncthreads();
    for (int row = tid >> 5; row < kRows && i0 + row < m; row += 8) {
        float m_all = part_m[0][row];
#pragma unroll
        for (int w = 1; w < 4; ++w) m_all = fmaxf(m_all, part_m[w][row]);
        float4 o = zero;
        float l = 0.f;
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            const float f = expf(part_m[w][row] - m_all);
            const float4 x = *reinterpret_cast<const float4*>(&part[w][row][col]);
            o.x = fmaf(f, x.x, o.x); o.y = fmaf(f, x.y, o.y); o.z = fmaf(f, x.z, o.z); o.w = fmaf(f, x.w, o.w);
            l = fmaf(f, part_l[w][row], l);
        }
        const float inv = 1.0f / l;
        const int p = tile_pos[row];
        *reinterpret_cast<float4*>(Ob + (long long)p * d.os[2] + col) = make_float4(o.x * inv, o.y * inv, o.z * inv, o.w * inv);
    }
    zero_rows();
}

}  // namespace

hipError_t launch_zero_filtered(const Dims& d, int dtype, const uint8_t* keep, void* O,
                                hipStream_t s)
{
    dim3 grid((d.n + 15) / 16, d.Hq, d.B);
    if (dtype == 0)
        zero_filtered_kernel<4><<<grid, dim3(256), 0, s>>>(d, keep, (char*)O);
    else
        zero_filtered_kernel<2><<<grid, dim3(256), 0, s>>>(d, keep, (char*)O);
    return hipGetLastError();
}

hipError_t launch_attend_f32(const Dims& d, float scale, const float* Q, const float* K,
                             const float* V, const int32_t* kept_idx, float* O,
                             const int32_t* counts, long long idx_stride, hipStream_t s)
{
    const int parts = counts ? 1 : zero_parts(d.n, d.m);   // (per-row counts: the kernel deals its workgroups itself)
    // far below 2^31 (each has a row of O of its own, 512 bytes), but not below 2^32 threads, which is as far
    // as one dimension of a grid goes: 2^22 workgroups a line
    const int ranks = (d.m + 15) / 16 * parts;
    const unsigned n_wg = (unsigned)ranks * d.Hq * d.B, line = std::min(n_wg, 1u << 22);
    attend_f32_kernel<<<dim3(line, (n_wg + line - 1) / line), dim3(256), 0, s>>>(
        d, scale, Q, K, V, kept_idx, O, counts, counts ? idx_stride : (long long)d.m, parts, ranks, line);
    return hipGetLastError();
}

}  // namespace tf
