// Bodies of the LSH path's smaller kernels, as device functions of a 256-thread block: each is launched alone by a large call, whose
// two halves run side by side, and beside another kernel's blocks by a small one (k_lsh_stage, k_lsh_count, k_lsh_result).
#pragma once
#include "aif_lsh_dev.h"

namespace aif {

typedef int v4i __attribute__((ext_vector_type(4)));
constexpr int SMT_TILE = 64;         // history items of a row tile: two a row

// thirty-two signature bits -> thirty-two fp4 values (-1)^bit, bit j in nibble j
__device__ __forceinline__ v4i fp4_signs(uint32_t bits)
{
    v4i r;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        uint32_t x = (bits >> (8 * q)) & 0xFFu;                                             // bit i of the eight to nibble i
        x = (x | x << 12) & 0x000F000Fu;
        x = (x | x << 6) & 0x03030303u;
        x = (x | x << 3) & 0x11111111u;
        r[q] = (int)(x << 3 | 0x22222222u);                                                 // 1.0 is 0010, the sign bit on top
    }
    return r;
}

// The history of every request as the instruction's row operand: [row tile][k-step of 32 bits][lane] of 16 bytes; lane =
// (row of the tile, which of the row's two items: item 32 h + row of the tile).  Items past the end are zero vectors.
// N: pieces a thread writes.
template <int KS, int N> __device__ __forceinline__ void lsh_expand_block(const LshReqDesc &rd, int r, int part, v4i *__restrict__ out, size_t req_stride)
{
    const int n = (rd.seq_len + SMT_TILE - 1) / SMT_TILE * KS * 64;
    uint32_t word[N];
    bool real[N];
#pragma unroll
    for (int u = 0; u < N; ++u) {
        const int idx = (part * N + u) * 256 + (int)threadIdx.x;
        const int lane = idx & 63, s = (idx >> 6) % KS, rt = idx / (64 * KS);
        const int item = rt * SMT_TILE + lane;
        real[u] = item < rd.seq_len;
        word[u] = real[u] ? ((const uint32_t *)rd.seq_sigs)[(size_t)item * KS + s] : 0u;
    }
#pragma unroll
    for (int u = 0; u < N; ++u) {
        const int idx = (part * N + u) * 256 + (int)threadIdx.x;
        if (idx < n) out[(size_t)r * req_stride + idx] = real[u] ? fp4_signs(word[u]) : v4i{0, 0, 0, 0};
    }
}

// The counts of one candidate as they come out of the planes -> Eq. 9's tiers.  Two corrections: the rows past the
// history's end were zero vectors and counted as d' / 2 equal bits; the last tier is the history less all the others.
__device__ __forceinline__ void simtier_store(const LshModel &m, const LshReqDesc &rd, int local, int sh, const int32_t (&n)[LSH_MAX_TIERS])
{
    const int64_t id = rd.cand_ids[local];
    int32_t *o = rd.tier_out + (size_t)local * m.n_tiers;
    if (id < 0 || id >= m.n_items) {
        for (int t = 0; t < m.n_tiers; ++t) o[t] = -1;
        return;
    }
    const int pad_tier = m.d_bits >> sh, pad = (rd.seq_len + SMT_TILE - 1) / SMT_TILE * SMT_TILE - rd.seq_len;
    int32_t below = 0;
#pragma unroll
    for (int t = 0; t < LSH_MAX_TIERS; ++t) {
        if (t < m.n_tiers - 1) {
            const int32_t v = n[t] - (t == pad_tier ? pad : 0);
            o[t] = v;
            below += v;
        }
    }
    o[m.n_tiers - 1] = rd.seq_len - below;
}

// The counts of the histories' parts added up.
__device__ __forceinline__ void lsh_finish_block(const LshModel &m, const LshBatch &b, int sh, const int32_t *__restrict__ parts, int n_parts, int blk)
{
    const int r = b.blk_req[blk];
    if (r < 0) return;
    const LshReqDesc rd = b.reqs[r];
    const int local = blk * LSH_BLOCK - rd.cand_base + (int)threadIdx.x;
    if (local >= rd.n_cand) return;
    int32_t n[LSH_MAX_TIERS];
#pragma unroll
    for (int t = 0; t < LSH_MAX_TIERS; ++t) n[t] = 0;
    for (int p = 0; p < n_parts; ++p) {
        const int4 *q = (const int4 *)(parts + ((size_t)p * b.n_blk * LSH_BLOCK + (size_t)blk * LSH_BLOCK + threadIdx.x) * LSH_MAX_TIERS);
        const int4 lo = q[0], hi = q[1];
        n[0] += lo.x, n[1] += lo.y, n[2] += lo.z, n[3] += lo.w;
        n[4] += hi.x, n[5] += hi.y, n[6] += hi.z, n[7] += hi.w;
    }
    simtier_store(m, rd, local, sh, n);
}

__device__ __forceinline__ uint32_t bf16_rne_bits(float x)
{
    const uint32_t u = __float_as_uint(x);
    return (u + 0x7FFFu + ((u >> 16) & 1u)) >> 16;          // finite inputs (sums of embeddings)
}

// D's pieces (k_lsh_din_mfma.hip), block = (k-step, feature tile): 16 bits x 32 features, one sum a thread (of 512) or two (of 256); the
// blocks past the last k-step add up total and lowest, eight threads each per feature.
template <int THREADS>
__device__ __forceinline__ void lsh_pieces_block(const LshModel &m, const LshReqDesc &rd, int r, int part_no, int part_stride, const float *__restrict__ part,
                                                 float *__restrict__ A, uint4 *__restrict__ out, size_t req_stride)
{
    __shared__ float D[16][33];
    __shared__ double S[16][33];
    const int ft_n = m.d_out / 32, ks_n = m.d_bits / 16, ft = part_no % ft_n, ks = part_no / ft_n;
    const int j = threadIdx.x & 31, shares = lsh_chunks(m.fine, rd.seq_len) * lsh_user_split(m.d_bits);
    const size_t n = (size_t)lsh_rows(m.d_bits) * m.d_out;
    const float *p = part + (size_t)r * part_stride * n + ft * 32 + j;
    if (ks == ks_n) {
        float *a = A + (size_t)r * n + (size_t)m.d_bits * m.d_out;
#pragma unroll
        for (int u = 0; u < 512 / THREADS; ++u) {
            const int k = (threadIdx.x >> 5) + 8 * u, row = k & 1 ? LSH_LOWEST : LSH_TOTAL, from = k >> 1;
            S[k][j] = lsh_sum_totals(p + (size_t)(m.d_bits + row) * m.d_out + from * n, 8 * n, m.d_out, (shares - from + 7) / 8);
        }
        __syncthreads();
        const int k = threadIdx.x >> 5;
        if (k < 2) {
            const int row = k & 1 ? LSH_LOWEST : LSH_TOTAL;
            double t = 0.0;
#pragma unroll
            for (int i = 0; i < 8; ++i) t += S[2 * i + k][j];
            t *= k == 0 ? 0.5 : 1.0 / m.d_bits;
            a += row * m.d_out + ft * 32 + j;
            a[0] = (float)t;
            a[m.d_out] = (float)(t - (double)(float)t);
        } else if (k == 2 && ft == 0 && j < 8)
            a[LSH_MAJORITY * m.d_out + j] = shares > 0 ? p[(size_t)(m.d_bits + LSH_MAJORITY) * m.d_out] : 0.f;
        return;
    }
    if constexpr (THREADS == 512) {
        const int k = threadIdx.x >> 5;
        D[k][j] = lsh_sum_parts(p + (size_t)(16 * ks + k) * m.d_out, n, shares);
    } else {
        static_assert(THREADS == 256);
        const int k = threadIdx.x >> 5;
        const float *q = p + (size_t)(16 * ks + k) * m.d_out;
        float a0, a1;
        lsh_sum_parts2(q, q + (size_t)8 * m.d_out, n, shares, a0, a1);
        D[k][j] = a0;
        D[k + 8][j] = a1;
    }
    __syncthreads();
    if (threadIdx.x >= 64) return;
    const int lane = threadIdx.x, c = lane & 31, h = lane >> 5;    // lane = (feature of the tile, which 8 of the k-step's bits)
    uint32_t piece[3][4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        uint32_t half[3][2];
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            const float w = D[8 * h + 2 * u + s][c];
            const uint32_t hi = bf16_rne_bits(w);
            const float r1 = w - __uint_as_float(hi << 16);
            const uint32_t mid = bf16_rne_bits(r1);
            const float r2 = r1 - __uint_as_float(mid << 16);
            half[0][s] = bf16_rne_bits(r2);                 // accumulated first
            half[1][s] = mid;
            half[2][s] = hi;
        }
#pragma unroll
        for (int q = 0; q < 3; ++q) piece[q][u] = half[q][0] | (half[q][1] << 16);
    }
    uint4 *o = out + (size_t)r * req_stride;
#pragma unroll
    for (int q = 0; q < 3; ++q)
        o[((size_t)(q * ks_n + ks) * ft_n + ft) * 64 + lane] = make_uint4(piece[q][0], piece[q][1], piece[q][2], piece[q][3]);
}

}  // namespace aif
