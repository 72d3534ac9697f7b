// LSH-based long-sequence behaviour modelling (Sec. 4.3): signature similarity
// by XNOR + population count (Eq. 6, 7), LSH-DIN (Eq. 8) and SimTier (Eq. 9).
//
// SimTier needs every (candidate, history item) similarity, so its kernel walks
// the b x l pairs: a lane owns one candidate, the history signatures are the
// same for all lanes and arrive through scalar loads, a pair costs two XNORs,
// two population counts and a handful of integer instructions that bump one
// byte of a packed 64-bit histogram (eight tiers, flushed before a byte can
// overflow).  Plain integer work, bound by the vector ALU.
//
// LSH-DIN does NOT need the pairs: Eq. 8 has no softmax, so it factors into
// d' + 1 vectors of the user alone (k_lsh_user_mfma.hip) and, per candidate,
// d' additions per output feature.  Same value as Eq. 8 up to the order of the
// fp32 additions.
#include "aif_lsh_dev.h"

namespace aif {

// ---------------------------------------------------------------------------
// Eq. 8.  Block = LSH_BLOCK candidates of one request; d / 16 threads per candidate, 16 features each.
// The user's table D[d'][d] is staged in LDS in slices of KC bits and added with the candidate's sign -- or, for a candidate
// unlike the history, twice that where it has the majority bit and not at all elsewhere (k_lsh_user_mfma.hip).
// ---------------------------------------------------------------------------
constexpr int LSH_DIN_LDS = 64 * 1024;

__global__ __launch_bounds__(256) void k_lsh_din(LshModel m, LshBatch b, const uint8_t *__restrict__ sig_table,
                                                 const float *__restrict__ A, int32_t *__restrict__ bad)
{
    extern __shared__ __align__(16) char lds[];
    float *sa = (float *)lds;                                   // [kc][d]
    int blk = blockIdx.x;                                       // a contiguous run of blocks per XCD, as in k_lsh_simtier: a user's table in one L2
    {
        const int per_xcd = b.n_blk >> 3;
        if (blk < 8 * per_xcd) blk = (blk & 7) * per_xcd + (blk >> 3);
    }
    const int r = b.blk_req[blk];
    if (r < 0) return;
    const LshReqDesc rd = b.reqs[r];
    const int local0 = blk * LSH_BLOCK - rd.cand_base;
    const int nrows = min(LSH_BLOCK, rd.n_cand - local0);
    if (nrows <= 0) return;
    const int d = m.d_out, jg = d / 16, nb = m.d_bits / 8, nw = m.d_bits / 32;
    const int per_round = 256 / jg;                             // candidates served at once
    const int kc = min(m.d_bits, LSH_DIN_LDS / (d * 4)) & ~7;       // bits per slice, whole bytes
    const float *Ar = A + (size_t)r * lsh_rows(m.d_bits) * d;
    const float *last = Ar + (size_t)m.d_bits * d;
    const uint8_t *maj = (const uint8_t *)(last + LSH_MAJORITY * d);
    const int sub = threadIdx.x / jg, j0 = (threadIdx.x - sub * jg) * 16;
    const float inv = 0.5f / (float)m.d_bits;
    int n_bad = 0;

    for (int c0 = 0; c0 < nrows; c0 += per_round) {
        const int cand = c0 + sub;
        const bool live = sub < per_round && cand < nrows;
        int64_t id = live ? rd.cand_ids[local0 + cand] : 0;
        const bool ok = id >= 0 && id < m.n_items;
        if (!ok) {
            id = 0;
            if (live && j0 == 0) ++n_bad;
        }
        const uint8_t *sig = sig_table + (size_t)id * nb;
        uint32_t same[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) same[i] = ~(((const uint32_t *)sig)[min(i, nw - 1)] ^ ((const uint32_t *)maj)[min(i, nw - 1)]);
        int n_maj = 0;
#pragma unroll
        for (int i = 0; i < 8; ++i) n_maj += i < nw ? __builtin_popcount(same[i]) : 0;
        const bool low = lsh_dissimilar(n_maj, m.d_bits);
        float acc[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[i] = 0.f;
        for (int k0 = 0; k0 < m.d_bits; k0 += kc) {
            const int kn = min(kc, m.d_bits - k0);
            __syncthreads();
            if (c0 == 0 || kc < m.d_bits) {                     // the whole table fits: staged once
                for (int i = threadIdx.x; i < kn * d / 4; i += 256) ((float4 *)sa)[i] = ((const float4 *)(Ar + (size_t)k0 * d))[i];
            }
            __syncthreads();
            if (live) {
                for (int kb = 0; kb < kn; kb += 8) {
                    const uint32_t byte = sig[(k0 + kb) >> 3], equal = ~(byte ^ maj[(k0 + kb) >> 3]);
#pragma unroll
                    for (int u = 0; u < 8; ++u) {
                        const float mag = !low ? 1.f : (equal >> (7 - u)) & 1 ? 2.f : 0.f, c = (byte >> (7 - u)) & 1 ? -mag : mag;
                        const float4 *a4 = (const float4 *)(sa + (size_t)(kb + u) * d + j0);
#pragma unroll
                        for (int q = 0; q < 4; ++q) {
                            const float4 v = a4[q];
                            acc[4 * q + 0] = fmaf(c, v.x, acc[4 * q + 0]);
                            acc[4 * q + 1] = fmaf(c, v.y, acc[4 * q + 1]);
                            acc[4 * q + 2] = fmaf(c, v.z, acc[4 * q + 2]);
                            acc[4 * q + 3] = fmaf(c, v.w, acc[4 * q + 3]);
                        }
                    }
                }
            }
        }
        if (live) {
            float4 *o = (float4 *)(rd.din_out + (size_t)(local0 + cand) * d + j0);
            const float nanv = __uint_as_float(0x7FC00000u);
            const float *hi = last + (low ? LSH_LOWEST : LSH_TOTAL) * d + j0, *lo = hi + d;
            auto at = [&](int i) { return hi[i] + fmaf(acc[i], inv, lo[i]); };
#pragma unroll
            for (int q = 0; q < 4; ++q)
                o[q] = ok ? make_float4(at(4 * q), at(4 * q + 1), at(4 * q + 2), at(4 * q + 3)) : make_float4(nanv, nanv, nanv, nanv);
        }
    }
    if (n_bad) atomicAdd(bad, n_bad);
}

hipError_t launch_lsh_din(const LshModel &m, const LshBatch &b, const uint8_t *sig_table, const float *A, int32_t *bad,
                          hipStream_t s)
{
    if (b.n_blk == 0) return hipSuccess;
    static bool attr_set = false;
    if (!attr_set) {
        hipError_t e = hipFuncSetAttribute((const void *)k_lsh_din, hipFuncAttributeMaxDynamicSharedMemorySize, LSH_DIN_LDS);
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    hipLaunchKernelGGL(k_lsh_din, dim3(b.n_blk), dim3(256), LSH_DIN_LDS, s, m, b, sig_table, A, bad);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Eq. 6, 7, 9.  A lane owns one candidate and walks the whole history.
// DW = signature width in 32-bit words.
// ---------------------------------------------------------------------------
template <int DW>
__global__ __launch_bounds__(256) void k_lsh_simtier(LshModel m, LshBatch b, const uint8_t *__restrict__ sig_table)
{
    // Workgroups go to the 8 XCDs in turn, each with an L2 of its own.  Every XCD takes a contiguous run of the
    // blocks, so that the blocks of one user -- which all walk that user's history signatures -- share an L2 instead
    // of all eight fetching them.
    int blk = blockIdx.x;
    {
        const int per_xcd = b.n_blk >> 3;
        if (blk < 8 * per_xcd) blk = (blk & 7) * per_xcd + (blk >> 3);
    }
    const int r = b.blk_req[blk];
    if (r < 0) return;
    const LshReqDesc rd = b.reqs[r];
    const int local = blk * LSH_BLOCK - rd.cand_base + threadIdx.x;
    const bool live = local < rd.n_cand;
    int64_t id = live ? rd.cand_ids[local] : 0;
    const bool ok = id >= 0 && id < m.n_items;
    if (!ok) id = 0;
    uint32_t sig[DW];
    {
        const uint32_t *p = (const uint32_t *)(sig_table + (size_t)id * (DW * 4));
#pragma unroll
        for (int w = 0; w < DW; ++w) sig[w] = p[w];
    }
    const uint32_t *__restrict__ hs = (const uint32_t *)rd.seq_sigs;    // the same for every lane: scalar loads
    const int L = rd.seq_len;
    // 8 * tier = min(8 (N - 1), ((equal * N * tier_mul) >> 17) & ~7); equal <= 256 and N * tier_mul < 2^19 fit a
    // 24-bit multiply, and the multiply-shift is exact for equal N <= 2048, d' <= 256
    const uint32_t scale = (uint32_t)m.n_tiers * (uint32_t)m.tier_mul, top8 = 8u * (uint32_t)(m.n_tiers - 1);
    uint32_t total[LSH_MAX_TIERS];
#pragma unroll
    for (int j = 0; j < LSH_MAX_TIERS; ++j) total[j] = 0;
    unsigned long long packed = 0;                          // eight byte-wide tier counters

    auto visit = [&](const uint32_t *h) {
        uint32_t equal = 0;
#pragma unroll
        for (int w = 0; w < DW; ++w) equal += __builtin_popcount(~(sig[w] ^ h[w]));
        uint32_t tier8 = (__umul24(equal, scale) >> 17) & ~7u;
        tier8 = tier8 < top8 ? tier8 : top8;
        packed += 1ull << tier8;
    };
    auto flush = [&]() {
#pragma unroll
        for (int j = 0; j < LSH_MAX_TIERS; ++j) total[j] += (uint32_t)(packed >> (8 * j)) & 255u;
        packed = 0;
    };
    constexpr int UNROLL = 16, PER_FLUSH = 15;              // 240 increments at most between flushes
    int t = 0;
    while (t + UNROLL <= L) {
        const int stop = min(L - UNROLL + 1, t + UNROLL * PER_FLUSH);
        for (; t < stop; t += UNROLL) {
            uint32_t h[UNROLL * DW];
#pragma unroll
            for (int u = 0; u < UNROLL * DW; ++u) h[u] = hs[(size_t)t * DW + u];
#pragma unroll
            for (int u = 0; u < UNROLL; ++u) visit(h + u * DW);
        }
        flush();
    }
    for (; t < L; ++t) {
        uint32_t h[DW];
#pragma unroll
        for (int w = 0; w < DW; ++w) h[w] = hs[(size_t)t * DW + w];
        visit(h);
    }
    flush();
    if (live) {
        int32_t *o = rd.tier_out + (size_t)local * m.n_tiers;
        for (int j = 0; j < m.n_tiers; ++j) o[j] = ok ? (int32_t)total[j] : -1;
    }
}

hipError_t launch_lsh_simtier(const LshModel &m, const LshBatch &b, const uint8_t *sig_table, hipStream_t s)
{
    if (b.n_blk == 0) return hipSuccess;
    const dim3 grid(b.n_blk), block(256);
    switch (m.d_bits / 32) {
    case 1: hipLaunchKernelGGL(k_lsh_simtier<1>, grid, block, 0, s, m, b, sig_table); break;
    case 2: hipLaunchKernelGGL(k_lsh_simtier<2>, grid, block, 0, s, m, b, sig_table); break;
    case 3: hipLaunchKernelGGL(k_lsh_simtier<3>, grid, block, 0, s, m, b, sig_table); break;
    case 4: hipLaunchKernelGGL(k_lsh_simtier<4>, grid, block, 0, s, m, b, sig_table); break;
    case 5: hipLaunchKernelGGL(k_lsh_simtier<5>, grid, block, 0, s, m, b, sig_table); break;
    case 6: hipLaunchKernelGGL(k_lsh_simtier<6>, grid, block, 0, s, m, b, sig_table); break;
    case 7: hipLaunchKernelGGL(k_lsh_simtier<7>, grid, block, 0, s, m, b, sig_table); break;
    case 8: hipLaunchKernelGGL(k_lsh_simtier<8>, grid, block, 0, s, m, b, sig_table); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace aif
