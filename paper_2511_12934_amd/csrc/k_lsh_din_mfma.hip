// Eq. 8 on the matrix cores.
//
// DIN_i = total / 2 + (1 / 2 d') sum_k c_ik D[k], or from `lowest` with x_ik = 2 c_ik or 0 in c's place for a candidate unlike
// the history (k_lsh_user_mfma.hip), is a contraction of the candidates' signs c = +-1 (or x), exact in bf16, with the user's fp32 table D [d'][d], which is not: it is cut into three bf16 pieces, D = hi + mid + lo
// (hi = bf16(D), mid = bf16(D - hi), lo = the rest: 8 + 8 + 8 significant bits, exact), each a contraction of its own into
// the SAME fp32 accumulator: every lo product first, then every mid, then every hi, so that the d' additions at full
// magnitude are what they are in the vector-ALU kernel and the two small pieces cost rounding errors 2^-8 and 2^-16 as
// large.
//
// k_lsh_din_pieces adds the history's shares up and writes D's pieces once per request in the order the instruction
// reads its column operand: [piece lo, mid, hi][k-step of 16 bits][feature tile of 32][lane] of 16 bytes -- the order in
// which a wave of k_lsh_din_mfma, 64 candidates (two row tiles) and every feature tile, reads them: one stream, three
// fragments ahead, no LDS and no barrier (at most 192 KB, read by every wave of a compute unit: from L1 and L2).
// What bounds it: the bytes.  64 x 10^4 candidates, d' = d = 64: 71 us for 164 MB of results and 82 MB of signature lines
// (8 of 128 bytes used); 8 x 10^4, d' = d = 128: 36 us, where twice the columns, staged through LDS, took 64 (79 above).
// Streaming stores: 75.
#include "k_lsh_blocks.h"

#include <type_traits>

namespace aif {

typedef __bf16 din_bf16x8 __attribute__((ext_vector_type(8)));
typedef float din_f32x16 __attribute__((ext_vector_type(16)));

__global__ __launch_bounds__(512) void k_lsh_din_pieces(LshModel m, LshBatch b, int part_stride, const float *__restrict__ part,
                                                        float *__restrict__ A, uint4 *__restrict__ out, size_t req_stride)
{
    lsh_pieces_block<512>(m, b.reqs[blockIdx.y], blockIdx.y, blockIdx.x, part_stride, part, A, out, req_stride);
}

hipError_t launch_lsh_din_pieces(const LshModel &m, const LshBatch &b, int part_stride, const float *part, float *A, void *pieces, hipStream_t s)
{
    if (b.n_req == 0) return hipSuccess;
    hipLaunchKernelGGL(k_lsh_din_pieces, dim3(lsh_pieces_blocks(m), b.n_req), dim3(512), 0, s, m, b, part_stride, part, A,
                       (uint4 *)pieces, lsh_din_pieces_stride(m));
    return hipGetLastError();
}

// RT: row tiles of 32 candidates a wave takes; FT: feature tiles, from ft0 on (ALL: all of them, d = 32 FT); the block's first candidate is
// number `first` of its LSH_BLOCK.
template <int RT, int FT, bool ALL>
__device__ __forceinline__ void lsh_din_block(const LshModel &m, const LshBatch &b, const uint8_t *__restrict__ sig_table, const float *__restrict__ A,
                                              const uint4 *__restrict__ pieces, size_t req_stride, int32_t *__restrict__ bad, int blk, int first, int ft0)
{
    constexpr int AHEAD = ALL ? 3 : 8;                          // fragments of every tile in flight
    const int n_ft = ALL ? FT : m.d_out / 32;
    {                                                           // a contiguous run of blocks per XCD: a user's pieces in one L2
        const int per_xcd = b.n_blk >> 3;
        if (blk < 8 * per_xcd) blk = (blk & 7) * per_xcd + (blk >> 3);
    }
    const int r = b.blk_req[blk];
    if (r < 0) return;
    const LshReqDesc rd = b.reqs[r];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, col = lane & 31, h = lane >> 5;
    const int local0 = blk * LSH_BLOCK + first - rd.cand_base + wave * 32 * RT;
    const int nrows = min(32 * RT, rd.n_cand - local0);
    if (nrows <= 0) return;
    const int nw = m.d_bits / 32, ks_n = m.d_bits / 16;

    // the first fragments on their way, then this lane's candidate in each of the wave's row tiles: its signature,
    // whether it exists, whether its id is valid
    const uint4 *src = pieces + (size_t)r * req_stride + lane;
    const int steps = 3 * ks_n;
    uint4 w[AHEAD][FT];
    auto fetch = [&](int i, uint4 (&f)[FT]) __attribute__((always_inline)) {
        i = i < steps ? i : steps - 1;
#pragma unroll
        for (int ft = 0; ft < FT; ++ft) f[ft] = src[(size_t)(i * n_ft + ft0 + ft) * 64];
    };
#pragma unroll
    for (int q = 0; q < AHEAD; ++q) fetch(q, w[q]);
    const float *last = A + ((size_t)r * lsh_rows(m.d_bits) + m.d_bits) * m.d_out;
    // the majority word, a part per lane (d >= 32; those past the signature's are not looked at)
    const int maj_lanes = (int)__float_as_uint(last[LSH_MAJORITY * m.d_out + (lane & 7)]);
    auto maj = [&](int q) __attribute__((always_inline)) { return (uint32_t)__builtin_amdgcn_readlane(maj_lanes, q); };
    // total / 2 and lowest, hi and lo; total is asked for now where there are registers to hold it
    auto load_base = [&](int row, float (&hi)[FT], float (&lo)[FT]) __attribute__((always_inline)) {
#pragma unroll
        for (int ft = 0; ft < FT; ++ft) {
            const float *p = last + (size_t)row * m.d_out + col + (ft0 + ft) * 32;
            hi[ft] = p[0];
            lo[ft] = p[m.d_out];
        }
    };
    // With few feature tiles a wave none of whose candidates is unlike the history has an end of its own, too (100 candidates, two
    // tiles: 9.1 us instead of 11.2; four tiles: 21.2 instead of 16.5)
    constexpr bool EARLY = FT <= 2;
    float hi[FT], lo[FT];
    if constexpr (EARLY) load_base(LSH_TOTAL, hi, lo);
    uint32_t sig[RT][8];
    uint32_t live_mask[RT], ok_mask[RT], low_mask[RT];
    uint32_t usual[RT], one[RT];                                // of this lane's candidate: see step()
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
        const int cand = rt * 32 + col;
        const bool live = cand < nrows;
        int64_t id = live ? rd.cand_ids[local0 + cand] : 0;
        const bool ok = id >= 0 && id < m.n_items;
        if (!ok) id = 0;
        const uint32_t *p = (const uint32_t *)(sig_table + (size_t)id * (nw * 4));
#pragma unroll
        for (int q = 0; q < 8; ++q) sig[rt][q] = q < nw ? p[q] : 0u;
        live_mask[rt] = (uint32_t)__ballot(live);               // lanes 0..31: one bit per candidate of the row tile
        ok_mask[rt] = (uint32_t)__ballot(ok);
        int n_maj = 0;
#pragma unroll
        for (int q = 0; q < 8; ++q) n_maj += q < nw ? __builtin_popcount(~(sig[rt][q] ^ maj(q))) : 0;
        const bool low = live && lsh_dissimilar(n_maj, m.d_bits);
        low_mask[rt] = (uint32_t)__ballot(low);
        usual[rt] = low ? 0u : ~0u;
        one[rt] = low ? 0u : 0x00800080u;
    }
    din_f32x16 acc[RT][FT];
#pragma unroll
    for (int rt = 0; rt < RT; ++rt)
#pragma unroll
        for (int ft = 0; ft < FT; ++ft)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[rt][ft][i] = 0.f;

    int ks = 0;
    // ODD: one of the wave's candidates is unlike the history
    auto step = [&](auto odd_c, int i, const uint4 (&f)[FT]) __attribute__((always_inline)) {
        constexpr bool ODD = decltype(odd_c)::value;
        if (i >= steps) return;
        din_bf16x8 x[RT];
        const uint32_t mword = ODD ? maj(ks >> 1) : 0u;
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) {
            uint32_t word = sig[rt][0];
#pragma unroll
            for (int q = 1; q < 8; ++q) word = (ks >> 1) == q ? sig[rt][q] : word;
            const uint32_t byte = word >> (16 * (ks & 1) + 8 * h);          // bits 16 ks + 8 h .. + 7, the first most significant
            const uint32_t twos = (~(word ^ mword) | usual[rt]) >> (16 * (ks & 1) + 8 * h);
            uint32_t xw[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                // two bits' signs onto a pair of ones -- or of magnitudes: 2 (0x4000) where `twos` has the bit, else 0; the usual
                // candidate has every bit, and its twos less one exponent are ones
                uint32_t mag = 0x3F803F80u;
                if constexpr (ODD) mag = (((twos << (7 + 2 * u)) & 0x4000u) | ((twos << (24 + 2 * u)) & 0x40000000u)) - one[rt];
                xw[u] = ((byte << (8 + 2 * u)) & 0x8000u) | ((byte << (25 + 2 * u)) & 0x80000000u) | mag;
            }
            x[rt] = __builtin_bit_cast(din_bf16x8, make_uint4(xw[0], xw[1], xw[2], xw[3]));
        }
#pragma unroll
        for (int ft = 0; ft < FT; ++ft)
#pragma unroll
            for (int rt = 0; rt < RT; ++rt)
                acc[rt][ft] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x[rt], __builtin_bit_cast(din_bf16x8, f[ft]), acc[rt][ft], 0, 0, 0);
        ks = ks + 1 == ks_n ? 0 : ks + 1;
    };
    auto all = [&](auto odd_c) __attribute__((always_inline)) {
        for (int i = 0; i < steps; i += AHEAD) {
#pragma unroll
            for (int q = 0; q < AHEAD; ++q) {
                step(odd_c, i + q, w[q]);
                fetch(i + q + AHEAD, w[q]);
            }
        }
    };
    // cell v of a lane: candidate 8 (v / 4) + 4 h + v % 4 of the row tile, feature `col` of the feature tile
    auto finish = [&](auto odd_c) __attribute__((always_inline)) {
        constexpr bool ODD = decltype(odd_c)::value;
        const float inv = 0.5f / (float)m.d_bits, nanv = __uint_as_float(0x7FC00000u);
        float low_hi[FT], low_lo[FT];
        if constexpr (ODD) load_base(LSH_LOWEST, low_hi, low_lo);
        if constexpr (!EARLY) load_base(LSH_TOTAL, hi, lo);
#pragma unroll
        for (int rt = 0; rt < RT; ++rt)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int c = 8 * (v / 4) + 4 * h + (v % 4);
                if (!((live_mask[rt] >> c) & 1u)) continue;
                const bool ok = (ok_mask[rt] >> c) & 1u, low = ODD && ((low_mask[rt] >> c) & 1u);
                float *o = rd.din_out + (size_t)(local0 + rt * 32 + c) * m.d_out + ft0 * 32 + col;
#pragma unroll
                for (int ft = 0; ft < FT; ++ft)
                    o[ft * 32] = ok ? (low ? low_hi[ft] : hi[ft]) + fmaf(acc[rt][ft][v], inv, low ? low_lo[ft] : lo[ft]) : nanv;
            }
    };
    uint32_t any_low = 0u;
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) any_low |= low_mask[rt];
    if (__builtin_amdgcn_readfirstlane(any_low)) {
        all(std::true_type{});
        if constexpr (EARLY) finish(std::true_type{});
    } else {
        all(std::false_type{});
        if constexpr (EARLY) finish(std::false_type{});
    }
    if constexpr (!EARLY) finish(std::true_type{});
    if (lane == 0 && ft0 == 0) {
        int n_bad = 0;
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) n_bad += __builtin_popcount(live_mask[rt] & ~ok_mask[rt]);
        if (n_bad) atomicAdd(bad, n_bad);
    }
}

// FT: feature tiles (d = 32 FT)
template <int FT>
__global__ __launch_bounds__(256, 2) void k_lsh_din_mfma(LshModel m, LshBatch b, const uint8_t *__restrict__ sig_table, const float *__restrict__ A,
                                                      const uint4 *__restrict__ pieces, size_t req_stride, int32_t *__restrict__ bad)
{
    lsh_din_block<2, FT, true>(m, b, sig_table, A, pieces, req_stride, bad, blockIdx.x, 0, 0);
}

// The same for few candidates, a wave to one row tile and one feature tile, beside the blocks that add up the histories' parts of Eq. 9.
__global__ __launch_bounds__(256, 4) void k_lsh_result(LshModel m, LshBatch b, const uint8_t *__restrict__ sig_table, const float *__restrict__ A,
                                                    const uint4 *__restrict__ pieces, size_t req_stride, int32_t *__restrict__ bad, int sh,
                                                    const int32_t *__restrict__ parts, int n_parts)
{
    int idx = blockIdx.x;
    const int n_din = 2 * b.n_blk * (m.d_out / 32);
    if (idx < n_din) {
        const int half = idx & 1, blk = (idx >> 1) % b.n_blk, ft = (idx >> 1) / b.n_blk;
        lsh_din_block<1, 1, false>(m, b, sig_table, A, pieces, req_stride, bad, blk, half * 128, ft);
        return;
    }
    lsh_finish_block(m, b, sh, parts, n_parts, idx - n_din);
}

hipError_t launch_lsh_result(const LshModel &m, const LshBatch &b, const uint8_t *sig_table, const float *A, const void *pieces, int32_t *bad,
                             int sh, const void *parts, int n_parts, hipStream_t s)
{
    if (b.n_blk == 0) return hipSuccess;
    if (!lsh_din_on_mfma(m) || !pieces) return hipErrorInvalidValue;
    const dim3 grid(2 * b.n_blk * (m.d_out / 32) + (n_parts > 1 ? b.n_blk : 0));
    hipLaunchKernelGGL(k_lsh_result, grid, dim3(256), 0, s, m, b, sig_table, A, (const uint4 *)pieces, lsh_din_pieces_stride(m), bad, sh,
                       (const int32_t *)parts, n_parts);
    return hipGetLastError();
}

bool lsh_din_on_mfma(const LshModel &m) { return m.d_out % 32 == 0 && m.d_out <= 128 && m.d_bits <= 256; }

size_t lsh_din_pieces_stride(const LshModel &m)                // 16-byte pieces per request
{
    return (size_t)3 * (m.d_bits / 16) * (m.d_out / 32) * 64;
}

hipError_t launch_lsh_din_mfma(const LshModel &m, const LshBatch &b, const uint8_t *sig_table, const float *A, const void *pieces,
                               int32_t *bad, hipStream_t s)
{
    if (b.n_blk == 0) return hipSuccess;
    if (!lsh_din_on_mfma(m) || !pieces) return hipErrorInvalidValue;
    auto go = [&](auto kern) {
        hipLaunchKernelGGL(kern, dim3(b.n_blk), dim3(256), 0, s, m, b, sig_table, A, (const uint4 *)pieces, lsh_din_pieces_stride(m), bad);
    };
    switch (m.d_out / 32) {
    case 1: go(k_lsh_din_mfma<1>); break;
    case 2: go(k_lsh_din_mfma<2>); break;
    case 3: go(k_lsh_din_mfma<3>); break;
    default: go(k_lsh_din_mfma<4>); break;
    }
    return hipGetLastError();
}

}  // namespace aif
