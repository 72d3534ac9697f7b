// The user side of Eq. 8 on the matrix cores.
//
// With the bits as signs, c = (-1)^bit, the similarity of candidate i and history item t is
//     m_it = (1/2) (1 + (1/d') sum_k c_ik c_tk),
// so Eq. 8 is, with U~_t the projected history embeddings,
//     DIN_i = (1/2) total + (1 / 2 d') sum_k c_ik D[k],   D[k] = sum_t c_tk U~_t,   total = sum_t U~_t:
// d' + 1 vectors that belong to the user alone, formed once per request.  D is a contraction over the history,
// (signs) [d' x l] times U~ [l x d].
//
// Where the similarities are small the two terms cancel, and what rounding left of D stands against a small sum.  So the
// history's majority word goes with the sums (per place the bit that most of it has), and
//     lowest = (1/d') sum_t w_t U~_t,   w_t = the places where signature t differs from the majority word,
// what a candidate opposite to that word gets; any other gets a place's D[k], with the majority bit's sign, on top of it for
// each place where it has the majority bit:
//     DIN_i = lowest + (1 / 2 d') sum_k x_ik D[k],   x_ik = 2 c_ik there and 0 elsewhere.
// Nothing cancels for a candidate with few such places; one with many is served by the first form, whose terms are half as
// large (the line: lsh_dissimilar).  The majority is that of 64 items spread over the history: any word gives a valid
// sum, and where it matters, where nearly all items agree, 64 show it.  Measured (2,000 items within 2 % of a prototype, d' = d = 64,
// fp32 embeddings of N(0, 0.1); errors against 64 bits, relative, 2-norms): candidates of similarity 0.02, 0.05, 0.13, 0.26: 4.8, 5.5,
// 5.4, 6.2 x 10^-8, where the first form has 240, 98, 40, 16; at 0.5, by the first form, 5.4.  It costs the smallest calls 0 to 4 us
// (100 candidates, 100 items, fp32: 31.2 -> 32.9) and most from a thousand items on nothing.
//
// Signs are exact in bf16, and so are bf16 embeddings; fp32 embeddings are cut into three bf16 pieces (8 + 8 + 8
// significant bits: exact), each a product of its own.  The contraction index t is the slow axis of both inputs as the
// caller stores them, while an MFMA operand wants a lane to hold eight consecutive t.  Neither passes through LDS for
// that: a lane loads VW neighbouring columns of its eight items (32 lanes together a whole row) and packs item pairs
// with one byte permute per pair, column f of its VW going to the f-th of VW column tiles (tile f = columns VW c + f);
// of the signatures a lane fetches one item's word per 64 items and every lane of a row tile receives the words of its
// eight items by ds_bpermute, shifts its own bit to the top, and merges two signs into a pair of bf16 ones.
//
// Block = (chunk of lsh_chunk_len items, request, up to four row tiles of 32 bits); its waves take a row tile each, and
// where there are fewer than four the chunk's items are shared out as well (lsh_user_split).  Loads run AHEAD
// steps of 16 items ahead.  Two barriers a block: the majority word's parts, formed while the first items are on their way,
// and at the end the waves' shares of total and lowest (they take the steps in turn).  All partial sums are added in a fixed order, a function of the request's own history
// length and the model.
//
// What bounds it: the loads in flight (the history's bytes would take half the time).  10^5 items of 128-bit signatures
// and 128 bf16 features for 8 users (216 MB): 92 us, where a block that transposed both inputs through LDS, with two
// barriers and a memory round trip per 64 items and tables for either value of a bit, took 328; 10^4 items, 64 bits, 64
// features, 64 users: 35 against 68.
#include "aif_dev.h"
#include "k_lsh_blocks.h"

#include <algorithm>
#include <type_traits>

namespace aif {

typedef __bf16 lsh_bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 lsh_bf16x2 __attribute__((ext_vector_type(2)));
typedef float lsh_f32x16 __attribute__((ext_vector_type(16)));

// Bit k < BITS: whether at least half of the wave's 64 words have it.
template <int BITS> __device__ __forceinline__ uint32_t lsh_majority(uint32_t word)
{
    uint32_t m = 0;
#pragma unroll
    for (int k = 0; k < BITS; ++k) m |= __builtin_popcountll(__ballot((word >> k) & 1u)) >= 32 ? 1u << k : 0u;
    return m;
}

// The request's tensors are known to lie in global memory: a load through a generic pointer counts as an LDS access as well,
// and every bpermute would wait for all loads in flight.
template <typename T> using lsh_global = const T __attribute__((address_space(1))) *;

// T: storage of the embeddings; VW: neighbouring columns a lane owns (32 VW columns a block); W: words a signature has at most
// chunk, z: which of the history's chunks, which group of row tiles and of columns
template <typename T, int VW, int W>
__device__ __forceinline__ void lsh_user_sums_block(const LshModel &m, const LshReqDesc &rd, int r, int chunk, int z, int part_stride, float *__restrict__ part)
{
    constexpr int P = sizeof(T) == 4 ? 3 : 1, WORDS = sizeof(T) == 4 ? VW : (VW + 1) / 2;   // 32-bit words of a lane's columns
    constexpr int AHEAD = 4;                                    // steps of 16 items in flight
    // fp32 embeddings: D's sums over 64 items are formed apart and then added on, one rounding at full size instead of twelve
    constexpr bool TWO = sizeof(T) == 4;
    typedef uint32_t vec __attribute__((ext_vector_type(WORDS)));
    const int d = m.d_out, db = m.d_bits, rts = db / 32;
    const int groups = (rts + 3) / 4, rg = z % groups, cg = z / groups;
    const int chunk_len = lsh_chunk_len(m.fine, rd.seq_len), t_lo = chunk * chunk_len;
    if (t_lo >= rd.seq_len) return;
    const int t_hi = min(rd.seq_len, t_lo + chunk_len);
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), col = lane & 31, h = lane >> 5;
    const int split = lsh_user_split(db), rt = rg * 4 + wave % (4 / split), sub = wave / (4 / split);
    const bool active = rt < rts, sums = rg == 0;               // sums: this block forms total and lowest
    const int n_steps = (t_hi - t_lo + 15) / 16, n_sum = min(4 / split, rts);               // n_sum: waves that share those
    const int s_lo = (int)((long)n_steps * sub / split), s_hi = active ? (int)((long)n_steps * (sub + 1) / split) : s_lo;

    const int j0 = (cg * 32 + col) * VW;
    const bool on = j0 < d;                                     // whole groups: d is a multiple of 16
    const lsh_global<uint32_t> sigs = (lsh_global<uint32_t>)rd.seq_sigs, sg = sigs + (active ? rt : 0);
    const int bit = 8 * (col >> 3) + 7 - (col & 7);             // bit k of a signature: byte k / 8, first bit most significant

    lsh_f32x16 acc[VW];
    double tot[VW], low[VW];                                    // 64 bits: see lsh_rows
#pragma unroll
    for (int f = 0; f < VW; ++f) {
        tot[f] = low[f] = 0.0;
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[f][e] = 0.f;
    }
    vec buf[AHEAD][8];
    const lsh_global<T> rows = (lsh_global<T>)rd.seq_emb + (size_t)t_lo * d;    // the same for every lane; row_at: the lane's first item of a step
    const uint32_t row_at = (uint32_t)(8 * h * d + (on ? j0 : 0));
    auto load = [&](int s, vec (&v)[8]) __attribute__((always_inline)) {
        auto get = [&](int i, lsh_global<T> p) __attribute__((always_inline)) {
            if constexpr (sizeof(T) == 2 && VW == 1) v[i][0] = *p;
            else v[i] = *(lsh_global<vec>)p;
        };
        if (t_lo + 16 * s + 16 <= t_hi) {
            const lsh_global<T> base = rows + (size_t)16 * s * d;
#pragma unroll
            for (int i = 0; i < 8; ++i) get(i, base + i * d + row_at);
        } else {                                                // the last item again, in place of those past the end
#pragma unroll
            for (int i = 0; i < 8; ++i) get(i, rows + (size_t)min(16 * s + 8 * h + i, t_hi - t_lo - 1) * d + (on ? j0 : 0));
        }
    };
    auto load_sig = [&](int s) { return sg[(size_t)min(t_lo + 16 * s + lane, t_hi - 1) * rts]; };      // one item's word per lane, 64 items
    auto load_words = [&](int s, uint32_t (&w)[W]) {            // ... and its whole signature
        const lsh_global<uint32_t> p = sigs + (size_t)min(t_lo + 16 * s + lane, t_hi - 1) * rts;
#pragma unroll
        for (int k = 0; k < W; ++k) w[k] = p[min(k, rts - 1)];
    };
    // into[f] += the step's items.  `weigh`: this wave's turn to add them to total and lowest as well, eight at a time in fp32 (on
    // the vector ALU: the matrix instruction's sums of fp32 pieces are cut off, not rounded, and over a history that adds up
    // -- 3e-7 instead of 3e-8 at 2 x 10^4 items).  weights: w_t in bf16 (whole numbers up to 256: exact), a pair per even lane, 64 items
    auto step = [&](int s, vec (&v)[8], uint32_t sig, uint32_t weights, int q, bool weigh, lsh_f32x16 (&into)[VW]) __attribute__((always_inline)) {
        if (!on || t_lo + 16 * s + 16 > t_hi) {                 // items past the end, columns past the width: zero
#pragma unroll
            for (int i = 0; i < 8; ++i)
                if (!on || t_lo + 16 * s + 8 * h + i >= t_hi)
#pragma unroll
                    for (int w = 0; w < WORDS; ++w) v[i][w] = 0u;
        }
        uint32_t sw[8], a4[4];
#pragma unroll
        for (int i = 0; i < 8; ++i) sw[i] = (uint32_t)__builtin_amdgcn_ds_bpermute(4 * (16 * q + 8 * h + i), (int)sig) << (31 - bit);
#pragma unroll
        for (int i = 0; i < 4; ++i)                             // (-1)^bit of two items as bf16: the sign bits onto a pair of ones
            a4[i] = (__builtin_amdgcn_perm(sw[2 * i + 1], sw[2 * i], 0x07060302u) & 0x80008000u) | 0x3F803F80u;
        const lsh_bf16x8 a = __builtin_bit_cast(lsh_bf16x8, make_uint4(a4[0], a4[1], a4[2], a4[3]));
        uint32_t w4[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) w4[i] = (uint32_t)__builtin_amdgcn_ds_bpermute(4 * (16 * q + 8 * h + 2 * i), (int)weights);
        auto pair = [&](int i, int f) __attribute__((always_inline)) {          // column f of items 2i and 2i + 1, bf16
            return __builtin_amdgcn_perm(v[2 * i + 1][f >> 1], v[2 * i][f >> 1], f & 1 ? 0x07060302u : 0x05040100u);
        };
#pragma unroll
        for (int f = 0; f < VW; ++f) {
            if constexpr (P == 1) {
                const lsh_bf16x8 u = __builtin_bit_cast(lsh_bf16x8, make_uint4(pair(0, f), pair(1, f), pair(2, f), pair(3, f)));
                into[f] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, u, into[f], 0, 0, 0);
            } else {
                lsh_bf16x8 p[P];
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    float x = __uint_as_float(v[i][f]);
#pragma unroll
                    for (int k = 0; k < P; ++k) {
                        p[k][i] = (__bf16)x;
                        x -= (float)p[k][i];
                    }
                }
#pragma unroll
                for (int k = P - 1; k >= 0; --k) into[f] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, p[k], into[f], 0, 0, 0);
            }
        }
        if (weigh)
#pragma unroll
            for (int f = 0; f < VW; ++f) {
                float sum = 0.f, wsum = 0.f;
                if constexpr (P == 1) {
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const lsh_bf16x2 x = __builtin_bit_cast(lsh_bf16x2, pair(i, f));
                        sum = __builtin_amdgcn_fdot2_f32_bf16(x, __builtin_bit_cast(lsh_bf16x2, 0x3F803F80u), sum, false);
                        wsum = __builtin_amdgcn_fdot2_f32_bf16(x, __builtin_bit_cast(lsh_bf16x2, w4[i]), wsum, false);
                    }
                } else {
#pragma unroll
                    for (int i = 0; i < 8; ++i) {
                        const float x = __uint_as_float(v[i][f]);
                        sum += x;
                        wsum = fmaf(x, __uint_as_float(i & 1 ? w4[i >> 1] & 0xFFFF0000u : w4[i >> 1] << 16), wsum);
                    }
                }
                tot[f] += (double)sum;
                low[f] += (double)wsum;
            }
    };
    // the majority word (of blocks that form the sums): the waves take a word of 64 items each, or a part of one, past four
    // words a second
    constexpr int PARTS = W < 4 ? 4 / W : 1, BITS = 32 / PARTS;
    uint32_t words[W], maj[W], sample[2];
    __shared__ uint32_t maj_shared[8];
    {
        const lsh_global<uint32_t> p = sigs + (size_t)((long)lane * rd.seq_len >> 6) * rts;
        sample[0] = p[min(wave / PARTS, rts - 1)];
        sample[1] = W > 4 ? p[min(wave + 4, rts - 1)] : 0u;
    }
    uint32_t sig = load_sig(s_lo);
    load_words(s_lo, words);
#pragma unroll
    for (int q = 0; q < AHEAD; ++q) load(s_lo + q, buf[q]);
    if (sums) {
        const int shift = BITS * (wave % PARTS);
        const uint32_t m = lsh_majority<BITS>(sample[0] >> shift) << shift, m2 = W > 4 ? lsh_majority<BITS>(sample[1]) : 0u;
        if (lane == 0) {
            maj_shared[wave] = m;
            maj_shared[wave + 4] = m2;
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < W; ++k) {
            maj[k] = 0u;
#pragma unroll
            for (int p = 0; p < PARTS; ++p) maj[k] |= (uint32_t)__builtin_amdgcn_readfirstlane((int)maj_shared[k * PARTS + p]);
        }
    }
    auto differing = [&]() {                                    // w_t of the lane's item and of its neighbour in the pair
        int n = 0;
#pragma unroll
        for (int k = 0; k < W; ++k) n += __builtin_popcount((words[k] ^ maj[k]) & (k < rts ? ~0u : 0u));
        const uint32_t w = __float_as_uint((float)n);
        return w >> 16 | ((uint32_t)__builtin_amdgcn_update_dpp(0, (int)w, 0xB1, 0xF, 0xF, true) & 0xFFFF0000u);      // quad_perm 1,0,3,2
    };
    if (s_lo < s_hi) {
        uint32_t weights = sums ? differing() : 0u;
        int turn = 0;
        for (int s = s_lo; s < s_hi; s += 4) {
            const uint32_t next = load_sig(s + 4);
            load_words(s + 4, words);
            lsh_f32x16 four[TWO ? VW : 1];
            if constexpr (TWO)
#pragma unroll
                for (int f = 0; f < VW; ++f) four[f] = lsh_f32x16{};
            auto at = [&](int q, lsh_f32x16 (&into)[VW]) __attribute__((always_inline)) {
                step(s + q, buf[q % AHEAD], sig, weights, q, sums && turn == rt, into);
                turn = turn + 1 == n_sum ? 0 : turn + 1;
                load(s + q + AHEAD, buf[q % AHEAD]);
            };
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if (s + q < s_hi) {
                    if constexpr (TWO) at(q, four);
                    else at(q, acc);
                }
            if constexpr (TWO)
#pragma unroll
                for (int f = 0; f < VW; ++f) acc[f] += four[f];
            sig = next;
            if (sums) weights = differing();
        }
    }
    float *out = part + ((size_t)r * part_stride + chunk * split + sub) * lsh_rows(db) * d;
    auto store = [&](float *p, const float *v) {
        if constexpr (VW == 4) *(float4 *)p = make_float4(v[0], v[1], v[2], v[3]);
        else if constexpr (VW == 2) *(float2 *)p = make_float2(v[0], v[1]);
        else *p = v[0];
    };
    if (on && active) {
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            float v[VW];
#pragma unroll
            for (int f = 0; f < VW; ++f) v[f] = acc[f][e];
            store(out + (size_t)(32 * rt + 8 * (e >> 2) + 4 * h + (e & 3)) * d + j0, v);
        }
    }
    if (!sums) return;                                          // the same for the whole block
    __shared__ double shared[4][2][VW][32];
#pragma unroll
    for (int f = 0; f < VW; ++f) {
        tot[f] += __shfl_xor(tot[f], 32, 64);
        low[f] += __shfl_xor(low[f], 32, 64);
        if (h == 0 && n_sum > 1) {
            shared[wave][0][f][col] = tot[f];
            shared[wave][1][f][col] = low[f];
        }
    }
    if (n_sum > 1) __syncthreads();
    if (rt != 0) return;
    float v[4][VW];
#pragma unroll
    for (int f = 0; f < VW; ++f) {
        for (int k = 1; k < n_sum; ++k) {                       // the other waves of this share, in order
            tot[f] += shared[wave + k][0][f][col];
            low[f] += shared[wave + k][1][f][col];
        }
        v[0][f] = (float)tot[f];
        v[1][f] = (float)(tot[f] - (double)v[0][f]);
        v[2][f] = (float)low[f];
        v[3][f] = (float)(low[f] - (double)v[2][f]);
    }
    if (on && h == 0) {
        store(out + (size_t)(db + LSH_TOTAL) * d + j0, v[0]);
        store(out + (size_t)(db + LSH_TOTAL + 1) * d + j0, v[1]);
        store(out + (size_t)(db + LSH_LOWEST) * d + j0, v[2]);
        store(out + (size_t)(db + LSH_LOWEST + 1) * d + j0, v[3]);
    }
    if (chunk == 0 && sub == 0 && cg == 0) {
#pragma unroll
        for (int k = 0; k < W; ++k)
            if (lane == k && k < rts) ((uint32_t *)out)[(size_t)(db + LSH_MAJORITY) * d + k] = maj[k];
    }
}

template <typename T, int VW, int W>
__global__ __launch_bounds__(256, 2) void k_lsh_user_sums(LshModel m, LshBatch b, int part_stride, float *__restrict__ part)
{
    lsh_user_sums_block<T, VW, W>(m, b.reqs[blockIdx.y], blockIdx.y, blockIdx.x, blockIdx.z, part_stride, part);
}

// The same beside the blocks that expand the histories for SimTier, in the first launch of a small call; FEW: its first blocks write the
// batch's tables.  KS: words of a signature.
// A small call is bound by its launches (2.2 us of host time each, the upload and an event besides) and by each kernel's chain of
// loads.  Three launches where seven were, chunks of a tenth of the history (up to 16 users) where they were of 1,024 items, LSH-DIN a wave to one
// tile of features: 1 x 100 candidates x 500 items (64 bits) 37.4 -> 21.6 us a call, 1 x 3,000 x 3,000 64.0 -> 31.8, 3 x 1,495 x 1,330
// (128 bits) 78.0 -> 39.7, 8 x 1,000 x 2,000 (128, fp32) 89.1 -> 48.8, 64 x 400 x 10^4 101.5 -> 87.6, 8 x 300 x 90,000 159 -> 146 (168
// with each request's expansion behind its own sums: the last sums began late; 191 with a piece a thread there).
struct LshStageArgs {
    LshFew few;
    LshModel m;
    LshBatch b;
    float *part;
    v4i *hist;
    size_t req_stride;
    int32_t part_stride, chunks, groups, expand, n_fill;        // chunks, groups, expand: blocks a request
};
constexpr int EXPAND_PIECES = 8;        // a thread's: the blocks have the registers of the sums, two to a compute unit
template <bool FEW, typename T, int VW, int KS>
__global__ __launch_bounds__(256, 2) void k_lsh_stage(LshStageArgs a)
{
    int idx = blockIdx.x;
    if constexpr (FEW) {
        if (idx < a.n_fill) {
            const int i = idx * 256 + (int)threadIdx.x;
            const auto args = kernel_arg<LshFew>(0);
            if (i < a.few.n_req) a.few.reqs[i] = arg_copy(&args->rd[i]);
            if (i < a.few.n_blk) {
                int r = 0;
                for (int q = 1; q < a.few.n_req; ++q)           // (a request without candidates has its successor's base)
                    if (args->rd[q].n_cand > 0 && i >= args->rd[q].cand_base / LSH_BLOCK) r = q;
                a.few.blk_req[i] = r;
            }
            return;
        }
        idx -= a.n_fill;
    }
    // the sums' blocks first, the longer ones
    const bool sums = idx < a.b.n_req * a.chunks * a.groups;
    if (!sums) idx -= a.b.n_req * a.chunks * a.groups;
    const int per = sums ? a.chunks * a.groups : a.expand, r = idx / per;
    idx -= r * per;
    LshReqDesc rd;
    if constexpr (FEW) rd = arg_copy(&kernel_arg<LshFew>(0)->rd[r]);
    else rd = a.b.reqs[r];
    if (sums) lsh_user_sums_block<T, VW, KS>(a.m, rd, r, idx % a.chunks, idx / a.chunks, a.part_stride, a.part);
    else lsh_expand_block<KS, EXPAND_PIECES>(rd, r, idx, a.hist, a.req_stride);
}

// columns a lane owns; and blocks a chunk takes: a lane's loads are at most eight bytes: four columns of fp32 leave no registers for
// a second wave a SIMD (1 x 10^3 candidates, 2,000 items, d' = d = 128: 92 us a call against 122)
static int user_sums_vw(const LshModel &m) { return m.d_out > 64 && m.dtype != 0 ? 4 : m.d_out > 32 ? 2 : 1; }
static int user_sums_groups(const LshModel &m)
{
    const int vw = user_sums_vw(m);
    return ((m.d_bits / 32 + 3) / 4) * ((m.d_out + 32 * vw - 1) / (32 * vw));
}
// f(storage type, words of a signature at most, columns a lane owns)
template <class F> static void user_sums_kernel(const LshModel &m, F &&f)
{
    const int vw = user_sums_vw(m);
    auto words = [&](auto t, auto w) {
        using T = decltype(t);
        if constexpr (sizeof(T) == 2)
            if (vw == 4) return f(t, w, std::integral_constant<int, 4>{});
        if (vw == 2) f(t, w, std::integral_constant<int, 2>{});
        else f(t, w, std::integral_constant<int, 1>{});
    };
    auto type = [&](auto t) {
        if (m.d_bits <= 32) words(t, std::integral_constant<int, 1>{});
        else if (m.d_bits <= 64) words(t, std::integral_constant<int, 2>{});
        else if (m.d_bits <= 128) words(t, std::integral_constant<int, 4>{});
        else words(t, std::integral_constant<int, 8>{});
    };
    if (m.dtype == 0) type(float{});
    else type(uint16_t{});
}

hipError_t launch_lsh_user_sums(const LshModel &m, const LshBatch &b, int grid_chunks, int part_stride, float *part, hipStream_t s)
{
    if (b.n_req == 0 || grid_chunks == 0) return hipSuccess;
    const dim3 grid(grid_chunks, b.n_req, user_sums_groups(m));
    user_sums_kernel(m, [&](auto t, auto w, auto vw) {
        hipLaunchKernelGGL((k_lsh_user_sums<decltype(t), decltype(vw)::value, decltype(w)::value>), grid, dim3(256), 0, s, m, b, part_stride, part);
    });
    return hipGetLastError();
}

hipError_t launch_lsh_stage(const LshModel &m, const LshBatch &b, const LshFew *few, int grid_chunks, int part_stride, float *part, void *hist,
                            size_t req_stride, int longest, hipStream_t s)
{
    if (b.n_req == 0) return hipSuccess;
    if (!hist || (m.d_bits != 32 && m.d_bits != 64 && m.d_bits != 128) || (few && (few->n_req != b.n_req || b.n_req > LSH_FEW))) return hipErrorInvalidValue;
    LshStageArgs a{};
    a.m = m;
    a.b = b;
    a.part = part;
    a.hist = (v4i *)hist;
    a.req_stride = req_stride;
    a.part_stride = part_stride;
    a.chunks = grid_chunks;
    a.groups = user_sums_groups(m);
    a.expand = ((longest + SMT_TILE - 1) / SMT_TILE * (m.d_bits / 32) * 64 + 256 * EXPAND_PIECES - 1) / (256 * EXPAND_PIECES);
    if (few) {
        a.few = *few;
        a.n_fill = (std::max(few->n_req, few->n_blk) + 255) / 256;
    }
    const dim3 grid(a.n_fill + b.n_req * (a.chunks * a.groups + a.expand));
    if (grid.x == 0) return hipSuccess;
    user_sums_kernel(m, [&](auto t, auto w, auto vw) {
        using T = decltype(t);
        constexpr int W = decltype(w)::value, VW = decltype(vw)::value;
        if constexpr (W <= 4) {
            if (few) hipLaunchKernelGGL((k_lsh_stage<true, T, VW, W>), grid, dim3(256), 0, s, a);
            else hipLaunchKernelGGL((k_lsh_stage<false, T, VW, W>), grid, dim3(256), 0, s, a);
        }
    });
    return hipGetLastError();
}

// the partial sums added in order (see launch_lsh_user_reduce)
__global__ __launch_bounds__(256) void k_lsh_user_reduce(LshModel m, LshBatch b, int part_stride, const float *__restrict__ part,
                                                         float *__restrict__ A)
{
    const int r = blockIdx.y, shares = lsh_chunks(m.fine, b.reqs[r].seq_len) * lsh_user_split(m.d_bits);
    const size_t n = (size_t)lsh_rows(m.d_bits) * m.d_out, nd = (size_t)m.d_bits * m.d_out;
    const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    const float *p = part + (size_t)r * part_stride * n;
    float *a = A + (size_t)r * n;
    if (i < nd) {
        a[i] = lsh_sum_parts(p + i, n, shares);
    } else if (i < nd + 2 * m.d_out) {
        const size_t j = i - nd, at = nd + (j < m.d_out ? LSH_TOTAL * m.d_out + j : LSH_LOWEST * m.d_out + j - m.d_out);
        const double t = lsh_sum_totals(p + at, n, m.d_out, shares) * (j < m.d_out ? 0.5 : 1.0 / m.d_bits);
        a[at] = (float)t;
        a[at + m.d_out] = (float)(t - (double)(float)t);
    } else if (i < nd + 2 * m.d_out + 8) {
        const size_t at = nd + (size_t)LSH_MAJORITY * m.d_out + (i - nd - 2 * m.d_out);
        a[at] = shares > 0 ? p[at] : 0.f;
    }
}

hipError_t launch_lsh_user_reduce(const LshModel &m, const LshBatch &b, int part_stride, const float *part, float *A, hipStream_t s)
{
    if (b.n_req == 0) return hipSuccess;
    const size_t n = (size_t)(m.d_bits + 2) * m.d_out + 8;      // a thread per element of D, total, lowest, and per word of the majority
    hipLaunchKernelGGL(k_lsh_user_reduce, dim3((unsigned)((n + 255) / 256), b.n_req), dim3(256), 0, s, m, b, part_stride, part, A);
    return hipGetLastError();
}

}  // namespace aif
