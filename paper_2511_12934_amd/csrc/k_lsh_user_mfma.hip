// The user side of Eq. 8 on the matrix cores.
//
// With the bits as signs, c = (-1)^bit, the similarity of candidate i and history item t is
//     m_it = (1/2) (1 + (1/d') sum_k c_ik c_tk),
// so Eq. 8 is, with U~_t the projected history embeddings,
//     DIN_i = (1/2) total + (1 / 2 d') sum_k c_ik D[k],   D[k] = sum_t c_tk U~_t,   total = sum_t U~_t:
// d' + 1 vectors that belong to the user alone, formed once per request.  D is a contraction over the history,
// (signs) [d' x l] times U~ [l x d].
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
// where there are fewer than four the chunk's items are shared out as well (lsh_user_split).  Loads run LSH_AHEAD
// steps of 16 items ahead; there is no barrier.  All partial sums are added in a fixed order, a function of the
// request's own history length and the model.
//
// What bounds it: the loads in flight (the history's bytes would take half the time).  10^5 items of 128-bit signatures
// and 128 bf16 features for 8 users (216 MB): 91 us, where a block that transposed both inputs through LDS, with two
// barriers and a memory round trip per 64 items and tables for either value of a bit, took 328; 10^4 items, 64 bits, 64
// features, 64 users: 35 against 68.
#include "aif_lsh_dev.h"

namespace aif {

typedef __bf16 lsh_bf16x8 __attribute__((ext_vector_type(8)));
typedef float lsh_f32x16 __attribute__((ext_vector_type(16)));

// T: storage of the embeddings; VW: neighbouring columns a lane owns (32 VW columns a block)
template <typename T, int VW>
__global__ __launch_bounds__(256) void k_lsh_user_sums(LshModel m, LshBatch b, int part_stride, float *__restrict__ part)
{
    constexpr int P = sizeof(T) == 4 ? 3 : 1, WORDS = sizeof(T) == 4 ? VW : (VW + 1) / 2;   // 32-bit words of a lane's columns
    constexpr int AHEAD = sizeof(T) == 4 && VW == 4 ? 2 : 4;                                 // steps of 16 items in flight
    typedef uint32_t vec __attribute__((ext_vector_type(WORDS)));
    const int d = m.d_out, db = m.d_bits, nb = db / 8, rts = db / 32, r = blockIdx.y;
    const int groups = (rts + 3) / 4, rg = blockIdx.z % groups, cg = blockIdx.z / groups;
    const LshReqDesc rd = b.reqs[r];
    const int chunk_len = lsh_chunk_len(rd.seq_len), t_lo = blockIdx.x * chunk_len;
    if (t_lo >= rd.seq_len) return;
    const int t_hi = min(rd.seq_len, t_lo + chunk_len);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, col = lane & 31, h = lane >> 5;
    const int split = lsh_user_split(db), rt = rg * 4 + wave % (4 / split), sub = wave / (4 / split);
    if (rt >= rts) return;
    const int n_steps = (t_hi - t_lo + 15) / 16;
    const int s_lo = (int)((long)n_steps * sub / split), s_hi = (int)((long)n_steps * (sub + 1) / split);

    const int j0 = (cg * 32 + col) * VW;
    const bool on = j0 < d;                                     // whole groups: d is a multiple of 16
    const uint8_t *sg = rd.seq_sigs + 4 * rt;
    const int bit = 8 * (col >> 3) + 7 - (col & 7);             // bit k of a signature: byte k / 8, first bit most significant

    lsh_f32x16 acc[VW];
    double tot[VW];                                             // 64 bits: see lsh_rows
#pragma unroll
    for (int f = 0; f < VW; ++f) {
        tot[f] = 0.0;
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[f][e] = 0.f;
    }
    vec buf[AHEAD][8];
    const T *rows = (const T *)rd.seq_emb + (size_t)t_lo * d;   // the same for every lane; row_at: the lane's first item of a step
    const uint32_t row_at = (uint32_t)(8 * h * d + (on ? j0 : 0));
    auto load = [&](int s, vec (&v)[8]) __attribute__((always_inline)) {
        const bool whole = t_lo + 16 * s + 16 <= t_hi;          // else the last item again, in place of those past the end
        const T *base = rows + (whole ? (size_t)16 * s * d : 0);
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const uint32_t at = whole ? row_at + (uint32_t)(i * d) : (uint32_t)(min(16 * s + 8 * h + i, t_hi - t_lo - 1) * d + (on ? j0 : 0));
            if constexpr (sizeof(T) == 2 && VW == 1) v[i][0] = base[at];
            else v[i] = *(const vec *)(base + at);
        }
    };
    auto load_sig = [&](int s) {                                // one item's word per lane, 64 items
        const int t = t_lo + 16 * s + lane;
        return *(const uint32_t *)(sg + (size_t)(t < t_hi ? t : t_hi - 1) * nb);
    };
    auto step = [&](int s, vec (&v)[8], uint32_t sig, int q) __attribute__((always_inline)) {
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
#pragma unroll
        for (int f = 0; f < VW; ++f) {
            if constexpr (P == 1) {
                uint32_t b4[4];
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    b4[i] = __builtin_amdgcn_perm(v[2 * i + 1][f >> 1], v[2 * i][f >> 1], f & 1 ? 0x07060302u : 0x05040100u);
                acc[f] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, __builtin_bit_cast(lsh_bf16x8, make_uint4(b4[0], b4[1], b4[2], b4[3])), acc[f], 0, 0, 0);
                if (rt == 0) {
                    float x[4];
#pragma unroll
                    for (int i = 0; i < 4; ++i) x[i] = __uint_as_float(b4[i] << 16) + __uint_as_float(b4[i] & 0xFFFF0000u);
                    tot[f] += (double)((x[0] + x[1]) + (x[2] + x[3]));
                }
            } else {
                lsh_bf16x8 p[P];
                float sum = 0.f;
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    float x = __uint_as_float(v[i][f]);
                    sum += x;
#pragma unroll
                    for (int k = 0; k < P; ++k) {
                        p[k][i] = (__bf16)x;
                        x -= (float)p[k][i];
                    }
                }
#pragma unroll
                for (int k = P - 1; k >= 0; --k) acc[f] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, p[k], acc[f], 0, 0, 0);
                if (rt == 0) tot[f] += (double)sum;
            }
        }
    };
    if (s_lo < s_hi) {
#pragma unroll
        for (int q = 0; q < AHEAD; ++q) load(s_lo + q, buf[q]);
        uint32_t sig = load_sig(s_lo);
        for (int s = s_lo; s < s_hi; s += 4) {
            const uint32_t next = load_sig(s + 4);
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if (s + q < s_hi) {
                    step(s + q, buf[q % AHEAD], sig, q);
                    load(s + q + AHEAD, buf[q % AHEAD]);
                }
            sig = next;
        }
    }
    float *out = part + ((size_t)r * part_stride + blockIdx.x * split + sub) * lsh_rows(db) * d;
    auto store = [&](float *p, const float *v) {
        if constexpr (VW == 4) *(float4 *)p = make_float4(v[0], v[1], v[2], v[3]);
        else if constexpr (VW == 2) *(float2 *)p = make_float2(v[0], v[1]);
        else *p = v[0];
    };
    if (on) {
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            float v[VW];
#pragma unroll
            for (int f = 0; f < VW; ++f) v[f] = acc[f][e];
            store(out + (size_t)(32 * rt + 8 * (e >> 2) + 4 * h + (e & 3)) * d + j0, v);
        }
    }
    if (rt == 0) {
#pragma unroll
        for (int f = 0; f < VW; ++f) tot[f] += __shfl_xor(tot[f], 32, 64);
        float v[2][VW];
#pragma unroll
        for (int f = 0; f < VW; ++f) {
            v[0][f] = (float)tot[f];
            v[1][f] = (float)(tot[f] - (double)v[0][f]);
        }
        if (on && h == 0) {
            store(out + (size_t)db * d + j0, v[0]);
            store(out + (size_t)(db + 1) * d + j0, v[1]);
        }
    }
}

hipError_t launch_lsh_user_sums(const LshModel &m, const LshBatch &b, int grid_chunks, int part_stride, float *part, hipStream_t s)
{
    if (b.n_req == 0 || grid_chunks == 0) return hipSuccess;
    const int vw = m.d_out > 64 ? 4 : m.d_out > 32 ? 2 : 1;
    const dim3 grid(grid_chunks, b.n_req, ((m.d_bits / 32 + 3) / 4) * ((m.d_out + 32 * vw - 1) / (32 * vw)));
    auto go = [&](auto kern) { hipLaunchKernelGGL(kern, grid, dim3(256), 0, s, m, b, part_stride, part); };
    if (m.dtype == 0) {
        if (vw == 4) go(k_lsh_user_sums<float, 4>);
        else if (vw == 2) go(k_lsh_user_sums<float, 2>);
        else go(k_lsh_user_sums<float, 1>);
    } else {
        if (vw == 4) go(k_lsh_user_sums<uint16_t, 4>);
        else if (vw == 2) go(k_lsh_user_sums<uint16_t, 2>);
        else go(k_lsh_user_sums<uint16_t, 1>);
    }
    return hipGetLastError();
}

// A[r][k][j] = D[k][j], A[r][d'][j] + A[r][d' + 1][j] = total[j]: the partial sums added in order
__global__ __launch_bounds__(256) void k_lsh_user_reduce(LshModel m, LshBatch b, int part_stride, const float *__restrict__ part,
                                                         float *__restrict__ A)
{
    const int r = blockIdx.y, shares = lsh_chunks(b.reqs[r].seq_len) * lsh_user_split(m.d_bits);
    const size_t n = (size_t)lsh_rows(m.d_bits) * m.d_out, nd = (size_t)m.d_bits * m.d_out;
    const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= nd + m.d_out) return;
    const float *p = part + (size_t)r * part_stride * n + i;
    float *a = A + (size_t)r * n + i;
    if (i < nd)
        *a = lsh_sum_parts(p, n, shares);
    else {
        const double t = lsh_sum_totals(p, n, m.d_out, shares);
        a[0] = (float)t;
        a[m.d_out] = (float)(t - (double)(float)t);
    }
}

hipError_t launch_lsh_user_reduce(const LshModel &m, const LshBatch &b, int part_stride, const float *part, float *A, hipStream_t s)
{
    if (b.n_req == 0) return hipSuccess;
    const size_t n = (size_t)(m.d_bits + 1) * m.d_out;          // a thread per element of D and of total
    hipLaunchKernelGGL(k_lsh_user_reduce, dim3((unsigned)((n + 255) / 256), b.n_req), dim3(256), 0, s, m, b, part_stride, part, A);
    return hipGetLastError();
}

}  // namespace aif
