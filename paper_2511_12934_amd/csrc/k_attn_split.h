// What the attention kernels share that give a tile of 32 candidates to a workgroup (k_attn_split in k_attn_mfma.hip,
// k_score_tile.hip), and the rules all attention kernels of the matrix cores go by.
#pragma once
#include "k_mfma.h"

namespace aif {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

// Streaming stores for the attention and cross blocks: they are written once and read by the next
// kernel, and lines left dirty in the eight L2s would have to be written back when the kernel ends.
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ void store_stream(bf16x8 *p, bf16x8 v) { __builtin_nontemporal_store(__builtin_bit_cast(u32x4, v), (u32x4 *)p); }
__device__ __forceinline__ void store_stream(bf16x4 *p, bf16x4 v) { __builtin_nontemporal_store(__builtin_bit_cast(u32x2, v), (u32x2 *)p); }

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
// acc + a[2i] b[2i] + a[2i + 1] b[2i + 1], i = 0..3, as four two-term dot products (one instruction each)
__device__ __forceinline__ float dot8(const bf16x8 &a, const bf16x8 &b, float acc)
{
    acc = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(a, a, 0, 1), __builtin_shufflevector(b, b, 0, 1), acc, false);
    acc = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(a, a, 2, 3), __builtin_shufflevector(b, b, 2, 3), acc, false);
    acc = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(a, a, 4, 5), __builtin_shufflevector(b, b, 4, 5), acc, false);
    acc = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(a, a, 6, 7), __builtin_shufflevector(b, b, 6, 7), acc, false);
    return acc;
}

// The first product is the weight's exponent in base 2.  Its size is bounded by |q| times the largest packed key norm;
// within this limit the exponent is used as it is -- weights between 2^-40 and 2^40, their sums far inside fp32, and the
// common factor cancels in the division -- beyond it the candidate's true maximum is found and subtracted.
constexpr float BOUND_LIMIT = 40.f;

// The streaming kernels sum a candidate's keys in KEY_PARTS runs of whole 64-key stages, run q = stages
// [q nst / KEY_PARTS, (q + 1) nst / KEY_PARTS), each run from zero, and add the runs' sums in the order of q.
// One wave walking all runs in turn (k_attn_mfma) and one wave per run (k_attn_split, for batches too small
// to fill the chip with a wave per 32 candidates) therefore give the same bits.
constexpr int KEY_PARTS = 8;
__host__ __device__ inline int key_part_begin(int q, int nst) { return q * nst / KEY_PARTS; }

// Whether a request's packed K/V of all heads fit in the LDS the resident kernel keeps them in.  A request is
// served by the resident kernel exactly when this holds (and the model has a resident kernel at all: the batch
// then has tile groups), whatever else is in the batch -- its bits do not depend on the company.
constexpr int RES_LDS_FRAGS = 152;            // 1 KB fragments of K/V that may stay resident
__host__ __device__ inline bool res_fits(const Model &m, int seq_len)
{
    const int nkt2 = ((((seq_len + 31) >> 5) + 1) & ~1);
    return (long)m.n_heads * nkt2 * (m.d_head / 8) <= RES_LDS_FRAGS;
}

// Floats a run leaves per head of DH: O's registers and the denominator, of 64 lanes.
template <int DH> constexpr int RUN_FLOATS = (DH / 32 * 16 + 1) * 64;

// Runs q0 .. q1 - 1 of one head for one tile by one wave: key tiles kt0 .. kt1 - 1, whole 64-key stages; end_of(q): the first tile
// past run q (looked at where a wave has several: MANY).  kvh: this lane's share of the head's packed keys and values, fragment i of
// tile t at kvh + (t FR + i) KB; kmh: the bounds of its key norms, a stage each.  query(): called when the first fragments have
// been asked for; q has to be there when it returns.  Run q's sums go to part + q RUN_FLOATS.
template <int DH, bool MANY, class EndOf, class Query>
__device__ __forceinline__ void attn_runs(const bf16x8 (&q)[DH / 16], const char *kvh, const float *kmh, int L, bool live, int lane, int kt0,
                                          int kt1, int q0, int q1, const EndOf &end_of, const Query &query, float *part)
{
    constexpr int FR = DH / 8, JS = DH / 16, FT = DH / 32, NREG = FT * 16;
    const int h = lane >> 5, nkt = (L + 31) >> 5, nst = (nkt + 1) >> 1;
    // the key-norm bounds are asked for first and looked at after the fragments have been asked for: a lane
    // takes stage `lane` (an index past the end re-reads the last stage: no condition, no wait on the spot)
    float km = nst > 0 ? kmh[lane < nst ? lane : nst - 1] : 0.f;
    // two sets of K fragments and two of V fragments take turns: while tile t's V and tile t + 1's K are in use,
    // tile t + 1's V and tile t + 2's K are in flight.  A tile index past the run re-reads the run's last tile
    // (fetched, not used), so the loop body has no conditions.
    const int ktl = kt1 > kt0 ? kt1 - 1 : 0;
    auto tile_src = [&](int kt) { return kvh + (size_t)(kt < ktl ? kt : ktl) * FR * 1024; };
    auto fetch_k = [&](bf16x8(&f)[JS], int kt) {
        const char *src = tile_src(kt);
#pragma unroll
        for (int i = 0; i < JS; ++i) f[i] = *(const bf16x8 *)(src + i * 1024);
    };
    auto fetch_v = [&](bf16x8(&f)[2 * FT], int kt) {
        const char *src = tile_src(kt) + JS * 1024;
#pragma unroll
        for (int i = 0; i < 2 * FT; ++i) f[i] = *(const bf16x8 *)(src + i * 1024);
    };
    // (the run's first K has a set of its own: a set that is both used and refilled ahead of the loop reaches the
    // loop through a register copy, and a copy of a register that a load is still filling waits for that load)
    bf16x8 k0[JS], ka[JS], kb[JS], va[2 * FT], vb[2 * FT];
    if (nkt > 0) {
        fetch_k(k0, kt0);
        fetch_k(kb, kt0 + 1);
        fetch_v(va, kt0);
        fetch_k(ka, kt0 + 2);
        fetch_v(vb, kt0 + 1);
    }
    for (int i = lane + 64; i < nst; i += 64) km = fmaxf(km, kmh[i]);       // sequences beyond 4096 keys

    query();
    float ss = 0.f;
#pragma unroll
    for (int j = 0; j < JS; ++j) ss = dot8(q[j], q[j], ss);
    ss += __shfl_xor(ss, 32, 64);
#pragma unroll
    for (int off = 32; off; off >>= 1) km = fmaxf(km, __shfl_xor(km, off, 64));
    float mc = sqrtf(ss) * 1.001f * km;
    const bool need_max = live && mc > BOUND_LIMIT;      // per candidate, as in k_attn_mfma
    const bool shifted = __any(need_max);                // the same in every lane: a scalar branch
    if (shifted) {
        // rare: the true maximum, by an extra pass over all of K in every wave (the maximum has no order)
        float mx = -INFINITY;
        for (int kt = 0; kt < nkt; ++kt) {
            const char *src = kvh + (size_t)kt * FR * 1024;
            f32x16 S;
#pragma unroll
            for (int i = 0; i < 16; ++i) S[i] = 0.f;
#pragma unroll
            for (int j = 0; j < JS; ++j)
                S = __builtin_amdgcn_mfma_f32_32x32x16_bf16(*(const bf16x8 *)(src + j * 1024), q[j], S, 0, 0, 0);
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int t = 32 * kt + 8 * (v >> 2) + 4 * h + (v & 3);
                if (t < L) mx = fmaxf(mx, S[v]);
            }
        }
        mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
        mc = need_max ? mx : 0.f;       // a candidate within the limit keeps its exponents as they are: x - 0 = x
    }

    f32x16 O[FT];
#pragma unroll
    for (int ft = 0; ft < FT; ++ft)
#pragma unroll
        for (int i = 0; i < 16; ++i) O[ft][i] = 0.f;
    float l4[4] = {0.f, 0.f, 0.f, 0.f};                 // as in k_attn_mfma
    // a finished run's sums go to LDS and the next run starts from zero
    int qn = q0;
    auto flush = [&]() {
        float *mine = part + (size_t)qn * (NREG + 1) * 64 + lane;
#pragma unroll
        for (int ft = 0; ft < FT; ++ft)
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                mine[(ft * 16 + i) * 64] = O[ft][i];
                O[ft][i] = 0.f;
            }
        mine[NREG * 64] = (l4[0] + l4[1]) + (l4[2] + l4[3]);
        l4[0] = l4[1] = l4[2] = l4[3] = 0.f;
        ++qn;
    };
    if (kt1 > kt0) {
        f32x16 S;
#pragma unroll
        for (int i = 0; i < 16; ++i) S[i] = 0.f;
#pragma unroll
        for (int j = 0; j < JS; ++j) S = __builtin_amdgcn_mfma_f32_32x32x16_bf16(k0[j], q[j], S, 0, 0, 0);
        // tile kt: exponentials of S (its scores), second product with vc (its V); meanwhile the S product of tile
        // kt + 1 from kn (after the run's last tile: of that tile again, unused); both sets are refilled, two tiles on
        auto body = [&](bf16x8(&vc)[2 * FT], bf16x8(&kn)[JS], int kt) {
            f32x16 Sn;
            float p[16];
            if (shifted) {              // rare: the candidate's maximum comes off every exponent (a scalar branch)
#pragma unroll
                for (int v = 0; v < 16; ++v) S[v] -= mc;
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int j = 0; j < JS; ++j) {
                if (j == 0) {
                    f32x16 Z;
#pragma unroll
                    for (int i = 0; i < 16; ++i) Z[i] = 0.f;
                    Sn = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kn[0], q[0], Z, 0, 0, 0);
                } else
                    Sn = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kn[j], q[j], Sn, 0, 0, 0);
#pragma unroll
                for (int v = 16 / JS * j; v < 16 / JS * (j + 1); ++v) {
                    p[v] = __builtin_amdgcn_exp2f(S[v]);
                    asm volatile("" : "+v"(p[v]));      // computed HERE: a value with no side effect would sink to its first use
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            fetch_k(kn, kt + 3);
            if (32 * kt + 32 > L) {
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int t = 32 * kt + 8 * (v >> 2) + 4 * h + (v & 3);
                    if (t >= L) p[v] = 0.f;
                }
            }
            bf16x8 P0, P1;
#pragma unroll
            for (int v = 0; v < 8; ++v) {
                P0[v] = (__bf16)p[v];
                P1[v] = (__bf16)p[8 + v];
            }
#pragma unroll
            for (int v = 0; v < 16; ++v) l4[v & 3] += p[v];
#pragma unroll
            for (int ft = 0; ft < FT; ++ft) {
                O[ft] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vc[ft], P0, O[ft], 0, 0, 0);
                O[ft] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vc[FT + ft], P1, O[ft], 0, 0, 0);
            }
            // the refill stays BEHIND the last use of the set (a load moved above it would need registers of its
            // own, and the copy back at the loop's end would wait for every load in flight)
            __builtin_amdgcn_sched_barrier(0);
            fetch_v(vc, kt + 2);
            __builtin_amdgcn_sched_barrier(0);
            S = Sn;
        };
        int bnd = end_of(qn);      // first tile of the next run
        for (int kt = kt0; kt < kt1; kt += 2) {
            if constexpr (MANY) {
                while (kt == bnd) {                     // a run ends here (empty runs: several)
                    flush();
                    bnd = end_of(qn);
                }
            }
            body(va, kb, kt);
            body(vb, ka, kt + 1);
        }
    }
    while (qn < q1) flush();              // the last run, and the empty ones around it
}

}  // namespace aif
