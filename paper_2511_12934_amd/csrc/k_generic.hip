// Shape-agnostic kernels of fp32 precision: the whole path for fp32 models and
// for any model whose sizes the bf16 MFMA kernels do not cover.  The
// contractions run on the bf16 matrix instruction all the same: an fp32 value
// is the sum of three bf16 values (8 + 8 + 8 significant bits), and of the
// nine products of two such sums the six that reach fp32's last bit are
// accumulated in fp32 -- 2.6 times the rate of the fp32 matrix instruction,
// which has 1/16 of the bf16 one's.  Tensors stored in bf16 are one piece and
// cost accordingly less (three products against an fp32 activation).  Every
// candidate is a column of its own: results do not depend on how a candidate
// list is sliced into requests.
#include "k_pieces.h"
#include "k_stage.h"

#include <algorithm>
#include <type_traits>

namespace aif {

__device__ __forceinline__ float wave_max(float v)
{
#pragma unroll
    for (int o = 32; o; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
    return v;
}
__device__ __forceinline__ float wave_sum(float v)
{
#pragma unroll
    for (int o = 32; o; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// ---------------------------------------------------------------------------
// a2 -- user fold.  [u|e|a|c] W1^T = u W1u^T + [e|a|c] W1rest^T: the first
// term is the same for every candidate of a request (the paper's own point:
// interaction-independent work is done once, Sec. 2), so it becomes a
// per-request bias.  One thread per output feature.
// ---------------------------------------------------------------------------
template <typename T>
__global__ __launch_bounds__(256) void k_user_fold(Model m, Batch b, const float *__restrict__ w1u,
                                                   const float *__restrict__ b1, float *__restrict__ bias1)
{
    user_fold_block<T>(blockIdx.y, blockIdx.x, m, TableReqs{b}, w1u, b1, bias1);
}

hipError_t launch_user_fold(const Model &m, const Batch &b, const float *w1u, const float *b1, float *bias1,
                            hipStream_t s)
{
    if (b.n_req == 0) return hipSuccess;
    dim3 grid((m.dims[1] + FOLD_FEATS - 1) / FOLD_FEATS, b.n_slots);      // once per distinct user of the call
    if (m.dtype == 0)
        hipLaunchKernelGGL(k_user_fold<float>, grid, dim3(256), 0, s, m, b, w1u, b1, bias1);
    else
        hipLaunchKernelGGL(k_user_fold<uint16_t>, grid, dim3(256), 0, s, m, b, w1u, b1, bias1);
    return hipGetLastError();
}

// The same for a batch of at most FEW_MAX requests whose descriptors travel in the launch's arguments: its first blocks
// write the device tables the later kernels read (few_fill), the others fold.  One launch where an upload and the fold
// were two (one fp32 request of 1,000 candidates: 5 us of 29).
template <typename T, int N>
__global__ __launch_bounds__(256) void k_user_fold_few(FewFill f /* first: kernel_arg */, Model m, int n_fill, int quads, const float *__restrict__ w1u,
                                                       const float *__restrict__ b1, float *__restrict__ bias1)
{
    const int idx = blockIdx.x;
    if (idx < n_fill) {
        few_fill<N>(f, kernel_arg<FewFill>(0), idx * 256 + (int)threadIdx.x);
        return;
    }
    user_fold_block<T>((idx - n_fill) / quads, (idx - n_fill) % quads, m, FewReqs<N>{f, kernel_arg<FewFill>(0)}, w1u, b1, bias1);
}

hipError_t launch_user_fold_few(const Model &m, const FewFill &f, const float *w1u, const float *b1, float *bias1, hipStream_t s)
{
    if (f.n_req < 1 || f.n_req > FEW_MAX) return hipErrorInvalidValue;
    const int n_fill = (few_fill_items(f) + 255) / 256, quads = (m.dims[1] + FOLD_FEATS - 1) / FOLD_FEATS;
    const dim3 grid(n_fill + f.n_slots * quads);
    auto go = [&](auto kern) { hipLaunchKernelGGL(kern, grid, dim3(256), 0, s, f, m, n_fill, quads, w1u, b1, bias1); };
    const bool one = f.n_req == 1 && f.n_slots == 1;
    if (m.dtype == 0) {
        if (one) go(k_user_fold_few<float, 1>);
        else go(k_user_fold_few<float, FEW_MAX>);
    } else {
        if (one) go(k_user_fold_few<uint16_t, 1>);
        else go(k_user_fold_few<uint16_t, FEW_MAX>);
    }
    return hipGetLastError();
}

// four consecutive elements at p + f of a row of n; `quad`: n is a multiple of four and the row 4-element aligned
template <typename T> __device__ __forceinline__ void load4(const T *p, int f, int n, bool quad, float *v)
{
    if (quad) {
        float4 a = make_float4(0, 0, 0, 0);
        if (f < n) {
            if constexpr (sizeof(T) == 4) a = *(const float4 *)(p + f);
            else {
                const uint2 w = *(const uint2 *)(p + f);
                a = make_float4(__uint_as_float(w.x << 16), __uint_as_float(w.x & 0xFFFF0000u), __uint_as_float(w.y << 16),
                                __uint_as_float(w.y & 0xFFFF0000u));
            }
        }
        v[0] = a.x, v[1] = a.y, v[2] = a.z, v[3] = a.w;
    } else {
#pragma unroll
        for (int j = 0; j < 4; ++j) v[j] = f + j < n ? ld_f<T>(p + f + j) : 0.f;
    }
}

// ---------------------------------------------------------------------------
// a3-a5 -- query, target attention (Eq. 3 form, query := candidate) and the
// real-time half of the cross features (Sec. 3.3) for heads wider than
// GEN_MAX_HEAD: one wave per candidate, ATTN_TS candidates per block, all
// waves step through the phases together.
// Per wave LDS: e[d_item], q[d_attn], score[max_seq_len].
// ---------------------------------------------------------------------------
constexpr int ATTN_TS = 16;

// sum_k a(k) * b(k) for k in [0, n), in order, with the loads of sixteen terms (then eight) issued before the first
// is used: a loop of load-then-multiply is waited for once per term -- a memory round trip each.
template <int U, class FA, class FB> __device__ __forceinline__ void dot_batches(int n, int &k, float &acc, FA a, FB b)
{
    for (; k + U <= n; k += U) {
        float av[U], bv[U];
#pragma unroll
        for (int j = 0; j < U; ++j) {
            av[j] = a(k + j);
            bv[j] = b(k + j);
        }
#pragma unroll
        for (int j = 0; j < U; ++j) acc += av[j] * bv[j];
    }
}
template <class FA, class FB> __device__ __forceinline__ float dot_in_order(int n, float acc, FA a, FB b)
{
    int k = 0;
    dot_batches<16>(n, k, acc, a, b);
    dot_batches<8>(n, k, acc, a, b);
    for (; k < n; ++k) acc += a(k) * b(k);
    return acc;
}

template <typename T>
__global__ __launch_bounds__(256) void k_attn_generic(Model m, Batch b, T *__restrict__ X,
                                                      const float *__restrict__ wq, int per_wave)
{
    extern __shared__ __align__(16) float smem[];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int tile = blockIdx.x;
    const int r = b.blk_req[tile / (ROW_BLOCK / ATTN_TS)];
    if (r < 0) return;
    const ReqDesc rd = b.reqs[r];
    const int row0 = tile * ATTN_TS;
    const int local0 = row0 - rd.row_base;
    int nrows = rd.n_cand - local0;
    if (nrows <= 0) return;
    if (nrows > ATTN_TS) nrows = ATTN_TS;

    float *sh_e = smem + (size_t)wave * per_wave;
    float *sh_q = sh_e + m.d_item;
    float *sh_s = sh_q + m.d_attn;
    const T *K = (const T *)rd.seq_keys;
    const T *V = (const T *)rd.seq_vals;
    const T *uc = (const T *)rd.cross_vecs;
    const int L = rd.seq_len, dh = m.d_head, da = m.d_attn;
    const float scale = 1.0f / sqrtf((float)dh);

    for (int it = 0; it < ATTN_TS / 4; ++it) {
        const int c = it * 4 + wave;
        const bool on = c < nrows;
        T *xrow = X + (size_t)(row0 + c) * m.ldx;
        if (on)
            for (int k = lane; k < m.d_item; k += 64) sh_e[k] = ld_f<T>(xrow + k);
        __syncthreads();
        if (on)
            for (int q = lane; q < da; q += 64) {
                float acc;
                if (wq) {
                    const float *wr = wq + (size_t)q * m.d_item;
                    acc = dot_in_order(m.d_item, 0.f, [&](int k) { return wr[k]; }, [&](int k) { return sh_e[k]; });
                } else
                    acc = sh_e[q];
                sh_q[q] = acc;
            }
        __syncthreads();
        for (int h = 0; h < m.n_heads; ++h) {
            const int o = h * dh;
            float mx = -INFINITY;
            if (on)
                for (int t = lane; t < L; t += 64) {
                    const T *kr = K + (size_t)t * da + o;
                    float acc = dot_in_order(dh, 0.f, [&](int k) { return sh_q[o + k]; }, [&](int k) { return ld_f<T>(kr + k); });
                    acc *= scale;
                    sh_s[t] = acc;
                    mx = fmaxf(mx, acc);
                }
            mx = wave_max(mx);
            float sum = 0.f;
            if (on)
                for (int t = lane; t < L; t += 64) {
                    const float p = expf(sh_s[t] - mx);
                    sh_s[t] = p;
                    sum += p;
                }
            sum = wave_sum(sum);
            __syncthreads();
            if (on)
                for (int k = lane; k < dh; k += 64) {
                    const float acc = dot_in_order(L, 0.f, [&](int t) { return sh_s[t]; },
                                                   [&](int t) { return ld_f<T>(V + (size_t)t * da + o + k); });
                    st_f<T>(xrow + m.d_item + o + k, L > 0 ? acc / sum : 0.f);
                }
            __syncthreads();
        }
        if (on) {
            T *xc = xrow + m.d_item + da;
            if (m.cross_in_mlp) {
                // the MLP chain forms the Hadamard products itself, or the block is folded into the user's layer-1 weights
            } else if (m.cross_mode == 1) {
                for (int k = lane; k < m.d_item; k += 64) st_f<T>(xc + k, ld_f<T>(uc + k) * sh_e[k]);
            } else if (m.cross_mode == 2) {
                const int S = m.d_item / m.d_cv;
                for (int idx = lane; idx < m.d_cross; idx += 64) {
                    const int j = idx / S, sg = idx - j * S;
                    const float acc = dot_in_order(m.d_cv, 0.f, [&](int k) { return ld_f<T>(uc + (size_t)j * m.d_cv + k); },
                                                   [&](int k) { return sh_e[sg * m.d_cv + k]; });
                    st_f<T>(xc + idx, acc);
                }
            } else if (m.cross_mode == 3) {
                // Algorithm 1 step 4: the row's trailing n_cross entries weigh the user-side vectors
                const int w0 = m.d_item - m.n_cross;
                for (int idx = lane; idx < m.d_cv; idx += 64) {
                    const float acc = dot_in_order(m.n_cross, 0.f, [&](int j) { return sh_e[w0 + j]; },
                                                   [&](int j) { return ld_f<T>(uc + (size_t)j * m.d_cv + idx); });
                    st_f<T>(xc + idx, acc);
                }
            }
        }
        __syncthreads();
    }
}

// ---------------------------------------------------------------------------
// The same for heads of up to GEN_MAX_HEAD, on the matrix cores and with the
// gather (a1) inside.  A wave owns 16 candidates, the columns of every product,
// and a block of WV waves shares the request's keys:
//   Q^T = W_q E^T (a head's features in tiles of 16), S^T = K Q^T, O^T = V^T P^T.
// A 16x16 result leaves features (keys) 4 g + i of one candidate in a lane
// (g = lane / 16), and two such tiles are, in place, the eight k-values a lane
// owes the next product's B operand once K (V) is read in the same order:
// k-value j of group g is feature (key) 4 g + j of the first tile, or
// 16 + 4 g + j - 4 of the second.  Nothing is exchanged between lanes but the
// softmax maximum.  Keys go through LDS as pieces in fragment order, split by
// the block's threads: all at once where they fit, else 32 at a time (the next 32
// are on their way from memory meanwhile); the softmax is the running one, its
// rescaling skipped by a wave none of whose candidates found a larger score (a
// factor of exactly one otherwise: same bits).
//
// What bounds it: short histories (L = 50, d = 32) the chain id -> row -> query
// -> scores of a wave, which is why a block of resident keys takes no barrier and
// stays under 128 registers (four waves a SIMD); then the vector ALU -- per key
// and candidate one exponential and three pieces of the weight.  Measured (L <=
// 50, d_attn 32 of W_q, rows of 64): fp32, 16 users of 6,200 candidates on average
// 32 us, bf16, 16 x 10^4: 32 -- 230 + 13 and 312 + 10 with a wave per candidate on
// the vector ALU after a gather launch, 48 and 55 with the keys 32 at a time in
// blocks of four waves; fp32, one request of 1,000: 10.4 against 22 + 6.
// ---------------------------------------------------------------------------
constexpr int GEN_KEYS = 32;

// A product that is not contracted with the difference it goes into: exp(a s - max) with the rounded product in the maximum and
// the exact one in the difference overflows from scores of 10^9 on.
__device__ __forceinline__ float rounded_product(float a, float s)
{
#pragma clang fp contract(off)
    return a * s;
}

// One head of one candidate by one wave in plain fp32 arithmetic: where a product of pieces met a value that is not
// finite (an infinity is not the sum of three pieces), so that infinities and NaN propagate as plain fp32 has them.
template <typename T>
__device__ __noinline__ void attn_plain(const T *e, const T *K, const T *V, const float *wq, int d_item, int da, int dh, int o,
                                        int L, float scale, T *out)
{
    const int lane = threadIdx.x & 63;
    float q[2], acc[2] = {0.f, 0.f};
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        const int k = lane + 64 * s;
        q[s] = 0.f;
        if (k < dh) {
            if (wq)
                for (int j = 0; j < d_item; ++j) q[s] += wq[(size_t)(o + k) * d_item + j] * ld_f<T>(e + j);
            else
                q[s] = ld_f<T>(e + o + k);
        }
    }
    auto score = [&](int t) {
        const T *kr = K + (size_t)(t < L ? t : 0) * da + o;
        float a = 0.f;
        for (int k = 0; k < dh; ++k) a += __shfl(k < 64 ? q[0] : q[1], k & 63, 64) * ld_f<T>(kr + k);
        return rounded_product(a, scale);
    };
    float mx = -INFINITY, sum = 0.f;
    for (int t0 = 0; t0 < L; t0 += 64) {
        const float s = score(t0 + lane);
        if (t0 + lane < L) mx = fmaxf(mx, s);
    }
    mx = wave_max(mx);
    for (int t0 = 0; t0 < L; t0 += 64) {
        const float s = score(t0 + lane), p = t0 + lane < L ? expf(s - mx) : 0.f;
        sum += p;
        for (int i = 0; i < 64 && t0 + i < L; ++i) {
            const float pi = __shfl(p, i, 64);
#pragma unroll
            for (int s2 = 0; s2 < 2; ++s2)
                if (lane + 64 * s2 < dh) acc[s2] += pi * ld_f<T>(V + (size_t)(t0 + i) * da + o + lane + 64 * s2);
        }
    }
    sum = wave_sum(sum);
#pragma unroll
    for (int s = 0; s < 2; ++s)
        if (lane + 64 * s < dh) st_f<T>(out + lane + 64 * s, L > 0 ? acc[s] / sum : 0.f);
}

// exp(x) for x <= 0 to about 1 ulp: the hardware's 2^t of the rounded t = x log2(e), corrected by what the rounding left.
// NaN for -infinity and NaN: the caller's plain route then takes over.
__device__ __forceinline__ float exp_neg(float x)
{
    constexpr float L = 1.44269502162933349609375f, L_LO = 1.925963033500011e-8f, LN2 = 0.693147182464599609375f;
    const float t = x * L, e = fmaf(x, L_LO, fmaf(x, L, -t)), p = __builtin_amdgcn_exp2f(t);
    return fmaf(p, e * LN2, p);
}

// f over the four groups' values of a candidate, in every lane: (0, 1), (2, 3), then both -- as a butterfly over lanes 16 and 32 away has
// them for an f that commutes, on the vector ALU's own swaps.
template <class F> __device__ __forceinline__ float groups_join(float v, F f)
{
    const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = f(__uint_as_float(a[0]), __uint_as_float(a[1]));
    const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return f(__uint_as_float(b[0]), __uint_as_float(b[1]));
}

// v / s for 1 <= s, 1 / s rounded in r: the quotient's estimate and one correction round as the division does (Markstein), in three
// instructions instead of twelve -- nothing needs scaling where s is neither large nor small.
__device__ __forceinline__ float quotient(float v, float s, float r)
{
    const float q = v * r;
    return fmaf(fmaf(-q, s, v), r, q);
}

// fragments of a chunk of keys: K (key tile, k-step), then V (feature tile)
__host__ __device__ constexpr int gen_chunk_frags(int ft) { return (ft + 1) / 2 * 2 + ft; }

// FT: tiles of 16 features a head has.  WV: waves of the block, 16 candidates each at a time.  wqp: W_q as pieces,
// [head][query_tiles(FT)][k-step of 32][piece][64 lanes][8], rows past the head's width zero (pack_pieces).
// table null: the item rows are in the workspace.
// RES: the pieces of all the request's keys, of every head, are staged at once, in dynamic LDS, and the block walks a whole
// ROW_BLOCK of candidates with no further barrier; else 32 keys of one head at a time for 16 WV candidates.
// TILES: column tiles of the block from row0 on; frag: LDS for the keys, [head][chunk][fragment][piece][lane] (not RES: one chunk).
template <typename T, int FT, int WV, bool WQ, bool RES, int TILES>
__device__ __forceinline__ void attn_gen_block(const Model &m, const ReqDesc &rd, int row0, T *X, const T *__restrict__ table,
                                               const bf16x8 *__restrict__ wqp, const float *__restrict__ wq, int32_t *__restrict__ bad, bf16x8 *frag)
{
    constexpr int P = stored<T>::P, PQ = WQ ? 3 : P, KS = (FT + 1) / 2, VEC = 16 / sizeof(T);
    constexpr int FRAGS = gen_chunk_frags(FT);
    constexpr int PER = RES ? 2 : (FRAGS + WV - 1) / WV;        // fragments a wave has on their way
    static_assert(2 * KS == query_tiles(FT), "the query's tiles are those that are packed");
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), col = lane & 15, g = lane >> 4;
    const int local0 = row0 - rd.row_base;
    const int L = rd.seq_len, dh = m.d_head, da = m.d_attn, chunks = (L + GEN_KEYS - 1) / GEN_KEYS;
    const bool quad = (dh & 3) == 0;
    const float scale = 1.0f / sqrtf((float)dh);
    const T *K = (const T *)rd.seq_keys, *V = (const T *)rd.seq_vals;

    // One tile: the waves share its parts -- the first its attention, the second its row (and cross block), the others the keys.
    constexpr bool ROLES = TILES == 1;
    static_assert(!ROLES || (RES && WV >= 4), "a wave for each part");
    const int tile_first = ROLES ? 0 : wave;
    // the lane's candidate in a tile, and its id: asked for ahead
    auto cand = [&](int tile) {
        const int at = local0 + tile * 16 + col;
        return at < rd.n_cand ? at : rd.n_cand - 1;
    };
    int32_t raw = table ? rd.cand_ids[cand(tile_first)] : 0;

    // fragment f of the chunk of keys from t0, head columns from o: its eight values of this lane, and as pieces to LDS
    auto fetch = [&](int f, int t0, int o, float (&v)[8]) __attribute__((always_inline)) {
        if (f < 2 * KS) {
            const int kt = f / KS, s = f - kt * KS, t = t0 + 16 * kt + col;
            const T *kr = K + (size_t)(t < L ? t : L - 1) * da + o;
            load4<T>(kr, 32 * s + 4 * g, dh, quad, v);
            load4<T>(kr, 32 * s + 16 + 4 * g, dh, quad, v + 4);
        } else {
            const int k = 16 * (f - 2 * KS) + col;
            const T *vr = V + o + (k < dh ? k : 0);
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const int t = t0 + 4 * g + (j & 3) + 16 * (j >> 2);
                v[j] = ld_f<T>(vr + (size_t)(t < L ? t : L - 1) * da);
            }
        }
    };
    auto put = [&](int f, int t0, float (&v)[8], bf16x8 *to) __attribute__((always_inline)) {
        if (f < 2 * KS) {
            const int t = t0 + 16 * (f / KS) + col;
#pragma unroll
            for (int j = 0; j < 8; ++j) v[j] = t < L ? v[j] : 0.f;
        } else {
            const bool on = 16 * (f - 2 * KS) + col < dh;
#pragma unroll
            for (int j = 0; j < 8; ++j) v[j] = on && t0 + 4 * g + (j & 3) + 16 * (j >> 2) < L ? v[j] : 0.f;
        }
        const Pieces<P> pc = split8<P>(v);
#pragma unroll
        for (int q = 0; q < P; ++q) to[(f * P + q) * 64 + lane] = pc.p[q];
    };
    float kv[PER][8];                                           // the chunk of keys on its way
    auto fetch_chunk = [&](int t0, int o) __attribute__((always_inline)) {
#pragma unroll
        for (int it = 0; it < PER; ++it)
            if (wave + WV * it < FRAGS) fetch(wave + WV * it, t0, o, kv[it]);
    };
    auto put_chunk = [&](int t0) __attribute__((always_inline)) {
#pragma unroll
        for (int it = 0; it < PER; ++it)
            if (wave + WV * it < FRAGS) put(wave + WV * it, t0, kv[it], frag);
    };
    if constexpr (RES) {
        constexpr int FIRST = ROLES ? 2 : 0, DEAL = WV - FIRST; // dealt round the waves, PER at a time
        const int n = m.n_heads * chunks * FRAGS;
        for (int i0 = wave < FIRST ? n : wave - FIRST; i0 < n; i0 += PER * DEAL) {
#pragma unroll
            for (int it = 0; it < PER; ++it) {
                const int i = i0 + it * DEAL, c = i / FRAGS, h = c / chunks;
                if (i < n) fetch(i - c * FRAGS, (c - h * chunks) * GEN_KEYS, h * dh, kv[it]);
            }
#pragma unroll
            for (int it = 0; it < PER; ++it) {
                const int i = i0 + it * DEAL, c = i / FRAGS, h = c / chunks;
                if (i < n) put(i - c * FRAGS, (c - h * chunks) * GEN_KEYS, kv[it], frag + (size_t)c * FRAGS * P * 64);
            }
        }
    } else if (L > 0)
        fetch_chunk(0, 0);

    int n_bad = 0;
    if (ROLES ? wave > 1 : RES && local0 + wave * 16 >= rd.n_cand) {
        __syncthreads();                                        // nothing left but the barrier after the keys
        return;
    }
    for (int tile = tile_first; tile < TILES; tile += WV) {
        if (RES && local0 + tile * 16 >= rd.n_cand) break;
        // a1: the lane's candidate and its item row
        const int at = local0 + tile * 16 + col;
        const bool live = at < rd.n_cand;
        const int c = live ? at : rd.n_cand - 1;
        T *xr = X + (size_t)(rd.row_base + c) * m.ldx;
        const T *er = xr;
        auto locate = [&]() __attribute__((always_inline)) {
            if (!table) return;
            int64_t id = raw;
            if (id < 0 || id >= m.n_items) {
                id = 0;
                if (live && g == 0 && (!ROLES || wave == 0)) ++n_bad;
            }
            er = table + (size_t)id * m.d_item;
            if (tile + WV < TILES) raw = rd.cand_ids[cand(tile + WV)];
        };
        if (!ROLES || wave == 1) locate();
        // the row into the workspace, and the Hadamard block beside it
        if (!ROLES || wave == 1) {
            const T *uc = (const T *)rd.cross_vecs;
            const bool had = m.cross_mode == 1 && !m.cross_in_mlp;
            constexpr int U = 4;
            // the user's pieces asked for beside the row's, but where their 16 registers cost the second block of a unit: resident keys
            // of heads of up to 64 (those of fp32 with W_q have one block anyway)
            constexpr bool ASK = !(RES && !ROLES && FT == 4 && !(WQ && P == 3));
            const int pieces = m.d_item / VEC;
            if (table || had)
                for (int p0 = 0; p0 < pieces; p0 += 4 * U) {
                    uint4 v[U], w[U];
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        const int p = p0 + 4 * u + g;
                        v[u] = *(const uint4 *)(er + (size_t)(p < pieces ? p : 0) * VEC);
                    }
                    if (ASK && had)
#pragma unroll
                        for (int u = 0; u < U; ++u) w[u] = *(const uint4 *)(uc + (size_t)(p0 + 4 * u + g < pieces ? p0 + 4 * u + g : 0) * VEC);
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        const int p = p0 + 4 * u + g;
                        if (p >= pieces || !live) continue;
                        if (table) *(uint4 *)(xr + (size_t)p * VEC) = v[u];
                        if (had) {
                            if constexpr (!ASK) w[u] = *(const uint4 *)(uc + (size_t)p * VEC);
                            const T *e = (const T *)&v[u], *x = (const T *)&w[u];
                            __align__(16) T o[VEC];
#pragma unroll
                            for (int k = 0; k < VEC; ++k) st_f<T>(o + k, ld_f<T>(x + k) * ld_f<T>(e + k));
                            *(uint4 *)(xr + m.d_item + da + (size_t)p * VEC) = *(const uint4 *)o;
                        }
                    }
                }
        }
        if ((!ROLES || wave == 1) && !m.cross_in_mlp && (m.cross_mode == 2 || m.cross_mode == 3)) {
            const T *uc = (const T *)rd.cross_vecs;
            const int S = m.cross_mode == 2 ? m.d_item / m.d_cv : 1;
            T *xc = xr + m.d_item + da;
            if (live)
                for (int idx = g; idx < m.d_cross; idx += 4) {
                    float acc;
                    if (m.cross_mode == 2) {
                        const int j = idx / S, sg = idx - j * S;
                        acc = dot_in_order(m.d_cv, 0.f, [&](int k) { return ld_f<T>(uc + (size_t)j * m.d_cv + k); },
                                           [&](int k) { return ld_f<T>(er + sg * m.d_cv + k); });
                    } else      // Algorithm 1 step 4: the row's trailing n_cross entries weigh the user-side vectors
                        acc = dot_in_order(m.n_cross, 0.f, [&](int j) { return ld_f<T>(er + m.d_item - m.n_cross + j); },
                                           [&](int j) { return ld_f<T>(uc + (size_t)j * m.d_cv + idx); });
                    st_f<T>(xc + idx, acc);
                }
        }

        if (ROLES && wave == 1) {
            __syncthreads();                                    // the keys are staged
            return;
        }
        // W_q's k-steps, UQ at a time where there are registers for it
        constexpr int UQ = WQ && KS == 1 && !ROLES && P == 1 ? 2 : 1;
        constexpr bool ASK_WQ = RES || WV != 4 || KS * P <= 6;  // a k-step ahead (the widest fp32 heads' small blocks: 96 registers, which are not there)
        const int ksn = (m.d_item + 31) / 32;
        Pieces<P> wf[UQ][2 * KS];
        auto ask_wq_tile = [&](int h, int ks0, int f) __attribute__((always_inline)) {
            const bf16x8 *wh = wqp + (size_t)h * query_tiles(FT) * ksn * P * 64 + lane;
#pragma unroll
            for (int u = 0; u < UQ; ++u)
#pragma unroll
                for (int q = 0; q < P; ++q) wf[u][f].p[q] = wh[((size_t)(f * ksn + min(ks0 + u, ksn - 1)) * P + q) * 64];
        };
        auto ask_wq = [&](int h, int ks0) __attribute__((always_inline)) {
#pragma unroll
            for (int f = 0; f < 2 * KS; ++f) ask_wq_tile(h, ks0, f);
        };
        if (ROLES) locate();

        for (int h = 0; h < m.n_heads; ++h) {
            const int o = h * dh;
            if (!RES && h > 0 && L > 0) fetch_chunk(0, o);      // the first keys on their way (head 0's: since the start)
            // a3: the query, as pieces in the order of K's fragments
            Pieces<PQ> qf[KS];
            if constexpr (WQ) {
                f32x4 qb[2 * KS], qs[2 * KS];
#pragma unroll
                for (int f = 0; f < 2 * KS; ++f) qb[f] = qs[f] = f32x4{0.f, 0.f, 0.f, 0.f};
                if (ASK_WQ) ask_wq(h, 0);
                for (int ks0 = 0; ks0 < ksn; ks0 += UQ) {
                    Pieces<P> e[UQ];
#pragma unroll
                    for (int u = 0; u < UQ; ++u) e[u] = load_pieces(er + 32 * (ks0 + u) + 8 * g, m.d_item - 32 * (ks0 + u) - 8 * g);
#pragma unroll
                    for (int u = 0; u < UQ; ++u) {
                        if (ks0 + u >= ksn) continue;
#pragma unroll
                        for (int f = 0; f < 2 * KS; ++f) {
                            if (!ASK_WQ) ask_wq_tile(h, ks0, f);
                            mfma_pieces(wf[u][f], e[u], qb[f], qs[f]);
                        }
                    }
                    if (ASK_WQ && ks0 + UQ < ksn) ask_wq(h, ks0 + UQ);
                }
#pragma unroll
                for (int s = 0; s < KS; ++s) {
                    float v[8];
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        v[j] = qb[2 * s][j] + qs[2 * s][j];
                        v[4 + j] = qb[2 * s + 1][j] + qs[2 * s + 1][j];
                    }
                    qf[s] = split8<PQ>(v);
                }
            } else {
#pragma unroll
                for (int s = 0; s < KS; ++s) {
                    float v[8];
                    load4<T>(er + o, 32 * s + 4 * g, dh, quad, v);
                    load4<T>(er + o, 32 * s + 16 + 4 * g, dh, quad, v + 4);
                    qf[s] = split8<PQ>(v);
                }
            }
            if (RES && h == 0 && tile == wave) __syncthreads(); // the keys are staged

            // a4: the keys, 32 at a time
            f32x4 ob[FT], os[FT];
            float mx = -INFINITY, sum = 0.f;
#pragma unroll
            for (int f = 0; f < FT; ++f) ob[f] = os[f] = f32x4{0.f, 0.f, 0.f, 0.f};
            for (int ch = 0; ch < chunks; ++ch) {
                const int t0 = ch * GEN_KEYS;
                const bf16x8 *fr = frag + lane;
                if constexpr (RES) fr += (size_t)(h * chunks + ch) * FRAGS * P * 64;
                else {
                    __syncthreads();                            // the chunk before has been read
                    put_chunk(t0);
                    __syncthreads();
                    if (ch + 1 < chunks) fetch_chunk(t0 + GEN_KEYS, o);
                }
                float sc[8];
#pragma unroll
                for (int kt = 0; kt < 2; ++kt) {
                    f32x4 sb = {0.f, 0.f, 0.f, 0.f}, ss = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int s = 0; s < KS; ++s) {
                        Pieces<P> k;
#pragma unroll
                        for (int q = 0; q < P; ++q) k.p[q] = fr[((kt * KS + s) * P + q) * 64];
                        mfma_pieces(k, qf[s], sb, ss);
                    }
#pragma unroll
                    for (int i = 0; i < 4; ++i) sc[4 * kt + i] = rounded_product(sb[i] + ss[i], scale);
                }
                // keys past the end: an infinitely low score, whatever the others' (a lane may hold no other: its maximum is
                // then the other lanes'), and a weight of zero
                const bool ragged = t0 + GEN_KEYS > L;
                auto past = [&](int j) __attribute__((always_inline)) { return ragged && t0 + 4 * g + (j & 3) + 16 * (j >> 2) >= L; };
                if (ragged)
#pragma unroll
                    for (int j = 0; j < 8; ++j) sc[j] = past(j) ? -INFINITY : sc[j];
                auto higher = [](float a, float b) { return __builtin_elementwise_maximum(a, b); };      // three at a time; NaN stays
                const float top = groups_join(higher(higher(higher(sc[0], sc[1]), sc[2]), higher(higher(higher(sc[3], sc[4]), sc[5]), higher(sc[6], sc[7]))), higher);
                if (__any(top > mx)) {                          // (the first chunk: 0 times what is 0)
                    const float now = fmaxf(mx, top), f = ch == 0 ? 0.f : exp_neg(mx - now);
                    mx = now;
                    sum *= f;
#pragma unroll
                    for (int k = 0; k < FT; ++k)
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            ob[k][i] *= f;
                            os[k][i] *= f;
                        }
                }
                float p[8];
#pragma unroll
                for (int j = 0; j < 8; ++j) p[j] = exp_neg(sc[j] - mx);
                if (ragged)
#pragma unroll
                    for (int j = 0; j < 8; ++j) p[j] = past(j) ? 0.f : p[j];
                sum += ((p[0] + p[1]) + (p[2] + p[3])) + ((p[4] + p[5]) + (p[6] + p[7]));
                const Pieces<3> pf = split8<3>(p);
#pragma unroll
                for (int f = 0; f < FT; ++f) {
                    Pieces<P> v;
#pragma unroll
                    for (int q = 0; q < P; ++q) v.p[q] = fr[((2 * KS + f) * P + q) * 64];
                    mfma_pieces(v, pf, ob[f], os[f]);
                }
            }
            // the block's result; `odd` is NaN if a lane met a value that is not finite
            sum = groups_join(sum, [](float a, float b) { return a + b; });
            float odd = sum * 0.f;
            const float inv = 1.0f / sum;                       // sum: 1 (the highest score's weight) to L
#pragma unroll
            for (int f = 0; f < FT; ++f) {
                float v[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    v[i] = ob[f][i] + os[f][i];
                    odd = fmaf(v[i], 0.f, odd);
                    v[i] = L > 0 ? quotient(v[i], sum, inv) : 0.f;
                }
                const int k = 16 * f + 4 * g;
                T *out = xr + m.d_item + o + k;
                if (live && k < dh) {
                    if (!quad) {
#pragma unroll
                        for (int i = 0; i < 4; ++i)
                            if (k + i < dh) st_f<T>(out + i, v[i]);
                    } else if constexpr (sizeof(T) == 4)
                        *(float4 *)out = make_float4(v[0], v[1], v[2], v[3]);
                    else
                        *(uint2 *)out = make_uint2(f2bf(v[0]) | ((uint32_t)f2bf(v[1]) << 16), f2bf(v[2]) | ((uint32_t)f2bf(v[3]) << 16));
                }
            }
            unsigned long long again = __ballot(live && odd != odd);
            again = (again | again >> 16 | again >> 32 | again >> 48) & 0xFFFFull;       // per candidate
            while (again) {
                const int cc = __ffsll((unsigned long long)again) - 1;
                again &= again - 1;
                const uint64_t ep = __shfl((unsigned long long)(uintptr_t)er, cc, 64), xp = __shfl((unsigned long long)(uintptr_t)xr, cc, 64);
                attn_plain<T>((const T *)ep, K, V, WQ ? wq : nullptr, m.d_item, da, dh, o, L, scale, (T *)xp + m.d_item + o);
            }
        }
    }
    if (n_bad) atomicAdd(bad, n_bad);
}

template <typename T, int FT, int WV, bool WQ, bool RES>
__global__ __launch_bounds__(64 * WV, FT <= 2 ? 4 : 2) void k_attn_gen(Model m, Batch b, T *__restrict__ X, const T *__restrict__ table,
                                                                       const bf16x8 *__restrict__ wqp, const float *__restrict__ wq,
                                                                       int32_t *__restrict__ bad)
{
    extern __shared__ __align__(16) char dyn[];
    const int row0 = blockIdx.x * (RES ? ROW_BLOCK : 16 * WV);
    const int r = b.blk_req[row0 / ROW_BLOCK];
    if (r < 0) return;
    const ReqDesc rd = b.reqs[r];
    if (row0 - rd.row_base >= rd.n_cand) return;
    if constexpr (RES) attn_gen_block<T, FT, WV, WQ, RES, ROW_BLOCK / 16>(m, rd, row0, X, table, wqp, wq, bad, (bf16x8 *)dyn);
    else {
        __shared__ bf16x8 one[gen_chunk_frags(FT) * stored<T>::P * 64];
        attn_gen_block<T, FT, WV, WQ, RES, WV>(m, rd, row0, X, table, wqp, wq, bad, one);
    }
}

size_t attn_generic_lds_bytes(const Model &m, int max_seq_len)
{
    return (size_t)4 * (m.d_item + m.d_attn + max_seq_len) * sizeof(float);
}

bool attn_generic_gathers(const Model &m) { return m.d_head <= GEN_MAX_HEAD; }

// bytes of LDS the pieces of all keys of a history take
template <typename T, int FT> static size_t gen_keys_lds(const Model &m, int longest)
{
    return (size_t)m.n_heads * ((longest + GEN_KEYS - 1) / GEN_KEYS) * gen_chunk_frags(FT) * stored<T>::P * 1024;
}

template <typename T, int FT, int WV, bool RES>
static void attn_gen_go(const Model &m, const Batch &b, void *X, const void *table, const void *wqp, const float *wq, int32_t *bad,
                        size_t lds, hipStream_t s)
{
    const dim3 grid(RES ? b.n_blk : b.n_blk * (ROW_BLOCK / (16 * WV)));
    auto go = [&](auto kern, const void *wp, const float *w) {
        if (RES) (void)hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        hipLaunchKernelGGL(kern, grid, dim3(64 * WV), RES ? lds : 0, s, m, b, (T *)X, (const T *)table, (const bf16x8 *)wp, w, bad);
    };
    if (wq) go(k_attn_gen<T, FT, WV, true, RES>, wqp, wq);
    else go(k_attn_gen<T, FT, WV, false, RES>, nullptr, nullptr);
}

// Three forms of the same arithmetic (the same bits): a batch of many ROW_BLOCKs whose longest keys leave room for two
// blocks on a compute unit keeps them resident, a block of eight waves to a whole ROW_BLOCK; other large batches take blocks of
// eight waves and half a ROW_BLOCK, 32 keys at a time; small ones blocks of four.
// The lines, us a call with the keys resident | 32 at a time (one build; queries of W_q over rows of 64, a head of one hidden layer):
// heads of 32, blocks    fp32, 50 keys    fp32, 128 keys    bf16, 50 keys    bf16, 200 keys
//       384               69.7 |  68.8     73.2 |  74.0      42.0 |  41.9     56.6 |  53.6    (500 keys 84.5 | 76.5)
//       432               72.7 |  77.8     76.4 |  83.9      42.8 |  46.2     57.3 |  60.9
//       512               81.4 |  84.7     84.2 |  90.5      44.5 |  47.5     58.6 |  62.3
//       528               96.4 |  91.1    101.8 |  98.6      56.7 |  53.7     74.7 |  72.4
//       640              103.9 |  99.5    109.5 | 107.1      57.6 |  54.8     75.5 |  73.5
//       656              133.0 | 134.1    138.6 | 141.6      85.7 |  86.5                     (8 users; the others 16)
//       768              114.5 | 116.3    120.1 | 123.7      60.8 |  61.8     78.7 |  84.1
//       832              126.6 | 125.3    132.2 | 134.8      69.6 |  68.4     93.8 |  94.3    (bf16, 128 keys: 32 at a time 1.5 % faster)
//       960              136.1 | 140.2    141.8 | 150.2      71.0 |  73.5     95.1 | 103.1
//     1,024              141.3 | 145.5    149.9 | 155.3      72.0 |  74.8     96.0 | 104.3
//     1,120              159.6 | 156.4    169.4 | 168.8      82.4 |  81.1    111.4 | 114.5
//     1,280              186.2 | 183.4    192.8 | 194.9      84.9 |  87.5    113.5 | 124.5
//     2,048              369.5 | 370.7    380.2 | 381.7     168.5 | 173.9    212.7 | 231.6
//     2,560              459.6 | 458.3    472.4 | 469.5     206.6 | 213.6    261.0 | 285.8
// lists and histories of all lengths, 492: 82.6 |  85.5    85.9 |  92.1      48.4 |  50.3     60.6 |  61.7
//     653                111.5 | 105.8    116.6 | 112.6      65.0 |  60.1     80.0 |  72.5
//     731                117.4 | 113.8    124.7 | 121.7      66.9 |  62.7     80.5 |  76.8
//     969                139.0 | 141.3    146.4 | 151.8      74.6 |  75.1     93.2 |  93.1
//   1,255                181.3 | 177.8    191.9 | 191.3      89.7 |  87.8    109.7 | 109.7
//   1,922                334.4 | 334.4    345.0 | 343.4     149.3 | 151.4    177.9 | 184.0
// one request a block, of few candidates (30 and 100 keys):
//       600 of 130      118.8 | 124.6    130.4 | 136.8      63.2 |  67.1     73.1 |  77.8
//       800 of 100      138.1 | 154.4    148.1 | 171.8      65.5 |  75.5     75.2 |  90.7
// heads of 64, blocks     fp32, 50 keys    no W_q            bf16, 50 keys    bf16, 128 keys
//       128               54.4 |  42.3     50.0 |  40.5      38.1 |  30.7     42.3 |  33.8
//       144               54.1 |  56.1     50.9 |  51.6      34.6 |  40.5     39.5 |  47.9
//       384               91.6 |  87.4     73.9 |  80.1      49.3 |  56.1     56.4 |  66.4
//       512              101.4 | 110.5     90.2 | 100.8      50.5 |  65.6     57.8 |  79.9
//     1,280              250.4 | 269.4    233.0 | 247.1      97.3 | 131.3    113.2 | 166.6
// Blocks of resident keys go 256 at a time (two share a unit), half-ROW_BLOCKs at 128 ROW_BLOCKs a time: the streamed form is the faster where
// it saves half of one.  So, narrow heads: resident in the only round of 512 if it is 4/5 full; then from seven times 128 on by the parity, long
// histories also where the other rounds make up for the half (bf16) or nothing is lost (fp32, seven); not at six, where lists of all
// lengths lose 3 to 7 % and like ones gain 2 to 6, and fp32 of short histories not beyond eight (within 1.5 % either way).  Blocks of
// few candidates (5/8 full at most) always: their keys are staged once, not for either half.
// Wide ones as soon as half-ROW_BLOCKs, one to a unit, need a second round.  LDS: two blocks fit up to 80 KB; at 64 to 80 KB resident keys
// are 7 % faster on 2,560 blocks and 5 % slower on 640; at 96 to 128 KB (one block a unit) 7 to 35 % slower.
constexpr size_t GEN_RES_LDS = 64 * 1024;
static bool narrow_keys_stay(const Model &m, const Batch &b, int longest)
{
    const int n_blk = b.n_blk, units = compute_units(), half = units / 2, halves = (n_blk + half - 1) / half;
    if (n_blk <= 2 * units) return 5 * n_blk >= 8 * units;
    if (b.n_tiles <= n_blk * (ROW_BLOCK / X_TILE) * 5 / 8) return true;
    const bool lengthy = longest > 2 * GEN_KEYS, bf16 = m.dtype == 1;
    if (halves < 7) return false;
    if (halves % 2) return lengthy && (bf16 ? halves > 10 : halves == 7);
    return halves == 8 || lengthy || (bf16 && halves > 10);
}
template <typename T, int FT> static bool attn_gen_keys_stay(const Model &m, const Batch &b, int longest)
{
    return (FT <= 2 ? narrow_keys_stay(m, b, longest) : b.n_blk > compute_units() / 2) && gen_keys_lds<T, FT>(m, longest) <= GEN_RES_LDS;
}
template <typename T, int FT>
static void attn_gen_ft(const Model &m, const Batch &b, void *X, const void *table, const void *wqp, const float *wq, int32_t *bad,
                        int longest, hipStream_t s)
{
    if (attn_gen_keys_stay<T, FT>(m, b, longest)) attn_gen_go<T, FT, 8, true>(m, b, X, table, wqp, wq, bad, gen_keys_lds<T, FT>(m, longest), s);
    else if (b.n_blk >= compute_units() / 2) attn_gen_go<T, FT, 8, false>(m, b, X, table, wqp, wq, bad, 0, s);
    else attn_gen_go<T, FT, 4, false>(m, b, X, table, wqp, wq, bad, 0, s);
}
template <typename T>
static hipError_t attn_gen_launch(const Model &m, const Batch &b, void *X, const void *table, const void *wqp, const float *wq,
                                  int32_t *bad, int longest, hipStream_t s)
{
    static_assert(attn_gen_tiles(GEN_MAX_HEAD) * 16 == GEN_MAX_HEAD, "eight feature tiles hold the widest head");
    switch (attn_gen_tiles(m.d_head)) {
    case 1: attn_gen_ft<T, 1>(m, b, X, table, wqp, wq, bad, longest, s); break;
    case 2: attn_gen_ft<T, 2>(m, b, X, table, wqp, wq, bad, longest, s); break;
    case 4: attn_gen_ft<T, 4>(m, b, X, table, wqp, wq, bad, longest, s); break;
    case 8: attn_gen_ft<T, 8>(m, b, X, table, wqp, wq, bad, longest, s); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_attn_generic(const Model &m, const Batch &b, void *X, const float *wq, const void *wq_pieces, const void *table,
                               int32_t *bad, int max_seq_len, int longest, hipStream_t s)
{
    if (b.n_blk == 0) return hipSuccess;
    if (m.d_head <= GEN_MAX_HEAD)
        return m.dtype == 0 ? attn_gen_launch<float>(m, b, X, table, wq_pieces, wq, bad, longest, s)
                            : attn_gen_launch<uint16_t>(m, b, X, table, wq_pieces, wq, bad, longest, s);
    if (table) return hipErrorInvalidValue;                 // this kernel finds the item rows in the workspace
    const int per_wave = m.d_item + m.d_attn + max_seq_len;
    const size_t lds = attn_generic_lds_bytes(m, max_seq_len);
    dim3 grid(b.n_blk * (ROW_BLOCK / ATTN_TS));
    if (m.dtype == 0) {
        (void)hipFuncSetAttribute((const void *)k_attn_generic<float>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        hipLaunchKernelGGL(k_attn_generic<float>, grid, dim3(256), lds, s, m, b, (float *)X, wq, per_wave);
    } else {
        (void)hipFuncSetAttribute((const void *)k_attn_generic<uint16_t>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        hipLaunchKernelGGL(k_attn_generic<uint16_t>, grid, dim3(256), lds, s, m, b, (uint16_t *)X, wq, per_wave);
    }
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// a6-a7 -- MLP head (Sec. 1: a small MLP) over the virtual input
// [u | e | a | c]: the u block arrives as bias1 (user fold), the rest is the
// workspace row.  H^T = W X^T: a block holds 16 NC candidates (columns), its
// WV waves share out the row tiles; the activations of the layer that is
// read and of the one that is written lie in LDS in B-fragment order, and
// weights come as ready-made pieces from the L2s, two k-steps ahead.
// SPLIT: the activations lie there as their bf16 pieces (written once, read by
// every wave), 96 bytes a feature and 16 candidates; without it as fp32, split
// by each wave that reads them, 64 bytes: for layers so wide that only this
// fits a compute unit's LDS.
// What bounds it: a block's chain of round trips (descriptors, rows, weights from
// the L2s), so several blocks share a compute unit: a layer overwrites its input
// once every wave has read it, and a block is four waves and 32 candidates.
// Measured (160 -> 128 -> 64 -> 1, fp32): 10^5 candidates 59 us, where a thread per
// feature and 16 candidates on the vector ALU took 210 (81 with 64 candidates, eight
// waves a block; 61 with the pieces cut value by value); 1,000 candidates 7 against 30; bf16, 160,000
// candidates 44 against 301 (k_generic_chain.hip: 28).
// ---------------------------------------------------------------------------
constexpr int MLP_TS = 16;              // candidates of a column tile

// widest activation of the plain route, per candidate
__host__ __device__ inline int mlp_plain_widest(const Model &m)
{
    int widest = m.k1;
    for (int l = 1; l <= m.n_layers; ++l) widest = m.dims[l] > widest ? m.dims[l] : widest;
    return widest;
}

struct GenMlp {
    MlpGenericWeights w;
    int32_t off1;                       // bytes: where the second activation buffer starts; 0: layers overwrite their input
};

// MLP_TS candidates in plain fp32 arithmetic (see attn_plain), the results of those in `mask` stored: activations in LDS
// as [feature][MLP_TS].
template <typename T, int THREADS>
__device__ __forceinline__ void mlp_plain(const Model &m, const T *X, const MlpGenericWeights &w, const float *bias1, int us, int row0,
                                       int nrows, uint32_t mask, float *bufA, float *bufB, const ReqDesc &rd, int local0)
{
    const int k1 = m.k1;
    for (int idx = threadIdx.x; idx < k1 * MLP_TS; idx += THREADS) {
        const int c = idx / k1, k = idx - c * k1;
        bufA[k * MLP_TS + c] = c < nrows ? ld_f<T>(X + (size_t)(row0 + c) * m.ldx + k) : 0.f;
    }
    __syncthreads();
    for (int l = 0; l < m.n_layers; ++l) {
        const int K = l == 0 ? k1 : m.dims[l], N = m.dims[l + 1];
        const float *wt = w.wt[l];
        for (int i = threadIdx.x; i < N * MLP_TS; i += THREADS) {
            const int n = i / MLP_TS, c = i - n * MLP_TS;
            float acc = l == 0 ? bias1[(size_t)us * N + n] : (w.bias[l] ? w.bias[l][n] : 0.f);
            for (int k = 0; k < K; ++k) acc += wt[(size_t)k * N + n] * bufA[k * MLP_TS + c];
            bufB[i] = l + 1 == m.n_layers ? acc : fmaxf(acc, 0.f);
        }
        __syncthreads();
        float *t = bufA;
        bufA = bufB;
        bufB = t;
    }
    if ((int)threadIdx.x < nrows && (mask >> threadIdx.x & 1u)) {
        const int c = threadIdx.x;
        float z = bufA[c];
        const int64_t id = rd.cand_ids[local0 + c];
        if (id < 0 || id >= m.n_items) z = __uint_as_float(0x7FC00000u);
        rd.logits_out[local0 + c] = z;
        if (rd.scores_out) rd.scores_out[local0 + c] = 1.0f / (1.0f + expf(-z));
    }
    __syncthreads();
}

// one row tile's (RT = 1) or two row tiles' results for all NC column tiles: W rows x activations over ksn k-steps.  w holds
// k-steps 0 and 1; the next but one is asked for as soon as a step is done.
template <int PW, int PX, int RT, int NC, bool SPLIT>
__device__ __forceinline__ void mlp_rows(const bf16x8 *__restrict__ wp, int ksn, const char *act, int lane, Pieces<PW> (&w)[2][RT],
                                         f32x4 (&big)[RT][NC], f32x4 (&small)[RT][NC])
{
    auto step = [&](int ks, const Pieces<PW> (&a)[RT]) __attribute__((always_inline)) {
#pragma unroll
        for (int n = 0; n < NC; ++n) {
            Pieces<PX> x;
            if constexpr (SPLIT) {
                const bf16x8 *f = (const bf16x8 *)act + (size_t)(ks * PX * NC + n) * 64 + lane;
#pragma unroll
                for (int q = 0; q < PX; ++q) x.p[q] = f[q * NC * 64];
            } else {
                const float4 *f = (const float4 *)act + (size_t)(ks * NC + n) * 128 + lane;
                const float4 a0 = f[0], a1 = f[64];
                const float v[8] = {a0.x, a0.y, a0.z, a0.w, a1.x, a1.y, a1.z, a1.w};
                x = split8<PX>(v);
            }
#pragma unroll
            for (int i = 0; i < RT; ++i) mfma_pieces(a[i], x, big[i][n], small[i][n]);
        }
    };
    auto load = [&](int ks, Pieces<PW> (&a)[RT]) __attribute__((always_inline)) {
        ks = ks < ksn ? ks : ksn - 1;
#pragma unroll
        for (int i = 0; i < RT; ++i)
#pragma unroll
            for (int q = 0; q < PW; ++q) a[i].p[q] = wp[((size_t)(i * ksn + ks) * PW + q) * 64 + lane];
    };
    for (int ks = 0; ks < ksn; ks += 2) {
        step(ks, w[0]);
        load(ks + 2, w[0]);
        if (ks + 1 < ksn) {
            step(ks + 1, w[1]);
            load(ks + 3, w[1]);
        }
    }
}

// act: the block's LDS (mlp_gen_lds)
template <typename T, int NC, int WV, bool SPLIT>
__device__ __forceinline__ void mlp_gen_block(const Model &m, const ReqDesc &rd, int row0, const T *X, const GenMlp &gm,
                                              const float *__restrict__ bias1, char *act)
{
    constexpr int P = stored<T>::P;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, col = lane & 15, g = lane >> 4;
    const int local0 = row0 - rd.row_base, nrows = min(rd.n_cand - local0, 16 * NC);
    const MlpGenericWeights &w = gm.w;
    const bool in_place = gm.off1 == 0;
    // the ids of the candidates whose logits this lane stores (the first wave's, at the end): asked for now
    int32_t ids[NC];
#pragma unroll
    for (int n = 0; n < NC; ++n) ids[n] = rd.cand_ids[local0 + min(n * 16 + col, nrows - 1)];

    // layer 1's input: the workspace rows as fragments (rows past the request's end zero), a few loads at a time
    {
        constexpr int U = 3;
        const int n_frag = (m.k1 + 31) / 32 * NC;
        for (int i0 = wave; i0 < n_frag; i0 += U * WV) {
            float v[U][8];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int i = i0 + u * WV, ks = i / NC, c = (i - ks * NC) * 16 + col;
                load8<T>(X + (size_t)(row0 + (c < nrows ? c : 0)) * m.ldx + 32 * ks + 8 * g, i < n_frag && c < nrows ? m.k1 - 32 * ks - 8 * g : 0, v[u]);
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int i = i0 + u * WV, ks = i / NC, ct = i - ks * NC;
                if (i >= n_frag) break;
                if constexpr (SPLIT) {
                    const Pieces<P> p = split8<P>(v[u]);
#pragma unroll
                    for (int q = 0; q < P; ++q) ((bf16x8 *)act)[((size_t)(ks * P + q) * NC + ct) * 64 + lane] = p.p[q];
                } else {
                    float4 *f = (float4 *)act + (size_t)(ks * NC + ct) * 128 + lane;
                    f[0] = make_float4(v[u][0], v[u][1], v[u][2], v[u][3]);
                    f[64] = make_float4(v[u][4], v[u][5], v[u][6], v[u][7]);
                }
            }
        }
    }
    float odd[NC];                      // per candidate of the lane: NaN where a value that is not finite has reached the logit
#pragma unroll
    for (int n = 0; n < NC; ++n) odd[n] = 0.f;
    char *in = act, *out = act + gm.off1;
    for (int l = 0; l < m.n_layers; ++l) {
        const int K = l == 0 ? m.k1 : m.dims[l], N = m.dims[l + 1], ksn = (K + 31) / 32;
        const bool last = l + 1 == m.n_layers;
        const int nrt = last ? 1 : layer_tiles(N);
        const bf16x8 *wl = (const bf16x8 *)w.pieces[l];
        const float *bl = l == 0 ? bias1 + (size_t)rd.slot * N : w.bias[l];
        // row tiles rt .. rt + RT - 1; `first` once per layer and wave, with the layer's barriers
        auto rows = [&](auto rt_c, auto px_c, int rt, bool first) __attribute__((always_inline)) {
            constexpr int RT = decltype(rt_c)::value, PX = decltype(px_c)::value;
            const bf16x8 *wp = wl + (size_t)rt * ksn * P * 64;
            Pieces<P> a[2][RT];
            f32x4 big[RT][NC], small[RT][NC];
            const bool on = rt < nrt;
            if (on) {
#pragma unroll
                for (int s = 0; s < 2; ++s)
#pragma unroll
                    for (int i = 0; i < RT; ++i)
#pragma unroll
                        for (int q = 0; q < P; ++q) a[s][i].p[q] = wp[((size_t)(i * ksn + min(s, ksn - 1)) * P + q) * 64 + lane];
#pragma unroll
                for (int i = 0; i < RT; ++i)
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const int f = 16 * (rt + i) + 4 * g + j;
                        const float b0 = bl && f < N ? bl[f] : 0.f;
#pragma unroll
                        for (int n = 0; n < NC; ++n) {
                            big[i][n][j] = b0;
                            small[i][n][j] = 0.f;
                        }
                    }
            }
            if (first) __syncthreads();                         // the weights are on their way while the layer's input settles
            if (on) mlp_rows<P, PX, RT, NC, SPLIT>(wp, ksn, in, lane, a, big, small);
            if (first && in_place) __syncthreads();             // the input has been read by every wave
            if (!on) return;
#pragma unroll
            for (int i = 0; i < RT; ++i)
#pragma unroll
                for (int n = 0; n < NC; ++n) {
                    float v[4];
#pragma unroll
                    for (int j = 0; j < 4; ++j) v[j] = big[i][n][j] + small[i][n][j];
                    const int f = 16 * (rt + i) + 4 * g;
                    if (last) {
                        const int c = n * 16 + col;
                        odd[n] = fmaf(v[0], 0.f, odd[n]);
                        if (g == 0 && c < nrows) {
                            float z = v[0];
                            if (ids[n] < 0 || ids[n] >= m.n_items) z = __uint_as_float(0x7FC00000u);
                            rd.logits_out[local0 + c] = z;
                            if (rd.scores_out) rd.scores_out[local0 + c] = 1.0f / (1.0f + expf(-z));
                        }
                    } else {
                        const int ks = f >> 5, half = (f >> 4) & 1;         // in place: the next layer's weights are packed in this order
#pragma unroll
                        for (int j = 0; j < 4; ++j) v[j] = relu_twice(v[j]);
                        if constexpr (SPLIT) {
                            uint32_t lo[3], hi[3];
                            split2<3>(v[0], v[1], lo);
                            split2<3>(v[2], v[3], hi);
#pragma unroll
                            for (int q = 0; q < 3; ++q)
                                *(uint2 *)(out + (((size_t)(ks * 3 + q) * NC + n) * 64 + lane) * 16 + half * 8) = make_uint2(lo[q], hi[q]);
                        } else
                            ((float4 *)out)[(size_t)(ks * NC + n) * 128 + half * 64 + lane] = make_float4(v[0], v[1], v[2], v[3]);
                    }
                }
        };
        auto all = [&](auto px_c) __attribute__((always_inline)) {
            if (nrt >= 2 * WV) {
                rows(std::integral_constant<int, 2>{}, px_c, 2 * wave, true);
                for (int rt = 2 * (wave + WV); rt < nrt; rt += 2 * WV) rows(std::integral_constant<int, 2>{}, px_c, rt, false);
            } else {
                rows(std::integral_constant<int, 1>{}, px_c, wave, true);
                for (int rt = wave + WV; rt < nrt; rt += WV) rows(std::integral_constant<int, 1>{}, px_c, rt, false);
            }
        };
        if (P == 1 && l == 0) all(std::integral_constant<int, 1>{});
        else all(std::integral_constant<int, 3>{});
        char *t = in;
        in = out;
        out = t;
    }
    // a candidate that met one is done again in plain arithmetic -- it alone, whatever shares its block. First, with one
    // barrier, whether any did: the usual block leaves here (with the ids' load up there 16 fp32 requests of 6,250: 108.9
    // -> 107.0 us a call, bf16: 94.7 -> 92.6)
    int *any_odd = (int *)act;          // (the widest layers leave no LDS beside the activations)
    __syncthreads();
    {
        bool mine = false;
#pragma unroll
        for (int n = 0; n < NC; ++n) mine |= odd[n] != odd[n];
        const bool any = __any(mine);
        if (lane == 0) any_odd[wave] = any;
    }
    __syncthreads();
    int some = 0;
#pragma unroll
    for (int i = 0; i < WV; ++i) some |= any_odd[i];
    if (!some) return;
    uint32_t *flag = (uint32_t *)act, again[NC];
    __syncthreads();
    if (threadIdx.x < NC) flag[threadIdx.x] = 0;
    __syncthreads();
#pragma unroll
    for (int n = 0; n < NC; ++n)
        if (odd[n] != odd[n]) atomicOr(&flag[n], 1u << col);
    __syncthreads();
#pragma unroll
    for (int n = 0; n < NC; ++n) again[n] = flag[n];
    __syncthreads();
#pragma unroll
    for (int n = 0; n < NC; ++n)
        if (again[n] && n * MLP_TS < nrows)
            mlp_plain<T, 64 * WV>(m, X, w, bias1, rd.slot, row0 + n * MLP_TS, min(nrows - n * MLP_TS, MLP_TS), again[n], (float *)act,
                                  (float *)act + (size_t)mlp_plain_widest(m) * MLP_TS, rd, local0 + n * MLP_TS);
}

template <typename T, int NC, int WV, bool SPLIT>
__global__ __launch_bounds__(64 * WV, NC == 1 ? 2 : sizeof(T) == 4 ? 3 : 4) void k_mlp_gen(Model m, Batch b, const T *__restrict__ X, GenMlp gm, const float *__restrict__ bias1)
{
    extern __shared__ __align__(16) char act[];
    const int row0 = blockIdx.x * (16 * NC);
    const int r = b.blk_req[row0 / ROW_BLOCK];
    if (r < 0) return;
    const ReqDesc rd = b.reqs[r];
    if (row0 - rd.row_base >= rd.n_cand) return;
    mlp_gen_block<T, NC, WV, SPLIT>(m, rd, row0, X, gm, bias1, act);
}

// ---------------------------------------------------------------------------
// Both for few candidates: a block of eight waves takes one column tile of 16 from its table rows to its logits.  A small call
// is its launches and their starts; here the head follows in the block that formed the features.  The waves split the keys
// for the one that owns the tile, meet, and share out the head's row tiles; the features go through the workspace all the
// same (aif_peek_features shows them), a trip to the L2 and back.  The arithmetic is that of the two kernels: the same bits.
// (One fp32 request of 1,000 over 50 keys: 13.2 us where the two took 10.4 and 7.0; W_q's fragments asked for ahead of the row
// spill at two blocks a unit: 14.5.)
// ---------------------------------------------------------------------------
constexpr int GEN_TILE_WAVES = 8;
template <typename T, int FT, bool WQ>
__global__ __launch_bounds__(64 * GEN_TILE_WAVES, FT <= 2 ? 4 : 2) void k_gen_tile(Model m, Batch b, T *X, const T *__restrict__ table, const bf16x8 *__restrict__ wqp,
                                                                                  const float *__restrict__ wq, int32_t *__restrict__ bad, GenMlp gm,
                                                                                  const float *__restrict__ bias1)
{
    extern __shared__ __align__(16) char dyn[];                 // the keys, then the activations
    // the first tile of every ROW_BLOCK, then the second ..: tiles past a request's end come late, behind those with work
    const int blk = (int)blockIdx.x % b.n_blk, row0 = blk * ROW_BLOCK + (int)blockIdx.x / b.n_blk * 16;
    const int r = b.blk_req[blk];
    if (r < 0) return;
    const ReqDesc rd = b.reqs[r];
    if (row0 - rd.row_base >= rd.n_cand) return;
    attn_gen_block<T, FT, GEN_TILE_WAVES, WQ, true, 1>(m, rd, row0, X, table, wqp, wq, bad, (bf16x8 *)dyn);
    __syncthreads();                                            // the features are in memory, the keys have been read
    mlp_gen_block<T, 1, GEN_TILE_WAVES, true>(m, rd, row0, X, gm, bias1, dyn);
}

// Bytes of LDS a block of k_mlp_gen takes: one activation buffer where every hidden layer is done in one go (its results
// wait in registers until all waves have read its input), else two in turn; and at least what the plain route needs.
static size_t mlp_gen_lds(const Model &m, int nc, int waves, bool split, int32_t *off1)
{
    size_t need[2] = {0, 0};
    bool in_place = true;
    for (int l = 0; l < m.n_layers; ++l) {
        const size_t ks = ((l == 0 ? m.k1 : m.dims[l]) + 31) / 32;
        const size_t bytes = ks * nc * (split ? 1024u * (l == 0 && m.dtype == 1 ? 1 : 3) : 2048u);
        const int nrt = layer_tiles(m.dims[l + 1]);
        if (l + 1 < m.n_layers && nrt > (nrt >= 2 * waves ? 2 * waves : waves)) in_place = false;
        need[l & 1] = std::max(need[l & 1], bytes);
    }
    *off1 = in_place ? 0 : (int32_t)need[0];
    return std::max(in_place ? std::max(need[0], need[1]) : need[0] + need[1], mlp_generic_lds_bytes(m));
}

size_t mlp_generic_lds_bytes(const Model &m) { return (size_t)2 * mlp_plain_widest(m) * MLP_TS * sizeof(float); }

template <typename T, int NC, int WV, bool SPLIT>
static hipError_t mlp_gen_go(const Model &m, const Batch &b, const void *X, GenMlp &gm, const float *bias1, hipStream_t s)
{
    const size_t lds = mlp_gen_lds(m, NC, WV, SPLIT, &gm.off1);
    (void)hipFuncSetAttribute((const void *)k_mlp_gen<T, NC, WV, SPLIT>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    hipLaunchKernelGGL((k_mlp_gen<T, NC, WV, SPLIT>), dim3(b.n_blk * (ROW_BLOCK / (16 * NC))), dim3(64 * WV), lds, s, m, b, (const T *)X,
                       gm, bias1);
    return hipGetLastError();
}

// What k_generic_chain.hip leaves: blocks of four waves and 32 candidates where the batch fills the chip with such blocks and they fit, else eight waves
// share 16 candidates: the shortest chain.
template <typename T>
static hipError_t mlp_gen_launch(const Model &m, const Batch &b, const void *X, const MlpGenericWeights &w, const float *bias1, hipStream_t s)
{
    constexpr size_t LDS = 160 * 1024;
    GenMlp gm{w, 0};
    int32_t off;
    if (b.n_blk * (ROW_BLOCK / 32) >= compute_units() && mlp_gen_lds(m, 2, 4, true, &off) <= LDS) return mlp_gen_go<T, 2, 4, true>(m, b, X, gm, bias1, s);
    if (mlp_gen_lds(m, 1, 8, true, &off) <= LDS) return mlp_gen_go<T, 1, 8, true>(m, b, X, gm, bias1, s);
    return mlp_gen_go<T, 1, 8, false>(m, b, X, gm, bias1, s);
}

hipError_t launch_mlp_generic(const Model &m, const Batch &b, const void *X, const MlpGenericWeights &w,
                              const float *bias1, hipStream_t s)
{
    if (b.n_blk == 0) return hipSuccess;
    if (gen_chain_serves(m, b)) return launch_gen_chain(m, b, X, w, bias1, s);
    return m.dtype == 0 ? mlp_gen_launch<float>(m, b, X, w, bias1, s) : mlp_gen_launch<uint16_t>(m, b, X, w, bias1, s);
}

// k_gen_tile: batches whose keys, and the head's activations, fit a compute unit's LDS, of one round of blocks.  Whole calls, us, two
// launches | one, by candidates (a block to 16; two blocks a unit where LDS and registers allow):
//             160-128-64 fp32, 50 keys | bf16, 50 keys | fp32, 200 keys (one block a unit) | 192-512-256 fp32, 60 keys (one)
//         60        22.0 | 18.8           21.4 | 17.5      29.3 | 23.1                       34.7 | 30.1
//      1,000        23.5 | 18.9           20.8 | 18.5
//      4,000        26.1 | 20.6           23.3 | 19.1      31.8 | 24.2                       37.9 | 32.0
//      6,000                                               34.2 | 42.0                       50.3 | 57.2
//      8,000        30.1 | 24.1           25.7 | 21.4
//     12,000        32.2 | 34.6           26.7 | 29.7
template <typename T, int FT>
static size_t gen_tile_lds(const Model &m, int longest)
{
    int32_t off;
    return std::max(gen_keys_lds<T, FT>(m, longest), mlp_gen_lds(m, 1, GEN_TILE_WAVES, true, &off));
}
template <class F> static void gen_head_tiles(const Model &m, F &&f)       // f(storage type, tiles of 16 features of a head)
{
    auto type = [&](auto t) {
        switch (attn_gen_tiles(m.d_head)) {
        case 1: f(t, std::integral_constant<int, 1>{}); break;
        case 2: f(t, std::integral_constant<int, 2>{}); break;
        case 4: f(t, std::integral_constant<int, 4>{}); break;
        default: f(t, std::integral_constant<int, 8>{}); break;
        }
    };
    if (m.dtype == 0) type(float{});
    else type(uint16_t{});
}

bool attn_generic_keys_stay(const Model &m, const Batch &b, int longest)
{
    bool stay = false;
    if (m.d_head <= GEN_MAX_HEAD && b.n_blk > 0)
        gen_head_tiles(m, [&](auto t, auto ft) { stay = attn_gen_keys_stay<decltype(t), decltype(ft)::value>(m, b, longest); });
    return stay;
}

bool gen_tile_serves(const Model &m, const Batch &b, int longest)
{
    if (m.d_head > GEN_MAX_HEAD || b.n_blk == 0) return false;
    size_t lds = 0;
    gen_head_tiles(m, [&](auto t, auto ft) { lds = gen_tile_lds<decltype(t), decltype(ft)::value>(m, longest); });
    const int blocks_per_cu = attn_gen_tiles(m.d_head) <= 2 && lds <= 80 * 1024 ? 2 : 1;
    return lds <= 160 * 1024 && 2 * b.n_tiles <= blocks_per_cu * compute_units();
}

hipError_t launch_gen_tile(const Model &m, const Batch &b, void *X, const float *wq, const void *wq_pieces, const void *table, int32_t *bad,
                           int longest, const MlpGenericWeights &w, const float *bias1, hipStream_t s)
{
    if (b.n_blk == 0) return hipSuccess;
    if (!gen_tile_serves(m, b, longest)) return hipErrorInvalidValue;
    hipError_t e = hipSuccess;
    gen_head_tiles(m, [&](auto t, auto ft) {
        using T = decltype(t);
        constexpr int FT = decltype(ft)::value;
        GenMlp gm{w, 0};
        (void)mlp_gen_lds(m, 1, GEN_TILE_WAVES, true, &gm.off1);
        const size_t lds = gen_tile_lds<T, FT>(m, longest);
        auto go = [&](auto kern, const void *wp, const float *wf) {
            (void)hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
            hipLaunchKernelGGL(kern, dim3(b.n_blk * (ROW_BLOCK / 16)), dim3(64 * GEN_TILE_WAVES), lds, s, m, b, (T *)X, (const T *)table,
                               (const bf16x8 *)wp, wf, bad, gm, bias1);
            e = hipGetLastError();
        };
        if (wq) go(k_gen_tile<T, FT, true>, wq_pieces, wq);
        else go(k_gen_tile<T, FT, false>, nullptr, nullptr);
    });
    return e;
}

// ---------------------------------------------------------------------------
// Weights as pieces in A-fragment order: [group][row tile of 16][k-step of 32][piece][lane][8], lane (row = lane % 16,
// g = lane / 16) holding W[group rows_per_group + 16 rt + row][32 ks + 8 g + j]; zero outside the matrix.  hidden: column
// 32 ks + 16 (j / 4) + 4 g + j % 4 instead, the order in which two row tiles of a 16x16 result leave a lane its features, and half
// the weight (relu_twice).
// ---------------------------------------------------------------------------
template <typename T>
__global__ void k_pack_pieces(const T *__restrict__ w, int n_in, int col0, int rows, int ncols, int ksn, int rt_n, bool hidden, size_t total,
                              bf16x8 *__restrict__ out)
{
    constexpr int P = stored<T>::P;
    const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= total) return;
    const int lane = (int)(i & 63);
    const size_t f = i >> 6;                                    // (group, row tile, k-step)
    const int ks = (int)(f % ksn), rt = (int)(f / ksn % rt_n), group = (int)(f / ksn / rt_n);
    const int row = 16 * rt + (lane & 15);
    float v[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const int k = 32 * ks + (hidden ? 16 * (j >> 2) + 4 * (lane >> 4) + (j & 3) : 8 * (lane >> 4) + j);
        v[j] = (hidden ? 0.5f : 1.f) * (row < rows && k < ncols ? ld_f<T>(w + ((size_t)group * rows + row) * n_in + col0 + k) : 0.f);
    }
    const Pieces<P> p = split8<P>(v);
#pragma unroll
    for (int q = 0; q < P; ++q) out[(f * P + q) * 64 + lane] = p.p[q];
}

// Every head width: its feature tiles hold it, and the packed tiles hold its rows.
constexpr bool head_tiles_hold()
{
    for (int d = 1; d <= GEN_MAX_HEAD; ++d)
        if (attn_gen_tiles(d) * 16 < d || query_tiles(attn_gen_tiles(d)) < attn_gen_tiles(d)) return false;
    return true;
}
static_assert(head_tiles_hold(), "heads of every width up to GEN_MAX_HEAD");

size_t pieces_bytes(int dtype, int groups, int tiles, int ncols)
{
    return (size_t)groups * tiles * ((ncols + 31) / 32) * (dtype == 0 ? 3 : 1) * 1024;
}

hipError_t launch_pack_pieces(int dtype, const void *w, int groups, int rows, int tiles, int n_in, int col0, int ncols, bool hidden, void *out, hipStream_t s)
{
    if (16 * tiles < rows) return hipErrorInvalidValue;
    const int ksn = (ncols + 31) / 32, rt_n = tiles;
    const size_t total = (size_t)groups * rt_n * ksn * 64;
    const dim3 grid((unsigned)((total + 255) / 256));
    if (dtype == 0)
        hipLaunchKernelGGL(k_pack_pieces<float>, grid, dim3(256), 0, s, (const float *)w, n_in, col0, rows, ncols, ksn, rt_n, hidden, total, (bf16x8 *)out);
    else
        hipLaunchKernelGGL(k_pack_pieces<uint16_t>, grid, dim3(256), 0, s, (const uint16_t *)w, n_in, col0, rows, ncols, ksn, rt_n, hidden, total, (bf16x8 *)out);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// init-time repacking
// ---------------------------------------------------------------------------
template <typename T>
__global__ void k_pack_transposed(const T *__restrict__ w, int n_out, int n_in, int col0, int ncols,
                                  float *__restrict__ wt)
{
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= (size_t)ncols * n_out) return;
    const int k = (int)(i / n_out), n = (int)(i - (size_t)k * n_out);
    wt[i] = ld_f<T>(w + (size_t)n * n_in + col0 + k);
}

hipError_t launch_pack_transposed(int dtype, const void *w, int n_out, int n_in, int col0, int ncols, float *wt,
                                  hipStream_t s)
{
    const size_t total = (size_t)ncols * n_out;
    if (!total) return hipSuccess;
    dim3 grid((unsigned)((total + 255) / 256));
    if (dtype == 0)
        hipLaunchKernelGGL(k_pack_transposed<float>, grid, dim3(256), 0, s, (const float *)w, n_out, n_in, col0, ncols, wt);
    else
        hipLaunchKernelGGL(k_pack_transposed<uint16_t>, grid, dim3(256), 0, s, (const uint16_t *)w, n_out, n_in, col0, ncols, wt);
    return hipGetLastError();
}

template <typename T>
__global__ void k_to_f32(const T *__restrict__ src, int64_t rows, int cols, int ld_src, int col0,
                         float *__restrict__ dst)
{
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= (size_t)rows * cols) return;
    const int64_t rr = (int64_t)(i / cols);
    const int cc = (int)(i - (size_t)rr * cols);
    dst[i] = ld_f<T>(src + (size_t)rr * ld_src + col0 + cc);
}

hipError_t launch_to_f32(int dtype, const void *src, int64_t rows, int cols, int ld_src, int col0, float *dst,
                         hipStream_t s)
{
    const size_t total = (size_t)rows * cols;
    if (!total) return hipSuccess;
    dim3 grid((unsigned)((total + 255) / 256));
    if (dtype == 0)
        hipLaunchKernelGGL(k_to_f32<float>, grid, dim3(256), 0, s, (const float *)src, rows, cols, ld_src, col0, dst);
    else
        hipLaunchKernelGGL(k_to_f32<uint16_t>, grid, dim3(256), 0, s, (const uint16_t *)src, rows, cols, ld_src, col0, dst);
    return hipGetLastError();
}

}  // namespace aif
