// a6-a7 of the shape-agnostic path for large batches of a bf16 model with hidden layers of up to 128 features: a wave takes 32
// candidates from their workspace rows to their logits, with the activations in its registers.
//
// k_mlp_gen passes the activations of a block's 32 candidates through LDS: every block reads all weights from the L2s, waits for
// them behind its rows, and meets at two barriers a layer.  Here the result of two row tiles of 16 is, in place, the eight
// k-values a lane owes the next layer (whose weights are packed in that order), so nothing leaves the wave between the rows and
// the logit; the weights, one piece each, lie in LDS from the start, and there is no barrier after it.  The ->1 layer takes a pair
// of the last hidden layer's row tiles as it is made.  Blocks are persistent, one a compute unit; the next rows are asked
// for during the second layer.  The products, their order and the roundings are k_mlp_gen's: the same bits.  (fp32 weights are
// three pieces: they do not fit LDS, and pairs of row tiles passed through it a block at a time took 63 to 68 us where k_mlp_gen
// takes 60 for 16 users of 6,250 candidates, 160 -> 128 -> 64.)
//
// What bounds it: the vector ALU (an activation is made of three pieces: 5.5 instructions for each) and the products, which
// the two waves of a SIMD overlap in part.
#include "k_pieces.h"

#include <algorithm>
#include <type_traits>

namespace aif {

constexpr int CHAIN_PAIRS = 4;          // pairs of row tiles (k-steps of the next layer) of a hidden layer at most
constexpr int CHAIN_KS = 8;             // k-steps of layer 1 at most
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
constexpr size_t CHAIN_LDS = 160 * 1024;

constexpr uint32_t CHAIN_AGAIN = 0x7FC00001u;  // a logit that is to be formed again: no sum has these bits

constexpr int CHAIN_WAVES = 8;          // of a block: what the registers allow
constexpr int CHAIN_COLS = 2, CHAIN_TILE = 16 * CHAIN_COLS;      // column tiles of 16 candidates a wave takes at a time

struct GenChain {
    MlpGenericWeights w;
    int32_t ks1, q1, q2;                // k-steps of layer 1; pairs of row tiles of the hidden layers (q2 = 0: there is one)
    int32_t last_at, bias_at, plain_at; // bytes into LDS: the ->1 layer's weights, later layers' biases, the plain route's room (a wave each)
    int32_t widest;                     // floats of half a wave's plain room
};

// The candidate whose workspace row is x, by one wave in plain fp32 arithmetic (mlp_plain of k_generic.hip: the same sums): where a
// value that is not finite has come up.
__device__ __forceinline__ float chain_plain(const Model &m, const uint16_t *x, const MlpGenericWeights &w, const float *bias1, float *bufA, float *bufB)
{
    const int lane = threadIdx.x & 63;
    auto settle = [&]() {
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    };
    for (int k = lane; k < m.k1; k += 64) bufA[k] = bf2f(x[k]);
    settle();
    for (int l = 0; l < m.n_layers; ++l) {
        const int K = l == 0 ? m.k1 : m.dims[l], N = m.dims[l + 1];
        const float *wt = w.wt[l];
        for (int n = lane; n < N; n += 64) {
            float acc = l == 0 ? bias1[n] : (w.bias[l] ? w.bias[l][n] : 0.f);
            for (int k = 0; k < K; ++k) acc += wt[(size_t)k * N + n] * bufA[k];
            bufB[n] = l + 1 == m.n_layers ? acc : fmaxf(acc, 0.f);
        }
        settle();
        float *t = bufA;
        bufA = bufB;
        bufB = t;
    }
    return bufA[0];
}

// KS1: k-steps of layer 1, or one more.  Q1: pairs of row tiles of the first hidden layer, or one more.
template <int KS1, int Q1>
__global__ __launch_bounds__(64 * CHAIN_WAVES, 2) void k_mlp_gen_chain(Model m, Batch b, const uint16_t *__restrict__ X, GenChain gc, const float *__restrict__ bias1)
{
    constexpr int WV = CHAIN_WAVES, THREADS = 64 * WV, NC = CHAIN_COLS;
    extern __shared__ __align__(16) char lds[];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), col = lane & 15;
    int g = lane >> 4;                                          // (opaque in the loop: the compiler would keep what follows from it in registers)
    const int n_tiles = b.n_blk * (ROW_BLOCK / CHAIN_TILE), ks1 = gc.ks1, q1 = gc.q1, q2 = gc.q2, n_hidden = q2 > 0 ? 2 : 1;
    const int H1 = m.dims[1];

    // ---- weights and biases ---------------------------------------------------------------------------------
    const u32x4 *const w1 = (const u32x4 *)gc.w.pieces[0], *const w2 = (const u32x4 *)gc.w.pieces[1];
    const int n1 = 2 * ks1 * 64, n2 = 2 * q1 * 64;      // 16-byte pieces of a pair of row tiles
    const bf16x8 *const wl = (const bf16x8 *)(lds + gc.last_at) + lane;
    float *const bias2 = (float *)(lds + gc.bias_at);           // of the second hidden layer, zeros past its end; the ->1 layer's
    {
        const u32x4 *src = (const u32x4 *)gc.w.pieces[n_hidden];
        for (int i = tid; i < (q2 > 0 ? q2 : q1) * 64; i += THREADS) ((u32x4 *)(lds + gc.last_at))[i] = src[i];
        if (tid < 32 * CHAIN_PAIRS) bias2[tid] = n_hidden == 2 && gc.w.bias[1] && tid < m.dims[2] ? gc.w.bias[1][tid] : 0.f;
        if (tid == 32 * CHAIN_PAIRS) bias2[tid] = gc.w.bias[n_hidden] ? gc.w.bias[n_hidden][0] : 0.f;
        for (int i = tid; i < q1 * n1; i += THREADS) ((u32x4 *)lds)[i] = w1[i];
        for (int i = tid; i < q2 * n2; i += THREADS) ((u32x4 *)lds)[q1 * n1 + i] = w2[i];
    }
    auto pair_weights = [&](int s) __attribute__((always_inline)) { return (const bf16x8 *)lds + (s < q1 ? s * n1 : q1 * n1 + (s - q1) * n2) + lane; };

    // ---- candidates -------------------------------------------------------------------------------------------
    struct Tile {
        const int32_t *ids;
        float *logits, *scores;
        int n, slot;                                            // candidates from this tile on (0 or less: none)
    };
    auto describe = [&](int tile) __attribute__((always_inline)) {
        const int r = ((ArgPtr<int32_t>)b.blk_req)[min(tile, n_tiles - 1) / (ROW_BLOCK / CHAIN_TILE)];
        const ReqDesc rd = arg_copy((ArgPtr<ReqDesc>)b.reqs + max(r, 0));
        const int local = tile * CHAIN_TILE - rd.row_base;
        return Tile{as_global(rd.cand_ids) + local, as_global(rd.logits_out) + local, rd.scores_out ? as_global(rd.scores_out) + local : nullptr,
                    tile < n_tiles && r >= 0 ? rd.n_cand - local : -(1 << 20), rd.slot};
    };
    u32x4 raw[NC][KS1];
    auto ask_rows = [&](int tile) __attribute__((always_inline)) {
        const uint16_t *x = X + (size_t)min(tile, n_tiles - 1) * CHAIN_TILE * m.ldx;
#pragma unroll
        for (int n = 0; n < NC; ++n) {
            const uint32_t row = (uint32_t)((n * 16 + col) * m.ldx);
#pragma unroll
            for (int k = 0; k < KS1; ++k) {
                const int c = 32 * k + 8 * g;                   // (past the row's end, not before the last two k-steps: its start)
                raw[n][k] = *(const u32x4 *)(x + (row + (uint32_t)(k < KS1 - 2 || c < m.k1 ? c : 0)));
            }
        }
    };
    // layer 1's biases for pair q (past the layer's end some of its others: its weights are zero there, and so are the next layer's)
    auto bias_of = [&](const float *p, int q, f32x4 (&v)[2]) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < 2; ++i) v[i] = *(const f32x4 *)(p + min(32 * q + 16 * i + 4 * g, H1 - 4));
    };
    // a pair of row tiles over ksn k-steps, KS or one less: their eight values of this lane's candidate
    auto pair = [&](auto ks_c, auto px_c, const bf16x8 *w, const auto &x, int ksn, const f32x4 (&bias)[2], float (&v)[NC][8]) __attribute__((always_inline)) {
        constexpr int KS = decltype(ks_c)::value, PX = decltype(px_c)::value;
        f32x4 big[2][NC], small[2][NC];
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int n = 0; n < NC; ++n) {
                big[t][n] = bias[t];
                small[t][n] = f32x4{0.f, 0.f, 0.f, 0.f};
            }
        // mfma_pieces of both tiles; the weights are read a k-step ahead (the fences: all of them at once would not fit the registers)
        bf16x8 a[2][2];
        auto read = [&](int k) __attribute__((always_inline)) {
#pragma unroll
            for (int t = 0; t < 2; ++t) a[k & 1][t] = w[(t * ksn + k) * 64];
        };
        read(0);
#pragma unroll
        for (int k = 0; k < KS; ++k) {
            if (k == KS - 1 && KS > ksn) break;
            if (k + 1 < KS) read(k + 1);                        // (one past the last: it is read in bounds and not used)
#pragma unroll
            for (int j = PX - 1; j >= 0; --j)
#pragma unroll
                for (int t = 0; t < 2; ++t)
#pragma unroll
                    for (int n = 0; n < NC; ++n) {
                        f32x4 &c = j > 0 ? small[t][n] : big[t][n];
                        c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[k & 1][t], x[n][k].p[j], c, 0, 0, 0);
                    }
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int n = 0; n < NC; ++n)
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int j = 0; j < 4; ++j) v[n][4 * t + j] = big[t][n][j] + small[t][n][j];
    };

    int tile = blockIdx.x * WV + wave;
    const int stride = gridDim.x * WV;
    Tile next = describe(tile);
    ask_rows(tile);
    __syncthreads();
    bool any_odd = false;
    for (; tile < n_tiles; tile += stride) {
        asm volatile("" : "+v"(g));
        const Tile t = next;
        Pieces<1> x[NC][KS1];
#pragma unroll
        for (int n = 0; n < NC; ++n)
#pragma unroll
            for (int k = 0; k < KS1; ++k)
                x[n][k].p[0] = __builtin_bit_cast(bf16x8, k >= KS1 - 2 && 32 * k + 8 * g >= m.k1 ? u32x4{0, 0, 0, 0} : raw[n][k]);
        next = describe(tile + stride);
        if (t.n <= 0) {
            ask_rows(tile + stride);
            continue;
        }
        int id[NC];
#pragma unroll
        for (int n = 0; n < NC; ++n) id[n] = t.ids[max(min(n * 16 + col, t.n - 1), 0)];
        const float *b1 = bias1 + (size_t)t.slot * H1;

        f32x4 big[NC], small[NC], bias[2];
        auto last_layer = [&](int q, const auto &z) __attribute__((always_inline)) {
            const Pieces<1> a{{wl[q * 64]}};
#pragma unroll
            for (int n = 0; n < NC; ++n) mfma_pieces(a, z(n), big[n], small[n]);
        };
        auto activate = [&](float (&v)[8]) __attribute__((always_inline)) {
#pragma unroll
            for (int j = 0; j < 8; ++j) v[j] = relu_twice(v[j]);
            return split8<3>(v);
        };
        Pieces<3> y[NC][Q1];
        bias_of(b1, 0, bias);
        auto first_layer = [&](int q) __attribute__((always_inline)) {
            const bf16x8 *w = pair_weights(q);
            const f32x4 bq[2] = {bias[0], bias[1]};
            bias_of(b1, q + 1, bias);
            float v[NC][8];
            pair(std::integral_constant<int, KS1>{}, std::integral_constant<int, 1>{}, w, x, ks1, bq, v);
#pragma unroll
            for (int n = 0; n < NC; ++n) y[n][q] = activate(v[n]);
        };
#pragma unroll
        for (int q = 0; q < Q1 - 1; ++q) first_layer(q);
#pragma unroll
        for (int n = 0; n < NC; ++n) y[n][Q1 - 1] = Pieces<3>{};
        if (q1 == Q1) first_layer(Q1 - 1);
        ask_rows(tile + stride);
#pragma unroll
        for (int n = 0; n < NC; ++n) {
            big[n] = small[n] = f32x4{0.f, 0.f, 0.f, 0.f};
            big[n][0] = g == 0 ? bias2[32 * CHAIN_PAIRS] : 0.f;
        }
        if (q2 == 0) {
#pragma unroll
            for (int q = 0; q < Q1; ++q)
                if (q < Q1 - 1 || q1 == Q1) last_layer(q, [&](int n) -> const Pieces<3> & { return y[n][q]; });
        }
        for (int q = 0; q < q2; ++q) {
            const bf16x8 *w = pair_weights(q1 + q);
            const f32x4 bq[2] = {*(const f32x4 *)(bias2 + 32 * q + 4 * g), *(const f32x4 *)(bias2 + 32 * q + 16 + 4 * g)};
            float v[NC][8];
            pair(std::integral_constant<int, Q1>{}, std::integral_constant<int, 3>{}, w, y, q1, bq, v);
            last_layer(q, [&](int n) { return activate(v[n]); });
        }
#pragma unroll
        for (int n = 0; n < NC; ++n) {
            float z = big[n][0] + small[n][0];                  // of the lanes of group 0
            // a value that is not finite: the plain route, once all is done (nothing else need stay in registers then); until then
            // the logit says so
            const int c = n * 16 + col;
            any_odd |= __any(c < t.n && g == 0 && !isfinite(z));
            if (c < t.n && g == 0) {
                if (!isfinite(z)) z = __uint_as_float(CHAIN_AGAIN);
                if (id[n] < 0 || id[n] >= m.n_items) z = __uint_as_float(0x7FC00000u);
                t.logits[c] = z;
                if (t.scores) t.scores[c] = 1.0f / (1.0f + expf(-z));
            }
        }
    }
    if (!any_odd) return;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");            // the marks, which this wave reads again
    for (tile = blockIdx.x * WV + wave; tile < n_tiles; tile += stride) {
        const Tile t = describe(tile);
        for (int c = 0; c < min(t.n, CHAIN_TILE); ++c) {
            if (__float_as_uint(((const volatile float *)t.logits)[c]) != CHAIN_AGAIN) continue;
            float *room = (float *)(lds + gc.plain_at) + (size_t)wave * 2 * gc.widest;
            const float z = chain_plain(m, X + (size_t)(tile * CHAIN_TILE + c) * m.ldx, gc.w, bias1 + (size_t)t.slot * H1, room, room + gc.widest);
            if (lane == 0) {
                t.logits[c] = z;
                if (t.scores) t.scores[c] = 1.0f / (1.0f + expf(-z));
            }
        }
    }
}

static bool gen_chain_plan(const Model &m, const MlpGenericWeights &w, GenChain &gc, size_t &lds)
{
    const int n_hidden = m.n_layers - 1;
    if (m.dtype != 1 || n_hidden < 1 || n_hidden > 2 || m.x_tiled || m.cross_in_mlp) return false;
    if (m.dims[1] % 4 || (n_hidden == 2 && m.dims[2] % 4)) return false;        // biases are read four at a time
    gc = GenChain{};
    gc.w = w;
    gc.ks1 = (m.k1 + 31) / 32;
    gc.q1 = (m.dims[1] + 31) / 32;
    gc.q2 = n_hidden == 2 ? (m.dims[2] + 31) / 32 : 0;
    if (gc.ks1 < 1 || gc.ks1 > CHAIN_KS || gc.q1 > CHAIN_PAIRS || gc.q2 > CHAIN_PAIRS) return false;
    const size_t weights = (size_t)(gc.q1 * 2 * gc.ks1 + gc.q2 * 2 * gc.q1) * 1024;
    gc.last_at = (int32_t)weights;
    gc.bias_at = (int32_t)(weights + (size_t)(gc.q2 > 0 ? gc.q2 : gc.q1) * 1024);
    gc.plain_at = gc.bias_at + (32 * CHAIN_PAIRS + 4) * (int32_t)sizeof(float);
    gc.widest = std::max(m.k1, std::max(m.dims[1], m.dims[2]));
    lds = gc.plain_at + (size_t)CHAIN_WAVES * 2 * gc.widest * sizeof(float);
    return lds <= CHAIN_LDS;
}

// A block loads all weights before its first row and has two waves a SIMD, so a batch has to give most of its waves a tile.  Whole
// calls, us, k_mlp_gen | here (160 -> 128 -> 64 -> 1 over 50 items; tiles of 32 candidates, 256 units):
//    388 tiles 26.5 | 28.5    750: 30.3 | 31.7    1,000: 31.8 | 33.0    1,250: 40.4 | 37.2    2,000: 43.4 | 38.4    2,504: 54.6 | 50.7
//    5,008 81.9 | 67.7        7,512: 117.9 | 92.8
bool gen_chain_serves(const Model &m, const Batch &b)
{
    GenChain gc;
    size_t lds;
    return 2 * b.n_tiles >= 9 * compute_units() && gen_chain_plan(m, MlpGenericWeights{}, gc, lds);
}

template <int KS1, int Q1>
static hipError_t gen_chain_go(const Model &m, const Batch &b, const void *X, const GenChain &gc, size_t lds, const float *bias1, hipStream_t s)
{
    constexpr int WV = CHAIN_WAVES;
    auto kern = k_mlp_gen_chain<KS1, Q1>;
    (void)hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    const int units = (b.n_blk * (ROW_BLOCK / CHAIN_TILE) + WV - 1) / WV;
    hipLaunchKernelGGL(kern, dim3(std::min(units, compute_units())), dim3(64 * WV), lds, s, m, b, (const uint16_t *)X, gc, bias1);
    return hipGetLastError();
}

hipError_t launch_gen_chain(const Model &m, const Batch &b, const void *X, const MlpGenericWeights &w, const float *bias1, hipStream_t s)
{
    if (b.n_blk == 0) return hipSuccess;
    GenChain gc;
    size_t lds;
    if (!gen_chain_plan(m, w, gc, lds)) return hipErrorInvalidValue;
    auto go = [&](auto q) {
        constexpr int Q1 = decltype(q)::value;
        if (gc.ks1 <= 2) return gen_chain_go<2, Q1>(m, b, X, gc, lds, bias1, s);
        if (gc.ks1 <= 4) return gen_chain_go<4, Q1>(m, b, X, gc, lds, bias1, s);
        if (gc.ks1 <= 6) return gen_chain_go<6, Q1>(m, b, X, gc, lds, bias1, s);
        return gen_chain_go<8, Q1>(m, b, X, gc, lds, bias1, s);
    };
    return gc.q1 <= 2 ? go(std::integral_constant<int, 2>{}) : go(std::integral_constant<int, CHAIN_PAIRS>{});
}

}  // namespace aif
