// a1, a3-a7 for few candidates: a workgroup takes ONE tile of 32 candidates from its table rows through target attention and the
// head to its logits.
//
// With fewer tiles than compute units the attention and the head are launches of a few microseconds each, most of it their start:
// tile -> request -> rows and weights, and for the head the trip of the tile's features through memory as well.  A candidate's
// head needs its own attention and nothing else, so the workgroup goes on with it: the runs' sums (k_attn_split) meet in
// LDS, the normalised attention joins the item row there as layer 1's column fragments, and the head's first weights are asked for
// as soon as a wave has done its keys.  The workspace rows are written all the same (aif_peek_features shows them).
//
// The arithmetic and its order are those of the kernels for larger batches, so a request's bits do not depend on its company: a
// request whose K/V the resident kernel would keep is summed as one run of keys, a wave to a head; a longer one (of one head)
// in KEY_PARTS runs shared out over the waves.
#include "k_attn_split.h"
#include "k_mlp_tile.h"

namespace aif {

template <int DH, class H> constexpr int score_tile_lds(int runs)
{
    const int parts = runs * RUN_FLOATS<DH> * 4;
    return H::kin(0) * 64 + (parts > H::lds_bytes ? parts : H::lds_bytes);
}

// K1, H1, H2: layer 1 over [item | attention], hidden widths (H2 = 0: one layer); DH: width of a head; NW: waves, KEY_PARTS or half
template <int DH, int K1, int H1, int H2, int NW>
__global__ __launch_bounds__(NW * 64, 2) void k_score_tile(Model m, Batch b, char *__restrict__ X, XLayout xl, const char *__restrict__ kvpack,
                                                           size_t pack_stride, const float *__restrict__ kmax, int nktp,
                                                           const char *__restrict__ table, int32_t *__restrict__ bad, MlpPack pk,
                                                           const float *__restrict__ bias1)
{
    using H = TileHead<K1, H1, H2, 0, NW>;
    constexpr int JS = DH / 16, FT = DH / 32, NREG = FT * 16, RPW = KEY_PARTS / NW, RUN = RUN_FLOATS<DH>;
    constexpr int EP = (K1 / 16 + NW - 1) / NW;                 // k-steps of the item row a wave moves at most
    extern __shared__ __align__(16) char lds[];                 // the tile's rows as column fragments; the runs' sums, then the head's
    char *const work = lds + K1 * 64;
    float *const part = (float *)work;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), col = lane & 31, h = lane >> 5;
    // the first tile of every ROW_BLOCK, then the second ..: tiles past a request's end come late, behind those with work
    const int blk = (int)blockIdx.x % b.n_blk, tile = blk * (ROW_BLOCK / 32) + (int)blockIdx.x / b.n_blk, r = b.blk_req[blk];
    if (r < 0) return;
    const ReqDesc rd = b.reqs[r];
    const int local0 = tile * 32 - rd.row_base, local = local0 + col;
    if (local0 >= rd.n_cand) return;                            // the rest of the request's last ROW_BLOCK
    const bool live = local < rd.n_cand;
    const int64_t raw = rd.cand_ids[live ? local : rd.n_cand - 1];
    const int L = rd.seq_len, HD = m.n_heads, nst = (((L + 31) >> 5) + 1) >> 1;
    const bool resident = b.n_groups > 0 && res_fits(m, L);     // one run of keys a head; else (one head) KEY_PARTS runs
    const char *kv = kvpack + (size_t)rd.slot * pack_stride + lane * 16;
    char *xrow = X + x_offset(xl, tile * 32 + col, 0);
    auto piece = [&](int p) { return xrow + (size_t)p * xl.piece_stride; };

    // the item row of the lane's candidate, in the table or in the workspace; its pieces into LDS (and the workspace), shared out
    bool inside = true;
    const char *erow = xrow;
    size_t estride = xl.piece_stride;
    auto rows = [&](bf16x8 (&q)[JS], int hd, bool first) __attribute__((always_inline)) {
        if (first) {
            inside = raw >= 0 && raw < m.n_items;
            if (table) {
                erow = table + (size_t)(inside ? raw : 0) * (size_t)(m.d_item * 2);
                estride = 16;
            }
        }
#pragma unroll
        for (int j = 0; j < JS; ++j) q[j] = *(const bf16x8 *)(erow + (hd * (DH / 8) + 2 * j + h) * estride);
        if (!first) return;
        bf16x8 e[EP];
#pragma unroll
        for (int i = 0; i < EP; ++i) {
            const int j = wave + i * NW;
            e[i] = *(const bf16x8 *)(erow + (2 * (j < m.d_item / 16 ? j : 0) + h) * estride);
        }
#pragma unroll
        for (int i = 0; i < EP; ++i) {
            const int j = wave + i * NW;
            if (j >= m.d_item / 16) continue;
            *(bf16x8 *)(lds + j * 1024 + lane * 16) = e[i];
            if (table && live) store_stream((bf16x8 *)piece(2 * j + h), e[i]);
        }
    };

    bool first = true;
    bf16x8 q[JS];
    for (int i = wave; i < (resident ? HD : NW); i += NW) {
        const int hd = resident ? i : 0, q0 = resident ? i : RPW * wave, q1 = resident ? i + 1 : RPW * (wave + 1);
        const int kt0 = resident ? 0 : 2 * key_part_begin(q0, nst), kt1 = resident ? 2 * nst : 2 * key_part_begin(q1, nst);
        attn_runs<DH, (RPW > 1)>(q, kv + (size_t)hd * nktp * (DH / 8) * 1024, kmax + ((size_t)rd.slot * HD + hd) * (nktp / 2), L, live, lane,
                                 kt0, kt1, q0, q1, [&](int qn) { return resident ? 0x7FFFFFFF : 2 * key_part_begin(qn + 1, nst); },
                                 [&]() { rows(q, hd, first); }, part);
        first = false;
    }
    if (first) rows(q, 0, true);                                // a wave without keys
    if (table && wave == 0 && h == 0 && live && !inside) atomicAdd(bad, 1);

    // the head's first weights are on their way while the runs' sums are added
    const char *w0 = pk.w0_user + (size_t)rd.slot * pk.w0_stride;
    const float *b0 = bias1 + (size_t)rd.slot * H1;
    TileMlp<H> mlp(work, lane, wave);
    const f32x4 wl = ((const f32x4 *)pk.wlast)[threadIdx.x < H::HL / 4 ? threadIdx.x : 0];
    const float blast = pk.blast[0];
    mlp.template ask<0>(w0, b0);
    mlp.ask_later(pk);
    tile_settle();
    // in the order of the runs, from zero; wave w normalises quads w, w + NW, ..
    for (int g = wave; g < HD * FT * 4; g += NW) {
        const int hd = g / (FT * 4), gq = g - hd * FT * 4;
        float lt = 0.f, t[4] = {0.f, 0.f, 0.f, 0.f};
        auto add = [&](int run) {
            const float *p = part + (size_t)run * RUN + lane;
            lt += p[NREG * 64];
#pragma unroll
            for (int i = 0; i < 4; ++i) t[i] += p[(4 * gq + i) * 64];
        };
        if (resident) add(hd);
        else
#pragma unroll
            for (int run = 0; run < KEY_PARTS; ++run) add(run);
        lt += __shfl_xor(lt, 32, 64);
        const float inv = L > 0 ? 1.0f / lt : 0.f;
        bf16x4 o4;
#pragma unroll
        for (int i = 0; i < 4; ++i) o4[i] = (__bf16)(t[i] * inv);
        // quad gq: features 8 gq + 4 h + i of the head, half h of one piece
        const int p = (m.d_item + hd * DH) / 8 + gq;
        *(bf16x4 *)(lds + p * 512 + col * 16 + 8 * h) = o4;
        if (live) store_stream((bf16x4 *)piece(p) + h, o4);
    }
    tile_settle();
    if (threadIdx.x < H::HL / 4) *(f32x4 *)(work + H::wl_at + threadIdx.x * 16) = wl;      // (where the runs' sums were)
    bf16x8 xin[K1 / 16];
#pragma unroll
    for (int j = 0; j < K1 / 16; ++j) xin[j] = *(const bf16x8 *)(lds + j * 1024 + lane * 16);
    mlp.run(pk, w0, b0, xin);
    if (wave != 0) return;
    float z = mlp.logit(blast);
    if (live && h == 0) {
        if (!inside) z = __uint_as_float(0x7FC00000u);
        rd.logits_out[local] = z;
        if (rd.scores_out) rd.scores_out[local] = 1.0f / (1.0f + __expf(-z));
    }
}

// Two workgroups of four waves share a compute unit, so a batch of at most two tiles a unit is one round; up to one a unit the
// workgroups have eight.  Where all histories are streamed the launch stands against k_attn_mfma, whose waves walk the whole history,
// for longer.  Whole calls, us, two launches | one (at the widths of the head given):
//   tiles     256-512-256, 100 items | 500 items | 256-256-128, 100 items | 1,000 items | 512-256, 200 items
//      3 (71) 24.7 | 17.8                          20.1 | 16.1              21.5 | 18.4   21.7 | 16.3 (100 items)
//    250      27.8 | 20.3                          22.6 | 18.3              24.2 | 20.4   25.2 | 19.1 (100 items)
//    313      28.6 | 24.0     31.3 | 26.6          23.6 | 20.5              27.7 | 24.3   28.7 | 23.2
//    512      28.9 | 24.8     32.1 | 27.7          24.2 | 21.7                            28.5 | 23.8
//    564      29.3 | 30.7     32.7 | 36.4          25.0 | 25.4                            29.5 | 29.0
//   1252                                                                    65.5 | 46.3
//   1878                                                                    76.1 | 65.1   (700 items 64.2 | 57.6; 512-256 head 77.4 | 77.3)
//   2504                                                                    77.4 | 78.8
bool score_tile_serves(const Model &m, const Batch &b, const MfmaPlan &plan)
{
    if (!plan.tile || !plan.attn || !plan.mlp || (plan.attn_variant != 0 && plan.attn_variant != 1)) return false;
    if (plan.mlp_variant < 0 || plan.mlp_variant > 2 || m.cross_in_mlp != 2 || !m.x_tiled) return false;
    if (b.n_streamed > 0 && m.n_heads > 1) return false;
    return b.n_tiles <= (b.n_groups == 0 ? 6 : 2) * n_cu();     // no group: no resident request
}

template <int DH, int K1, int H1, int H2, int NW>
static hipError_t score_tile_go(const Model &m, const Batch &b, void *X, const MfmaPlan &plan, const MlpPack &pk, const float *bias1,
                                const void *table, int32_t *bad, hipStream_t s)
{
    using H = TileHead<K1, H1, H2, 0, NW>;
    if (m.d_item + m.d_attn != K1) return hipErrorInvalidValue;
    auto kern = k_score_tile<DH, K1, H1, H2, NW>;
    constexpr int MOST = K1 / DH > KEY_PARTS ? K1 / DH : KEY_PARTS;            // runs: a head each, or KEY_PARTS
    static bool attr_set = false;
    if (!attr_set) {
        hipError_t e = hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, score_tile_lds<DH, H>(MOST));
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    const int runs = b.n_streamed > 0 ? KEY_PARTS : m.n_heads;
    hipLaunchKernelGGL(kern, dim3(b.n_blk * (ROW_BLOCK / 32)), dim3(NW * 64), (score_tile_lds<DH, H>(runs)), s, m, b, (char *)X, x_layout(m),
                       (const char *)plan.kvpack, plan.pack_stride, (const float *)plan.kmax, plan.nktp, (const char *)table, bad, pk, bias1);
    return hipGetLastError();
}

template <int DH>
static hipError_t score_tile_dh(const Model &m, const Batch &b, void *X, const MfmaPlan &plan, const MlpPack &pk, const float *bias1,
                                const void *table, int32_t *bad, hipStream_t s)
{
    switch (plan.mlp_variant) {
    case 0:
        return b.n_tiles <= n_cu() ? score_tile_go<DH, 128, 256, 128, KEY_PARTS>(m, b, X, plan, pk, bias1, table, bad, s)
                                   : score_tile_go<DH, 128, 256, 128, KEY_PARTS / 2>(m, b, X, plan, pk, bias1, table, bad, s);
    case 1:
        return b.n_tiles <= n_cu() ? score_tile_go<DH, 128, 512, 256, KEY_PARTS>(m, b, X, plan, pk, bias1, table, bad, s)
                                   : score_tile_go<DH, 128, 512, 256, KEY_PARTS / 2>(m, b, X, plan, pk, bias1, table, bad, s);
    case 2:
        return b.n_tiles <= n_cu() ? score_tile_go<DH, 256, 256, 0, KEY_PARTS>(m, b, X, plan, pk, bias1, table, bad, s)
                                   : score_tile_go<DH, 256, 256, 0, KEY_PARTS / 2>(m, b, X, plan, pk, bias1, table, bad, s);
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_score_tile(const Model &m, const Batch &b, void *X, const MfmaPlan &plan, const MlpPack &pk, const float *bias1,
                             const void *table, int32_t *bad, hipStream_t s)
{
    if (b.n_blk == 0) return hipSuccess;
    if (!pk.w0_user) return hipErrorInvalidValue;
    return plan.attn_variant == 0 ? score_tile_dh<64>(m, b, X, plan, pk, bias1, table, bad, s)
                                  : score_tile_dh<32>(m, b, X, plan, pk, bias1, table, bad, s);
}

}  // namespace aif
