// a6-a7 for few candidates: the fused head (k_mlp_mfma.hip), a workgroup to ONE tile of 32 candidates.
//
// The chain gives a wave 32 candidates and lets it walk every row tile of every layer: a straight line of 80 to 2,176
// products, each of them 32 cycles behind the one before, whatever the batch.  With fewer tiles than compute units that line
// is the launch.  Here the waves of a workgroup share the row tiles of a layer out, and its activations pass to the next
// layer through LDS, in the order the matrix instruction reads them (a lane's sixteen results are, in place, its share of
// two k-steps: two 16-byte stores).  Nobody shares a weight, so fragments come straight from the L2s into registers, a ring
// of them per wave; those of layer 2 that fit are asked for before the tile's request, slot and layer-1 weights are known.
// The same products, sums in the same order and the same roundings as the chain's: the same bits.
//
// What bounds it: the weights through one compute unit's L1 (256 -> 512 -> 256: 393 KB a workgroup, 2.6 us at 64 bytes a
// cycle) behind three round trips (tile -> request and slot -> weights).
#include "k_mlp_tile.h"

namespace aif {

template <int K1, int H1, int H2, int H3, int NW>
__global__ __launch_bounds__(NW * 64, 2) void k_mlp_tile(int64_t n_items, const ReqDesc *__restrict__ reqs, const int32_t *__restrict__ blk_req,
                                                         const int32_t *__restrict__ blk_slot, const char *__restrict__ X, XLayout xl, MlpPack pk,
                                                         const float *__restrict__ bias1, int n_blk)
{
    using H = TileHead<K1, H1, H2, H3, NW>;
    extern __shared__ __align__(16) char lds[];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), col = lane & 31, h = lane >> 5;
    // the first tile of every ROW_BLOCK, then the second ..: tiles past a request's end come late, behind those with work
    const int blk = (int)blockIdx.x % n_blk, tile = blk * (ROW_BLOCK / 32) + (int)blockIdx.x / n_blk;
    const int r = blk_req[blk], slot = blk_slot[blk];

    // nothing here waits for the request: the tile's rows, the ->1 weights, layer 2's first fragments
    bf16x8 xin[K1 / 16];
    {
        const char *xr = X + x_offset(xl, tile * 32 + col, h);
#pragma unroll
        for (int j = 0; j < K1 / 16; ++j) xin[j] = *(const bf16x8 *)(xr + (size_t)(2 * j) * xl.piece_stride);
    }
    const f32x4 wl = ((const f32x4 *)pk.wlast)[threadIdx.x < H::HL / 4 ? threadIdx.x : 0];
    const float blast = pk.blast[0];
    TileMlp<H> mlp(lds, lane, wave);
    mlp.ask_later(pk);

    const ReqDesc *rq = reqs + r;
    const int n_cand = rq->n_cand, local = tile * 32 - rq->row_base + col;
    if (local - col >= n_cand) return;                          // the rest of the request's last ROW_BLOCK
    const bool live = h == 0 && local < n_cand;
    const int64_t id = rq->cand_ids[local < n_cand ? local : n_cand - 1];
    const char *w0 = pk.w0_user + (size_t)slot * pk.w0_stride;
    const float *b0 = bias1 + (size_t)slot * H1;
    if (threadIdx.x < H::HL / 4) *(f32x4 *)(lds + H::wl_at + threadIdx.x * 16) = wl;
    mlp.template ask<0>(w0, b0);
    mlp.run(pk, w0, b0, xin);
    if (wave != 0) return;
    float z = mlp.logit(blast);
    if (live) {
        if (id < 0 || id >= n_items) z = __uint_as_float(0x7FC00000u);
        rq->logits_out[local] = z;
        if (rq->scores_out) rq->scores_out[local] = 1.0f / (1.0f + __expf(-z));
    }
}

template <int K1, int H1, int H2, int H3, int NW>
static hipError_t tile_go(const Model &m, const Batch &b, const void *X, const MlpPack &pk, const float *bias1, hipStream_t s)
{
    using H = TileHead<K1, H1, H2, H3, NW>;
    auto kern = k_mlp_tile<K1, H1, H2, H3, NW>;
    static bool attr_set = false;
    if (!attr_set) {
        hipError_t e = hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, H::lds_bytes);
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    hipLaunchKernelGGL(kern, dim3(b.n_blk * (ROW_BLOCK / 32)), dim3(NW * 64), H::lds_bytes, s, m.n_items, b.reqs, b.blk_req, b.blk_slot,
                       (const char *)X, x_layout(m), pk, bias1, b.n_blk);
    return hipGetLastError();
}

// One workgroup a compute unit at a time, but for the smallest head: batches of at most as many tiles as there are units.  What comes here
// is the widest head, and of the others what k_score_tile.hip does not take: several heads with a history that is streamed (and
// calls that time a stage).  Whole calls, us, the chain (the widest head: k_mlp_acc3) | here, 1 request of 71, 1,000, 4,000 and 8,000 candidates:
//   512, 256        (2 heads, 1,000 items)  26.6 | 22.6    28.0 | 23.5    29.0 | 24.8    30.3 | 26.6
//   256 (of 256)    (4 heads, 500 items)    25.5 | 24.1    27.8 | 26.2    29.2 | 27.6    30.9 | 29.5
//   256, 128        (2 heads, 600 items)    22.0 | 20.2    22.7 | 21.0    23.6 | 22.1    24.9 | 23.9     (2,000 items 24.1 | 22.8 to 28.3 | 26.6)
//   1024, 512, 256  (100 items)             82.4 | 60.2    83.7 | 61.1                   91.8 | 70.2     (10,000, a second round: 92.6 | 89.9)
bool mlp_tile_serves(int variant, const Model &m, const Batch &b)
{
    return m.cross_in_mlp == 2 && m.x_tiled && variant >= 0 && variant <= 3 && b.n_tiles <= n_cu();
}

hipError_t launch_mlp_tile(int variant, const Model &m, const Batch &b, const void *X, const MlpPack &pk, const float *bias1, hipStream_t s)
{
    if (!pk.w0_user) return hipErrorInvalidValue;
    switch (variant) {
    case 0: return tile_go<128, 256, 128, 0, 4>(m, b, X, pk, bias1, s);
    case 1: return tile_go<128, 512, 256, 0, 8>(m, b, X, pk, bias1, s);
    case 2: return tile_go<256, 256, 0, 0, 8>(m, b, X, pk, bias1, s);
    case 3: return tile_go<384, 1024, 512, 256, 8>(m, b, X, pk, bias1, s);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace aif
