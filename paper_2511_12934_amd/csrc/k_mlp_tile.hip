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
#include <utility>

#include "k_mlp_chain.h"

namespace aif {

// A head's shape, and how NW waves share it out: layer l has row tiles w, w + NW, .. of wave w.
template <int K1, int H1, int H2, int H3, int NW> struct TileHead {
    static constexpr int NH = H3 ? 3 : (H2 ? 2 : 1);
    static constexpr int kin(int l) { return l == 0 ? K1 : (l == 1 ? H1 : H2); }
    static constexpr int nout(int l) { return l == 0 ? H1 : (l == 1 ? H2 : H3); }
    static constexpr int ks(int l) { return kin(l) / 16; }
    static constexpr int rows(int l) { return nout(l) / 32 / NW; }             // row tiles per wave
    static constexpr int frags(int l) { return rows(l) * ks(l); }
    static constexpr int first(int l, int ring) { return frags(l) < ring ? frags(l) : ring; }
    static constexpr int HL = nout(NH - 1);                                    // width entering the ->1 layer
    // LDS: the activations of the hidden layers that are read by another (bf16 fragments), the last one's in fp32, the ->1 weights
    static constexpr int act_at(int l) { return l == 0 ? 0 : H1 / 16 * 1024; }
    static constexpr int last_at = (NH > 1 ? H1 / 16 * 1024 : 0) + (NH > 2 ? H2 / 16 * 1024 : 0);
    static constexpr int wl_at = last_at + HL * 32 * 4;
    static constexpr int lds_bytes = wl_at + HL * 4;
    static_assert(H1 % (32 * NW) == 0 && H2 % (32 * NW) == 0 && H3 % (32 * NW) == 0, "every wave has as many row tiles");
    static_assert(lds_bytes <= 160 * 1024 && HL / 4 <= 64 * NW, "LDS; the ->1 weights in one go");
};

template <int K1, int H1, int H2, int H3, int NW>
__global__ __launch_bounds__(NW * 64, 2) void k_mlp_tile(int64_t n_items, const ReqDesc *__restrict__ reqs, const int32_t *__restrict__ blk_req,
                                                         const int32_t *__restrict__ blk_slot, const char *__restrict__ X, XLayout xl, MlpPack pk,
                                                         const float *__restrict__ bias1)
{
    using H = TileHead<K1, H1, H2, H3, NW>;
    constexpr int RING = 16;                                    // fragments a wave has in flight
    constexpr int PRE = H::NH > 1 && K1 <= 256 ? H::first(1, RING) : 0;                 // ... of layer 2, before layer 1's, where there is room
    extern __shared__ __align__(16) char lds[];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), col = lane & 31, h = lane >> 5;
    const int tile = blockIdx.x;
    const int r = blk_req[tile / (ROW_BLOCK / 32)], slot = blk_slot[tile / (ROW_BLOCK / 32)];

    // nothing here waits for the request: the tile's rows, the ->1 weights, layer 2's first fragments and biases
    bf16x8 xin[K1 / 16];
    {
        const char *xr = X + x_offset(xl, tile * 32 + col, h);
#pragma unroll
        for (int j = 0; j < K1 / 16; ++j) xin[j] = *(const bf16x8 *)(xr + (size_t)(2 * j) * xl.piece_stride);
    }
    const f32x4 wl = ((const f32x4 *)pk.wlast)[threadIdx.x < H::HL / 4 ? threadIdx.x : 0];
    const float blast = pk.blast[0];
    auto frag_of = [&](auto lc, auto fc, const char *w) {       // fragment F of this wave's share of layer L
        constexpr int L = decltype(lc)::value, F = decltype(fc)::value;
        return *(const bf16x8 *)(w + (size_t)((F / H::ks(L) * NW + wave) * H::ks(L) + F % H::ks(L)) * 1024 + lane * 16);
    };
    auto bias_of = [&](const float *b, int rt, f32x16 &a) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const f32x4 v = *(const f32x4 *)(b + 32 * rt + 8 * q + 4 * h);
            a[4 * q + 0] = v.x;
            a[4 * q + 1] = v.y;
            a[4 * q + 2] = v.z;
            a[4 * q + 3] = v.w;
        }
    };
    f32x16 acc[2];                                              // of the row tile under way and of the next
    bf16x8 pre[PRE ? PRE : 1];
    static_for<0, PRE>([&](auto fc) { pre[decltype(fc)::value] = frag_of(IC<1>{}, fc, pk.w[1]); });
    __builtin_amdgcn_sched_barrier(0);

    const ReqDesc *rq = reqs + r;
    const int n_cand = rq->n_cand, local = tile * 32 - rq->row_base + col;
    if (local - col >= n_cand) return;                          // the rest of the request's last ROW_BLOCK
    const bool live = h == 0 && local < n_cand;
    const int64_t id = rq->cand_ids[local < n_cand ? local : n_cand - 1];
    const char *w0 = pk.w0_user + (size_t)slot * pk.w0_stride;
    const float *b0 = bias1 + (size_t)slot * H1;
    if (threadIdx.x < H::HL / 4) *(f32x4 *)(lds + H::wl_at + threadIdx.x * 16) = wl;

    // Layer L: this wave's row tiles in turn, its fragments RING ahead (the first of them in `ring` already), `next`: what to ask
    // for behind the last one.
    auto layer = [&](auto lc, const char *w, const float *b, bf16x8 *ring) __attribute__((always_inline)) {
        constexpr int L = decltype(lc)::value, KS = H::ks(L), R = H::rows(L), NF = H::frags(L);
        constexpr int AHEAD = 4;                                // activations from LDS
        bf16x8 x[L == 0 ? 1 : AHEAD];
        const char *act = lds + (L == 0 ? 0 : H::act_at(L - 1)) + lane * 16;
        if constexpr (L > 0)
#pragma unroll
            for (int k = 0; k < AHEAD; ++k) x[k] = *(const bf16x8 *)(act + k * 1024);
        static_for<0, NF>([&](auto fc) {
            constexpr int F = decltype(fc)::value, K = F % KS, T = F / KS;
            if constexpr (K == 0 && T + 1 < R) bias_of(b, (T + 1) * NW + wave, acc[(T + 1) & 1]);
            if constexpr (L == 0) {
                acc[T & 1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ring[F % RING], xin[K], acc[T & 1], 0, 0, 0);
            } else {
                acc[T & 1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ring[F % RING], x[F % AHEAD], acc[T & 1], 0, 0, 0);
                if constexpr (F + AHEAD < NF) x[F % AHEAD] = *(const bf16x8 *)(act + (F + AHEAD) % KS * 1024);
            }
            if constexpr (F + RING < NF) ring[F % RING] = frag_of(lc, IC<F + RING>{}, w);
            if constexpr (K == KS - 1) {
                const f32x16 &a = acc[T & 1];
                const int rt = T * NW + wave;
                if constexpr (L == H::NH - 1) {
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        *(f32x4 *)(lds + H::last_at + (rt * 4 + q) * 1024 + lane * 16) =
                            f32x4{relu(a[4 * q]), relu(a[4 * q + 1]), relu(a[4 * q + 2]), relu(a[4 * q + 3])};
                } else {
#pragma unroll
                    for (int j = 0; j < 2; ++j) {               // slot s of half h <-> feature 16 j + 8 (s / 4) + 4 h + s % 4
                        bf16x8 o;
#pragma unroll
                        for (int s = 0; s < 8; ++s) o[s] = (__bf16)relu(a[8 * j + s]);
                        *(bf16x8 *)(lds + H::act_at(L) + (2 * rt + j) * 1024 + lane * 16) = o;
                    }
                }
            }
            __builtin_amdgcn_sched_barrier(0);
        });
    };
    // (the barrier is hand-issued: loads in flight stay in flight)
    auto settle = [&]() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); };

    // layer L from its first fragment on; `met`: its input is the tile's rows, no other wave's work
    auto from_first = [&](auto lc, const char *w, const float *b, bool met) __attribute__((always_inline)) {
        bf16x8 ring[RING];
        bias_of(b, wave, acc[0]);
        static_for<0, H::first(decltype(lc)::value, RING)>([&](auto fc) { ring[decltype(fc)::value] = frag_of(lc, fc, w); });
        __builtin_amdgcn_sched_barrier(0);
        if (!met) settle();
        layer(lc, w, b, ring);
    };
    from_first(IC<0>{}, w0, b0, true);
    if constexpr (PRE > 0) {
        bias_of(pk.bias[1], wave, acc[0]);
        settle();
        layer(IC<1>{}, pk.w[1], pk.bias[1], pre);
    } else if constexpr (H::NH > 1)
        from_first(IC<1>{}, pk.w[1], pk.bias[1], false);
    if constexpr (H::NH > 2) from_first(IC<2>{}, pk.w[2], pk.bias[2], false);
    settle();
    if (wave != 0) return;
    // the ->1 layer, a lane's features in the chain's order
    float zpart = 0.f;
#pragma unroll
    for (int i = 0; i < H::HL / 8; ++i) {
        const f32x4 a = *(const f32x4 *)(lds + H::last_at + i * 1024 + lane * 16);
        const f32x4 v = *(const f32x4 *)(lds + H::wl_at + (8 * i + 4 * h) * 4);
        zpart = dot4(zpart, v, a.x, a.y, a.z, a.w);
    }
    float z = zpart + __shfl_xor(zpart, 32, 64) + blast;
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
                       (const char *)X, x_layout(m), pk, bias1);
    return hipGetLastError();
}

// One workgroup a compute unit at a time, but for the smallest head: batches of at most as many tiles as there are units.  Whole
// calls over 100 history items, us, the chain (the widest head: k_mlp_acc3) | here, 1 request of 71, 1,000, 8,000 and 10,000 candidates
// (313 tiles: a second round):
//   512, 256        24.0 | 22.2    24.9 | 22.6    27.4 | 24.4    27.7 | 30.1
//   256 (of 256)    22.2 | 21.6    23.4 | 22.4    25.8 | 25.0    26.3 | 28.1
//   256, 128        18.6 | 19.4    19.6 | 19.9    23.0 | 22.2    23.1 | 23.5     (over 1,000 items 21.1 | 19.9, 22.3 | 20.7, 24.4 | 22.5, 27.4 | 26.6)
//   1024, 512, 256  82.4 | 60.2    83.7 | 61.1    91.8 | 70.2    92.6 | 89.9
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
