// The fused head for ONE tile of 32 candidates by one workgroup (k_mlp_tile.hip, k_score_tile.hip): how its waves share out the
// row tiles, and the layers themselves.
#pragma once
#include <utility>

#include "k_mlp_chain.h"

namespace aif {

// A head's shape, and how NW waves share it out: layer l has row tiles w, w + NW, .. of wave w (none, for the last waves of a
// layer of fewer than NW).
template <int K1, int H1, int H2, int H3, int NW> struct TileHead {
    static constexpr int NH = H3 ? 3 : (H2 ? 2 : 1);
    static constexpr int WAVES = NW;
    static constexpr int kin(int l) { return l == 0 ? K1 : (l == 1 ? H1 : H2); }
    static constexpr int nout(int l) { return l == 0 ? H1 : (l == 1 ? H2 : H3); }
    static constexpr int ks(int l) { return kin(l) / 16; }
    static constexpr int waves(int l) { return nout(l) / 32 < NW ? nout(l) / 32 : NW; }        // that have row tiles
    static constexpr int rows(int l) { return nout(l) / 32 / waves(l); }       // row tiles of such a wave
    static constexpr int frags(int l) { return rows(l) * ks(l); }
    static constexpr int RING = 16;                                            // fragments a wave has in flight
    static constexpr int first(int l) { return frags(l) < RING ? frags(l) : RING; }
    static constexpr int PRE = NH > 1 && K1 <= 256 ? first(1) : 0;             // of layer 2, asked for beside layer 1's: where there is room
    static constexpr int HL = nout(NH - 1);                                    // width entering the ->1 layer
    // LDS: the activations of the hidden layers that are read by another (bf16 fragments), the last one's in fp32, the ->1 weights
    static constexpr int act_at(int l) { return l == 0 ? 0 : H1 / 16 * 1024; }
    static constexpr int last_at = (NH > 1 ? H1 / 16 * 1024 : 0) + (NH > 2 ? H2 / 16 * 1024 : 0);
    static constexpr int wl_at = last_at + HL * 32 * 4;
    static constexpr int lds_bytes = wl_at + HL * 4;
    static constexpr bool whole(int l) { return l >= NH || nout(l) / 32 % waves(l) == 0; }
    static_assert(whole(0) && whole(1) && whole(2), "every wave that has row tiles has as many");
    static_assert(lds_bytes <= 160 * 1024 && HL / 4 <= 64 * NW, "LDS; the ->1 weights in one go");
};

// (the barrier is hand-issued: loads in flight stay in flight)
__device__ __forceinline__ void tile_settle() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// What a wave holds of the head: ask_later() and ask() issue the first loads of layer 2 and of layer 1, run() does the layers.
template <class H> struct TileMlp {
    static constexpr int RING = H::RING, PRE = H::PRE;
    const int lane, wave, h;
    char *lds;
    bf16x8 pre[PRE ? PRE : 1], ring[RING];
    f32x16 acc[2];                                              // of the row tile under way and of the next

    __device__ __forceinline__ TileMlp(char *lds_, int lane_, int wave_) : lane(lane_), wave(wave_), h(lane_ >> 5), lds(lds_) {}

    template <int L, int F> __device__ __forceinline__ bf16x8 frag(const char *w) const       // fragment F of this wave's share of layer L
    {
        return *(const bf16x8 *)(w + (size_t)((F / H::ks(L) * H::waves(L) + wave) * H::ks(L) + F % H::ks(L)) * 1024 + lane * 16);
    }
    __device__ __forceinline__ void bias_of(const float *b, int rt, f32x16 &a) const
    {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const f32x4 v = *(const f32x4 *)(b + 32 * rt + 8 * q + 4 * h);
            a[4 * q + 0] = v.x;
            a[4 * q + 1] = v.y;
            a[4 * q + 2] = v.z;
            a[4 * q + 3] = v.w;
        }
    }
    template <int L> __device__ __forceinline__ bool mine() const { return H::waves(L) == H::WAVES || wave < H::waves(L); }

    __device__ __forceinline__ void ask_later(const MlpPack &pk)
    {
        if constexpr (PRE > 0)
            if (mine<1>()) static_for<0, PRE>([&](auto fc) { pre[decltype(fc)::value] = frag<1, decltype(fc)::value>(pk.w[1]); });
        __builtin_amdgcn_sched_barrier(0);
    }
    template <int L> __device__ __forceinline__ void ask(const char *w, const float *b)
    {
        if (!mine<L>()) return;
        bias_of(b, wave, acc[0]);
        static_for<0, H::first(L)>([&](auto fc) { ring[decltype(fc)::value] = frag<L, decltype(fc)::value>(w); });
        __builtin_amdgcn_sched_barrier(0);
    }
    // Layer L: this wave's row tiles in turn, its first fragments in `r` already, the others RING ahead.
    template <int L, class X> __device__ __forceinline__ void layer(const char *w, const float *b, bf16x8 *r, const X &xin)
    {
        if (!mine<L>()) return;
        constexpr int KS = H::ks(L), R = H::rows(L), NF = H::frags(L);
        constexpr int AHEAD = 4;                                // activations from LDS
        bf16x8 x[L == 0 ? 1 : AHEAD];
        const char *act = lds + (L == 0 ? 0 : H::act_at(L - 1)) + lane * 16;
        if constexpr (L > 0)
#pragma unroll
            for (int k = 0; k < AHEAD; ++k) x[k] = *(const bf16x8 *)(act + k * 1024);
        static_for<0, NF>([&](auto fc) {
            constexpr int F = decltype(fc)::value, K = F % KS, T = F / KS;
            if constexpr (K == 0 && T + 1 < R) bias_of(b, (T + 1) * H::waves(L) + wave, acc[(T + 1) & 1]);
            if constexpr (L == 0) {
                acc[T & 1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(r[F % RING], xin[K], acc[T & 1], 0, 0, 0);
            } else {
                acc[T & 1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(r[F % RING], x[F % AHEAD], acc[T & 1], 0, 0, 0);
                if constexpr (F + AHEAD < NF) x[F % AHEAD] = *(const bf16x8 *)(act + (F + AHEAD) % KS * 1024);
            }
            if constexpr (F + RING < NF) r[F % RING] = frag<L, F + RING>(w);
            if constexpr (K == KS - 1) {
                const f32x16 &a = acc[T & 1];
                const int rt = T * H::waves(L) + wave;
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
    }
    // Everything from layer 1 (asked for) to the last hidden layer's activations; xin: the tile's rows as layer 1's column fragments.
    template <class X> __device__ __forceinline__ void run(const MlpPack &pk, const char *w0, const float *b0, const X &xin)
    {
        layer<0>(w0, b0, ring, xin);
        if constexpr (PRE > 0) {
            if (mine<1>()) bias_of(pk.bias[1], wave, acc[0]);
            tile_settle();
            layer<1>(pk.w[1], pk.bias[1], pre, xin);
        } else if constexpr (H::NH > 1) {
            ask<1>(pk.w[1], pk.bias[1]);
            tile_settle();
            layer<1>(pk.w[1], pk.bias[1], ring, xin);
        }
        if constexpr (H::NH > 2) {
            ask<2>(pk.w[2], pk.bias[2]);
            tile_settle();
            layer<2>(pk.w[2], pk.bias[2], ring, xin);
        }
        tile_settle();
    }
    // the ->1 layer by one wave: a lane's features in the chain's order (both halves of the wave have the logit)
    __device__ __forceinline__ float logit(float blast) const
    {
        float zpart = 0.f;
#pragma unroll
        for (int i = 0; i < H::HL / 8; ++i) {
            const f32x4 a = *(const f32x4 *)(lds + H::last_at + i * 1024 + lane * 16);
            const f32x4 v = *(const f32x4 *)(lds + H::wl_at + (8 * i + 4 * h) * 4);
            zpart = dot4(zpart, v, a.x, a.y, a.z, a.w);
        }
        return zpart + __shfl_xor(zpart, 32, 64) + blast;
    }
};

}  // namespace aif
