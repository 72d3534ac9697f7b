// a6-a7 on the matrix cores: the widest head, 384 -> 1024 -> 512 -> 256 -> 1 (layer 1 over [item | attention]), in the order of
// work of k_mlp_acc.hip: a row tile of layer 1 is contracted into all 16 row tiles of layer 2 (the 256 accumulation registers)
// as soon as it is through its ReLU.  Same products and orders of addition as the chain of k_mlp_chain.h, the same bits.
//
// A wave owns 32 candidates, a block 128; one wave per SIMD.  Blocks are persistent over contiguous runs of tiles.  Stage
// t = 1 .. 31 of a tile: layer 1's row tile t alternating with layer 2's two k-steps of row tile t - 1 (layer 1's products
// form a chain on one accumulator, so none follows another directly).  The tail: layer 2's last two k-steps, layer 3 (its
// accumulators take the registers of layer 2's first eight row tiles once those are operands), then row tile 0 of the next
// tile with the ->1 layer behind its products.  The weights of all that are one stream of pieces of eight 1 KB fragments
// through a ring of 12 in LDS; in a piece every wave moves two fragments.
//
// What bounds it: waits, and power.  32 x 10^4 candidates, this and the chain in turn on one box: 541 us (1.24 PFLOP/s) against 589
// (497 and 573 on another), in 926 k cycles against 1178 k.  Matrix cores busy 0.71 of the cycles (the chain 0.56), in s_waitcnt or at
// a barrier 0.23, neither matrix cores nor vector ALU 0.14; a fifth fewer cycles are 8 % less time, because the clock is 1.71 against
// 2.00 GHz.  The chain's products all follow one another on one accumulator and its stages' loads went out in a row;
// spreading the loads alone gave 1 %.
#include "k_mlp_chain.h"
#include "k_mlp_acc.h"

namespace aif {

struct Acc3 {
    static constexpr int WAVES = 4, ROWS = 128, SLOTS = 12, KS1 = 24, NT1 = 32, NT2 = 16, NT3 = 8, KS2 = 2 * NT1, KS3 = 2 * NT2;
    static constexpr int H1 = 32 * NT1, H2 = 32 * NT2, H3 = 32 * NT3;
    static constexpr int SF = KS1 + 2 * NT2, SP = SF / 8;                       // fragments, pieces of a stage
    static constexpr int Q3 = 2 * NT2 / 8, Q0 = Q3 + KS3, QT = Q0 + KS1 / 8;    // pieces of the tail: layer 3 from Q3, row tile 0 from Q0
    static constexpr int slot_bytes = 8 * 1024, ring_bytes = SLOTS * slot_bytes, AHEAD = SLOTS - 1;
    // input rows pass through LDS in quarters of XQ k-steps, two at a time
    static constexpr int XQ = KS1 / 4, x_wave = 2 * XQ * 1024;
    static constexpr int o_x = ring_bytes, o_b1 = o_x + WAVES * x_wave, o_b2 = o_b1 + 2 * H1 * 4, o_b3 = o_b2 + H2 * 4,
                         o_wl = o_b3 + H3 * 4, o_id = o_wl + H3 * 4, lds_bytes = o_id + 2 * WAVES * 256;
    // Loads a wave sends besides the weights in piece q of the tail: quarters 0, 1 of the next tile's input rows, its layer-1
    // biases and ids, quarters 2, 3 once the first two are in registers (read in piece QX).
    static constexpr int QX = 18, QR = XQ + 1;
    static constexpr int extra(int q) { return (q >= 0 && q < XQ) || (q > QX && q <= QX + XQ) || q == QR ? 2 : 0; }
    // how many of its loads may be in flight in piece q for the next piece to have landed
    static constexpr int left(int q)
    {
        int n = 0;
        for (int k = 1; k < AHEAD - 1; ++k) n += 2 + extra(q - k);
        return n;
    }
    static_assert(lds_bytes <= 160 * 1024 && SF % 8 == 0 && KS1 % 8 == 0, "LDS; whole pieces");
    static_assert(XQ + AHEAD <= QX && QX + XQ + AHEAD <= Q0 && QR + AHEAD < Q0 - 2, "what is sent for has landed when it is read");
};

__global__ __launch_bounds__(256, 1) void k_mlp_acc3(int64_t n_items, const ReqDesc *__restrict__ reqs,
                                                     const int32_t *__restrict__ blk_req, const int32_t *__restrict__ blk_slot,
                                                     const char *__restrict__ X, uint32_t xtile_bytes, MlpPack pk,
                                                     const float *__restrict__ bias1, int n_tiles)
{
    using C = Acc3;
    constexpr int KS1 = C::KS1, NT1 = C::NT1, NT2 = C::NT2, NT3 = C::NT3, H1 = C::H1, H2 = C::H2, H3 = C::H3, RING = 8, KB = 1024;
    extern __shared__ __align__(16) char lds[];
    const int lane = threadIdx.x & 63, h = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t L0 = lds_address(lds), lane16 = lane * 16;

    // contiguous runs of tiles; the 8 XCDs, which take the workgroups in turn, each a contiguous run of blocks (k_mlp_acc.hip)
    const int nb = (int)gridDim.x, b = (int)blockIdx.x;
    const int idx = nb % 8 ? b : (b & 7) * (nb >> 3) + (b >> 3);
    const int first = (int)((int64_t)idx * n_tiles / nb), n_mine = (int)((int64_t)(idx + 1) * n_tiles / nb) - first;
    constexpr int TPB = ROW_BLOCK / C::ROWS;
    auto out_of = [&](int r) {
        const ReqDesc *q = reqs + r;
        return AccOut{q->cand_ids, q->logits_out, q->scores_out, q->n_cand, q->row_base};
    };

    // ---- copies into LDS, untracked.  Position i of a stage: layer 1's k-step (i - 1) / 2 where i < 2 KS1 is odd, else layer 2's
    // j-th fragment (row tile j % 16, k-step j / 16 of the two), j = i / 2 or i - KS1.  Wave w moves positions w and w + 4 of
    // every piece: odd waves layer 1's fragments, even ones layer 2's, all of them layer 2's in the last piece.
    const bool odd = wave & 1;
    const char *const w1 = pk.w[1], *const w2 = pk.w[2] + (size_t)wave * C::KS3 * KB;
    const size_t inc = odd ? KS1 * KB : 2 * KB;                 // from one stage to the next
    uint32_t vo[6][2], v256 = lane16 + 256 * KB, v128 = lane16 + 128 * KB, v4 = lane16 + 4 * KB;
#pragma unroll
    for (int p = 0; p < 6; ++p)
#pragma unroll
        for (int m = 0; m < 2; ++m)
            vo[p][m] = lane16 + (odd ? p * 4 * KB + m * 2 * KB : (4 * p + 2 * m) % NT2 * C::KS2 * KB + (p >= 4 ? KB : 0));
    const uint64_t even_base = (uint64_t)w1 + (wave >> 1) * C::KS2 * KB;
    auto stage_base = [=](const char *w0, int t) {
        const uint64_t o = (uint64_t)w0 + ((wave >> 1) + t * KS1) * KB, e = even_base + 2 * (t - 1) * KB;
        return (const char *)(odd ? o : e);
    };
    auto last_base = [&](int t) { return w1 + ((8 + wave) * C::KS2 + 2 * (t - 1) + 1) * KB; };
    const uint32_t wdst = L0 + wave * KB;
    // load M of piece p of a stage / of piece q of the tail, into the slot at `dst`
    auto send_stage = [&](auto pc, auto mc, const char *base, const char *last, uint32_t dst) {
        constexpr int P = decltype(pc)::value, M = decltype(mc)::value;
        if constexpr (P < 6)
            dma_s<16>(base, vo[P][M], dst, M * 4 * KB);
        else
            dma_s<16>(last, M ? v256 : lane16, dst, M * 4 * KB);
    };
    auto send_tail = [&](auto qc, auto mc, const char *w0, uint32_t dst) {
        constexpr int Q = decltype(qc)::value, M = decltype(mc)::value;
        if constexpr (Q < C::Q3)                                // position i: row tile i / 2, k-step i % 2
            dma_s<16>(w1 + ((wave >> 1) * C::KS2 + 2 * (NT1 - 1) + (wave & 1)) * KB + Q * 4 * C::KS2 * KB, M ? v128 : lane16, dst, M * 4 * KB);
        else if constexpr (Q < C::Q0)                           // a piece = a k-step of layer 3, position = row tile
            dma_s<16>(w2 + (Q - C::Q3) * KB, M ? v128 : lane16, dst, M * 4 * KB);
        else
            dma_s<16>(w0 + wave * KB + (Q - C::Q0) * 8 * KB, M ? v4 : lane16, dst, M * 4 * KB);
    };
    const uint32_t xdst = L0 + C::o_x + wave * C::x_wave;
    auto x_of = [&](int tile) { return X + (size_t)(tile * (C::ROWS / X_TILE) + wave) * xtile_bytes; };
    auto send_x = [&](auto kc, const char *src) { dma_s<16>(src + decltype(kc)::value * KB, lane16, xdst, decltype(kc)::value % (2 * C::XQ) * KB); };
    auto send_bias = [&](int slot, int par) { dma_s<16>((const char *)(bias1 + (size_t)slot * H1) + wave * KB, lane16, wdst + C::o_b1 + par * H1 * 4, 0); };
    auto send_ids = [&](int tile, const AccOut &rd, int par) {
        int local = tile * C::ROWS - rd.row_base + wave * 32 + (lane & 31);     // a lane with no candidate reads the first id
        if (local >= rd.n_cand) local = 0;
        dma_s<4>(rd.cand_ids, 4 * local, L0 + C::o_id + (par * C::WAVES + wave) * 256, 0);
    };

    auto lds8 = [&](uint32_t a) -> bf16x8 { return *(const bf16x8 __attribute__((address_space(3))) *)(uintptr_t)a; };
    auto lds4 = [&](uint32_t a) -> f32x4 { return *(lds_f32x4_t)(uintptr_t)a; };
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    f32x16 acc1;                            // layer 1's accumulator; layer 2's: a0 .. a255, layer 3's: a0 .. a127
    bf16x8 x[KS1], areg[RING];
    u32x4 hb[2] = {}, hn = {};              // row tile of layer 1 as operands; the next one's second half until the stage ends
    float z = 0.f;
    f32x4 wlv[2][4];
    reserve_acc();
    const uint32_t h16 = L0 + 16 * h, rb_x = xdst + lane16;

    // ---- the first tile: input rows, biases, ids, the pieces from its row tile 0 on
    int tile = first;
    auto at = [&](int t) { return t < n_tiles ? t : n_tiles - 1; };
    const int r0 = blk_req[tile / TPB], sl0 = blk_slot[tile / TPB];
    int cslot = sl0, nr = blk_req[at(tile + 1) / TPB], nslot = blk_slot[at(tile + 1) / TPB];
    AccOut cur = out_of(r0), nxt = cur, prev = cur;
    prev.n_cand = INT32_MIN;                                    // no tile before the first
    const char *w0c = pk.w0_user + (size_t)sl0 * pk.w0_stride, *w0n = w0c;
    {
        const char *src = x_of(tile);
        static_for<0, 2 * C::XQ>([&](auto kc) { send_x(kc, src); });
        static_for<0, C::AHEAD>([&](auto ic) {
            constexpr int I = decltype(ic)::value, A = KS1 / 8;
            static_for<0, 2>([&](auto mc) {
                if constexpr (I < A)
                    send_tail(IC<C::Q0 + I>{}, mc, w0c, wdst + I * C::slot_bytes);
                else
                    send_stage(IC<(I - A) % C::SP>{}, mc, stage_base(w0c, 1 + (I - A) / C::SP), last_base(1 + (I - A) / C::SP), wdst + I * C::slot_bytes);
            });
        });
        send_bias(sl0, 0);
        send_ids(tile, cur, 0);
        float *sb2 = (float *)(lds + C::o_b2), *sb3 = (float *)(lds + C::o_b3), *swl = (float *)(lds + C::o_wl);
        for (int i = threadIdx.x; i < H2; i += 256) sb2[i] = pk.bias[1][i];
        for (int i = threadIdx.x; i < H3; i += 256) {
            sb3[i] = pk.bias[2][i];
            swl[i] = pk.wlast[i];
        }
        wait_vmcnt<0>();
        __syncthreads();
        static_for<0, 2 * C::XQ>([&](auto kc) { x[decltype(kc)::value] = lds8(rb_x + decltype(kc)::value * KB); });
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        static_for<2 * C::XQ, KS1>([&](auto kc) { send_x(kc, src); });
        wait_vmcnt<0>();
        static_for<2 * C::XQ, KS1>([&](auto kc) { x[decltype(kc)::value] = lds8(rb_x + (decltype(kc)::value - 2 * C::XQ) * KB); });
    }
    static_for<32, 64>([&](auto wc) {                           // layer 2's biases in row tiles 8 .. 15 (0 .. 7: behind row tile 0)
        constexpr int W = decltype(wc)::value;
        acc_from_lds<4 * W, W / 4 * 128 + W % 4 * 32>(h16 + C::o_b2);
    });
    const float bl = pk.blast[0];
    uint32_t b1c = h16 + C::o_b1, b1n = b1c + H1 * 4;           // this and the next tile's layer-1 biases
    auto preload_q = [&](uint32_t addr, int q) {                // four of acc1's biases: features 8 q + 4 h + i
        const f32x4 v = lds4(addr + 32 * q);
        acc1[4 * q + 0] = v.x;
        acc1[4 * q + 1] = v.y;
        acc1[4 * q + 2] = v.z;
        acc1[4 * q + 3] = v.w;
    };
#pragma unroll
    for (int q = 0; q < 4; ++q) preload_q(b1c, q);
    // the ring: offset of the current piece, this lane's place in it and in the next
    uint32_t ring = 0;
    auto past = [&](uint32_t r, int pieces) {
        const uint32_t p = r + pieces * C::slot_bytes;
        return p < (uint32_t)C::ring_bytes ? p : p - C::ring_bytes;
    };
    uint32_t rb = L0 + lane16, rbn = rb + C::slot_bytes;
    static_for<0, RING - 1>([&](auto fc) { areg[decltype(fc)::value] = lds8(rb + decltype(fc)::value * KB); });

#define AIF_FENCE __builtin_amdgcn_sched_barrier(0)
    // Position S of a piece: the fragment RING - 1 positions on, one product, the work behind it.  Before position 1, the first
    // that looks into the next piece: this wave's share of it has landed (N younger loads may be in flight), behind the barrier
    // everyone's has, and nobody reads the piece before any more.
    auto position = [&](auto sc, auto nc, auto &&product, auto &&gap) {
        constexpr int S = decltype(sc)::value;
        if constexpr (S == 1) {
            wait_vmcnt<decltype(nc)::value>();
            asm volatile("s_barrier" ::: "memory");
        }
        areg[(S + RING - 1) % RING] = S == 0 ? lds8(rb + (RING - 1) * KB) : lds8(rbn + (S - 1) * KB);
        product(areg[S]);
        AIF_FENCE;
        gap();
        if constexpr (S == 7) {
            ring = past(ring, 1);
            rb = rbn;
            rbn = L0 + lane16 + past(ring, 1);
        }
        AIF_FENCE;
    };
    // pair S = 0 .. 7 of acc1's features into operands
    auto convert = [&](auto sc, u32x4 &second) {
        constexpr int S = decltype(sc)::value;
        const uint32_t v = relu_pair(acc1[2 * S], acc1[2 * S + 1]);
        if constexpr (S < 4)
            hb[0][S] = v;
        else
            second[S - 4] = v;
    };
    // Stage t; send(p, m, dst): load M of the piece AHEAD of piece P
    auto stage = [&](uint32_t bnext, auto &&send, auto &&extra) {
        static_for<0, C::SP>([&](auto pc) {
            constexpr int P = decltype(pc)::value;
            const uint32_t dst = wdst + past(ring, C::AHEAD);
            static_for<0, 8>([&](auto sc) {
                constexpr int I = 8 * P + decltype(sc)::value;
                position(sc, IC<2 * (C::AHEAD - 2)>{},
                         [&](const bf16x8 &a) {
                             if constexpr (I < 2 * KS1 && I % 2)
                                 mfma_v(acc1, a, x[I / 2]);
                             else {
                                 constexpr int J = I < 2 * KS1 ? I / 2 : I - KS1;
                                 mfma_a<16 * (J % NT2)>(a, __builtin_bit_cast(bf16x8, hb[J / NT2]));
                             }
                         },
                         [&]() {
                             if constexpr (I % 8 == 1) send(pc, IC<0>{}, dst);
                             if constexpr (I % 8 == 2) send(pc, IC<1>{}, dst);
                             // row tile t is complete behind position 47: operands (layer 2 has only the second k-step's
                             // still to read), then the next row tile's biases
                             constexpr int G = I - 2 * KS1 - 1;
                             if constexpr (G >= 0 && G < 3) static_for<3 * G, (3 * G + 3 < 8 ? 3 * G + 3 : 8)>([&](auto vc) { convert(vc, hn); });
                             if constexpr (G >= 3 && G < 5) {
                                 preload_q(bnext, 2 * (G - 3));
                                 preload_q(bnext, 2 * (G - 3) + 1);
                             }
                             if constexpr (I == C::SF - 1) hb[1] = hn;
                             extra(IC<I>{});
                         });
            });
        });
    };
    // the ->1 layer: unit V = 0 .. 31, features 8 (V % 4) .. of row tile V / 4
    auto dot_unit = [&](auto vc) {
        constexpr int V = decltype(vc)::value, A = 4 * V;
        z = dot4(z, wlv[V / 4 & 1][V % 4], acc_relu<A>(), acc_relu<A + 1>(), acc_relu<A + 2>(), acc_relu<A + 3>());
        asm volatile("" : "+v"(z));
    };
    auto read_wl = [&](auto rc) {
        constexpr int T = decltype(rc)::value;
#pragma unroll
        for (int q = 0; q < 4; ++q) wlv[T & 1][q] = lds4(h16 + C::o_wl + T * 128 + 32 * q);
    };
    auto finish = [&](int t, int par, const AccOut &rd, float zp) {      // logits and scores of a tile
        const float zz0 = zp + __shfl_xor(zp, 32, 64) + bl;
        const int32_t id = *(const int32_t __attribute__((address_space(3))) *)(uintptr_t)(L0 + C::o_id + (par * C::WAVES + wave) * 256 + lane * 4);
        const int local = t * C::ROWS - rd.row_base + wave * 32 + (lane & 31);
        if (h == 0 && local < rd.n_cand) {
            const float zz = id < 0 || id >= n_items ? __uint_as_float(0x7FC00000u) : zz0;
            typedef float __attribute__((address_space(1))) *gfloat_t;
            ((gfloat_t)rd.logits_out)[local] = zz;
            if (rd.scores_out) ((gfloat_t)rd.scores_out)[local] = 1.0f / (1.0f + __expf(-zz));
        }
    };

    // load M of the piece AHEAD of piece Q of the tail; w0: layer 1's weights of the tile that begins
    auto tail_send = [&](auto qc, auto mc, uint32_t dst, const char *w0) {
        constexpr int Q = decltype(qc)::value + C::AHEAD, R = Q - C::QT;
        if constexpr (R < 0)
            send_tail(IC<Q>{}, mc, w0, dst);
        else
            send_stage(IC<R % C::SP>{}, mc, stage_base(w0, 1 + R / C::SP), last_base(1 + R / C::SP), dst);
    };

    for (int n = 0;; ++n) {
        // the request of the tile after this one, and the index of the one after that
        nxt = out_of(nr);
        w0n = pk.w0_user + (size_t)nslot * pk.w0_stride;
        const int nr2 = blk_req[at(tile + 2) / TPB], ns2 = blk_slot[at(tile + 2) / TPB];
        // row tile 0; behind its products the ->1 layer of the tile before and layer 2's biases in row tiles 0 .. 7
        z = 0.f;
        static_for<C::Q0, C::QT>([&](auto qc) {
            constexpr int Q = decltype(qc)::value;
            const uint32_t dst = wdst + past(ring, C::AHEAD);
            static_for<0, 8>([&](auto sc) {
                constexpr int S = decltype(sc)::value, K = 8 * (Q - C::Q0) + S;
                position(sc, IC<C::left(Q)>{}, [&](const bf16x8 &a) { mfma_v(acc1, a, x[K]); },
                         [&]() {
                             if constexpr (S == 1) tail_send(qc, IC<0>{}, dst, w0c);
                             if constexpr (S == 2) tail_send(qc, IC<1>{}, dst, w0c);
                             if constexpr (K % 3 == 0 && K / 3 + 1 < NT3) read_wl(IC<K / 3 + 1>{});
                             static_for<0, (K % 3 == 2 ? 2 : 1)>([&](auto vc) {      // four units in three positions
                                 constexpr int V = K / 3 * 4 + K % 3 + decltype(vc)::value, W = V - 4;
                                 dot_unit(IC<V>{});
                                 if constexpr (W >= 0) acc_from_lds<4 * W, W / 4 * 128 + W % 4 * 32>(h16 + C::o_b2);
                             });
                         });
            });
        });
        static_for<28, 32>([&](auto wc) {
            constexpr int W = decltype(wc)::value;
            acc_from_lds<4 * W, W / 4 * 128 + W % 4 * 32>(h16 + C::o_b2);
        });
        // acc1's last product; layer 2's biases and the scalar loads above (k_mlp_acc.hip)
        asm volatile("s_nop 15" ::: "memory");
        __builtin_amdgcn_s_waitcnt(0xC07F);                     // lgkmcnt(0)
        asm volatile("" ::"s"(nxt.cand_ids), "s"(nxt.logits_out), "s"(nxt.scores_out), "s"(nxt.n_cand), "s"(nxt.row_base), "s"(nr2), "s"(ns2));
        if (n == n_mine) break;
        static_for<0, 8>([&](auto vc) { convert(vc, hb[1]); });
#pragma unroll
        for (int q = 0; q < 4; ++q) preload_q(b1c + 128, q);
        const char *pa = stage_base(w0c, 2), *la = last_base(2);        // of stage t + 1
        uint32_t bias = b1c + 128;
        for (int t = 1; t < NT1 - 2; ++t) {
            const char *const pb = pa + inc, *const lb = la + 2 * KB;
            bias += 128;
            stage(bias,
                  [&](auto pc, auto mc, uint32_t dst) {
                      constexpr int F = decltype(pc)::value + C::AHEAD - C::SP;
                      send_stage(IC<F % C::SP>{}, mc, F < C::SP ? pa : pb, F < C::SP ? la : lb, dst);
                  },
                  [](auto) {});
            pa = pb;
            la = lb;
        }
        const float zp = z;
        stage(bias + 128,
              [&](auto pc, auto mc, uint32_t dst) {
                  constexpr int F = decltype(pc)::value + C::AHEAD - C::SP;
                  if constexpr (F < C::SP)
                      send_stage(IC<F>{}, mc, pa, la, dst);
                  else
                      send_tail(IC<F - C::SP>{}, mc, w0n, dst);
              },
              [&](auto ic) {
                  if constexpr (decltype(ic)::value == 4) finish(tile - 1, (n - 1) & 1, prev, zp);
              });
        stage(bias,                                             // (acc1 is loaded again in the tail)
              [&](auto pc, auto mc, uint32_t dst) { send_tail(IC<decltype(pc)::value + C::AHEAD - C::SP>{}, mc, w0n, dst); }, [](auto) {});
        prev = cur;
        cur = nxt;
        w0c = w0n;
        cslot = nslot;
        nr = nr2;
        nslot = ns2;
        const uint32_t bt = b1c;
        b1c = b1n;
        b1n = bt;
        ++tile;
        {                                   // layers 2 and 3 of the tile that ends; tile, cur, w0c, b1c are the next one's
            const char *xsrc = x_of(at(tile));
            u32x4 h2[8][2];                 // row tiles of layer 2 as operands
            static_for<0, C::Q0>([&](auto qc) {
                constexpr int Q = decltype(qc)::value;
                const uint32_t dst = wdst + past(ring, C::AHEAD);
                static_for<0, 8>([&](auto sc) {
                    constexpr int S = decltype(sc)::value, I = 8 * Q + S, E = I - 8 * C::Q3;
                    // layer 3's biases, the last read behind position 27, have landed: only fragments were asked for since
                    if constexpr (E == 0) asm volatile("s_waitcnt lgkmcnt(4)" ::: "memory");
                    if constexpr (Q == C::QX + 1 && S == 0) asm volatile("s_waitcnt lgkmcnt(2)" ::: "memory");      // the input rows of piece QX are in registers
                    position(sc, IC<C::left(Q)>{},
                             [&](const bf16x8 &a) {
                                 if constexpr (E < 0)
                                     mfma_a<16 * (I / 2)>(a, __builtin_bit_cast(bf16x8, hb[I % 2]));
                                 else
                                     mfma_a<16 * S>(a, __builtin_bit_cast(bf16x8, h2[(Q - C::Q3) / 2 % 8][(Q - C::Q3) % 2]));
                             },
                             [&]() {
                                 if constexpr (S == 1) tail_send(qc, IC<0>{}, dst, w0c);
                                 if constexpr (S == 2) tail_send(qc, IC<1>{}, dst, w0c);
                                 if constexpr (S == 4 || S == 5) {
                                     if constexpr (Q < C::XQ) send_x(IC<2 * Q + S - 4>{}, xsrc);
                                     if constexpr (Q > C::QX && Q <= C::QX + C::XQ) send_x(IC<2 * C::XQ + 2 * (Q - C::QX - 1) + S - 4>{}, xsrc);
                                     if constexpr (Q == C::QR && S == 4) send_bias(cslot, (n + 1) & 1);
                                     if constexpr (Q == C::QR && S == 5) send_ids(at(tile), cur, (n + 1) & 1);
                                 }
                                 if constexpr (Q == C::QX && S < 6) {
                                     x[2 * S] = lds8(rb_x + 2 * S * KB);
                                     x[2 * S + 1] = lds8(rb_x + (2 * S + 1) * KB);
                                 }
                                 if constexpr (Q == C::Q0 - 1 && S < 6) {
                                     x[2 * C::XQ + 2 * S] = lds8(rb_x + 2 * S * KB);
                                     x[2 * C::XQ + 2 * S + 1] = lds8(rb_x + (2 * S + 1) * KB);
                                 }
                                 if constexpr (Q == C::Q0 - 2 && S >= 6) {
                                     preload_q(b1c, 2 * (S - 6));
                                     preload_q(b1c, 2 * (S - 6) + 1);
                                 }
                                 // layer 2's row tiles 0 .. 7 into operands (row tile T is complete behind position 2 T + 1),
                                 // each followed by layer 3's biases in its registers
                                 if constexpr (I >= 4 && I < 26)
                                     static_for<3 * (I - 4), (3 * (I - 4) + 3 < 64 ? 3 * (I - 4) + 3 : 64)>([&](auto vc) {
                                         constexpr int V = decltype(vc)::value, T = V / 8, s = V % 8;
                                         h2[T][s / 4][s % 4] = acc_pair<16 * T + 2 * s>();
                                     });
                                 static_for<0, 8>([&](auto tc) {
                                     constexpr int T = decltype(tc)::value;
                                     if constexpr (I == 6 + (8 * T + 8) / 3)
                                         static_for<0, 4>([&](auto q) { acc_from_lds<16 * T + 4 * decltype(q)::value, T * 128 + 32 * decltype(q)::value>(h16 + C::o_b3); });
                                 });
                                 // row tiles 8 .. 15 while layer 3 works on 0 .. 7: row tile 8 + U takes the operands of row
                                 // tile U behind its last product; then layer 2's biases for the next tile
                                 if constexpr (E >= 16 && E < 144 && E % 2 == 0) {
                                     constexpr int U = E / 16 - 1, s = E % 16 / 2;
                                     h2[U][s / 4][s % 4] = acc_pair<16 * (8 + U) + 2 * s>();
                                 }
                                 if constexpr (E >= 32 && E < 160 && E % 16 % 2 == 1 && E % 16 < 8) {
                                     constexpr int T = 8 + E / 16 - 2, q = E % 16 / 2;
                                     acc_from_lds<16 * T + 4 * q, T * 128 + 32 * q>(h16 + C::o_b2);
                                 }
                                 if constexpr (E == 8 * C::KS3 - 16) read_wl(IC<0>{});
                             });
                });
            });
        }
    }
#undef AIF_FENCE
    finish(tile - 1, (n_mine - 1) & 1, prev, z);
    wait_vmcnt<0>();                                            // what was sent for behind the last tile has landed
}

hipError_t mlp_acc_c5f(const Model &m, const Batch &b, const void *X, const MlpPack &pk, const float *bias1, hipStream_t s)
{
    auto kern = k_mlp_acc3;
    if (!pk.w0_user || !m.x_tiled) return hipErrorInvalidValue;
    static bool attr_set = false;
    if (!attr_set) {
        hipError_t e = hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, Acc3::lds_bytes);
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    const int n_tiles = b.n_blk * (ROW_BLOCK / Acc3::ROWS), blocks = n_tiles < n_cu() ? n_tiles : n_cu();
    hipLaunchKernelGGL(kern, dim3(blocks), dim3(256), Acc3::lds_bytes, s, m.n_items, b.reqs, b.blk_req, b.blk_slot, (const char *)X,
                       x_layout(m).tile_bytes, pk, bias1, n_tiles);
    return hipGetLastError();
}

}  // namespace aif
