// a6-a7 on the matrix cores for large batches: a head of two hidden layers whose second layer accumulates while the first is
// produced.
//
// Same products, operands and orders of addition as k_mlp_chain.h (a candidate's bits do not depend on which of the two
// serves it), in another order of work: as soon as a row tile of layer 1 is through its ReLU it is contracted into ALL row
// tiles of layer 2, whose accumulators stay in registers for the whole tile.  Layer 1's activations then live for one row
// tile only, and the registers that frees (512 a lane with one wave per SIMD) take a SECOND column tile: a wave owns 64
// candidates and every weight fragment read from LDS feeds two MFMAs.  A block is persistent: it takes a contiguous run of
// tiles of 256 candidates, the weight stream runs on from tile to tile, and the next tile's input rows, biases and ids
// arrive in LDS while this one is computed.
//
// Stage t = 1 .. NT1 - 1 of a tile: layer 1's row tile t (KS1 fragments), then layer 2's k-steps of row tile t - 1 (2 NT2
// fragments) while the vector ALU turns row tile t into the next stage's operands.  Stage 0 (the edge): the previous
// tile's last k-steps of layer 2 with its ->1 layer, then row tile 0 of this one.
//
// What bounds it: the vector work that does not overlap, and power.  64 x 10^4 candidates, 128 -> 512 -> 256, this and the chain
// in turn on one box: 192 us against 213 (187 and 205 on another; 1.31 PFLOP/s), in as many cycles, 331 k against 336 k -- every weight
// fragment read from LDS feeds two MFMAs, and what that saves in energy comes back as clock, 1.72 against 1.58 GHz (a bare loop
// of MFMAs on such operands holds 1.81).  Matrix cores busy 0.75 of the cycles (the chain 0.73); with the other vector instructions
// laid end to end 0.96, so a tile gets shorter only with fewer of those or with some under an MFMA.  Copies of it without the barriers and
// waits took the same time, without the fragment reads 9 us less, without the weight loads 5 us less.  With the other work in lumps
// (a stage's loads at once, the ->1 layer at the tile's end) it took 215-224 us: one wave has nothing else to issue.
#include "k_mlp_chain.h"
#include "k_mlp_acc.h"

namespace aif {

template <int KS1, int NT1, int NT2> struct Acc {
    static constexpr int WAVES = 4, SLOTS = 7, ROWS = WAVES * 64;
    static constexpr int H1 = 32 * NT1, H2 = 32 * NT2, KS2 = 2 * NT1;
    static constexpr int SF = KS1 + 2 * NT2;                                    // fragments of a stage
    static constexpr int HF = SF / 2, LPW = HF / WAVES;                         // fragments of half a stage, loads per wave
    static constexpr int slot_bytes = HF * 1024, ring_bytes = SLOTS * slot_bytes;
    static constexpr int x_wave = 2 * KS1 * 1024;                               // input fragments of a wave's 64 candidates
    static constexpr int o_x = ring_bytes, o_b1 = o_x + WAVES * x_wave, o_b2 = o_b1 + 2 * H1 * 4, o_wl = o_b2 + H2 * 4,
                         o_id = o_wl + H2 * 4, lds_bytes = o_id + 2 * ROWS * 4;
    // Loads a wave sends besides the weights in the middle of half I (0 .. 2 NT1 - 1, over the end of a tile): the next
    // tile's input rows one by one, then its layer-1 biases and ids.
    static constexpr int IX = 4, IREQ = IX + 2 * KS1 + 2;
    static constexpr int extra(int I) { return I < 0 ? extra(I + 2 * NT1) : I >= IX && I < IX + 2 * KS1 ? 1 : I == IREQ ? 2 : 0; }
    // how many of its loads may be in flight there for the half `ahead` halves on to have landed
    static constexpr int left(int I, int ahead)
    {
        int n = 0;
        for (int k = 1; k <= SLOTS - 2 - ahead; ++k) n += LPW + extra(I - k);
        return n;
    }
    static_assert(KS1 % WAVES == 0 && SF % (2 * WAVES) == 0 && KS1 <= HF, "every wave moves the same number of fragments per half");
    static_assert(lds_bytes <= 160 * 1024, "LDS");
    static_assert(ROWS == ROW_BLOCK, "a tile is one scheduling block: one request, one user slot");
    static_assert(H1 * 4 == 2048, "layer-1 biases: 1 KB a wave, twice");
    static_assert(2 * NT2 * 16 <= 256, "layer 2's accumulators");
    static_assert(KS1 <= NT2 && KS1 >= 4, "the input rows are read while layer 2 of the tile before ends");
    static_assert(IREQ + SLOTS < 2 * NT1, "the next tile's data has landed before its edge");
};

template <int KS1, int NT1, int NT2, int RING>
__global__ __launch_bounds__(256, 1) void k_mlp_acc(int64_t n_items, const ReqDesc *__restrict__ reqs,
                                                    const int32_t *__restrict__ blk_req, const int32_t *__restrict__ blk_slot,
                                                    const char *__restrict__ X, uint32_t xtile_bytes, MlpPack pk,
                                                    const float *__restrict__ bias1, int n_tiles)
{
    using C = Acc<KS1, NT1, NT2>;
    constexpr int SF = C::SF, HF = C::HF, H1 = C::H1, H2 = C::H2, LPW = C::LPW;
    static_assert(SF % RING == 0 && RING - 1 <= HF / 2, "fragment registers carry over; never read past a confirmed half");
    extern __shared__ __align__(16) char lds[];
    const int lane = threadIdx.x & 63, h = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t L0 = lds_address(lds), lane16 = lane * 16;

    // workgroups go to the 8 XCDs in turn, each with an L2 of its own; every XCD takes a contiguous run of the tiles, so
    // that the tiles that stream one user's layer-1 weights share an L2
    const int nb = (int)gridDim.x, b = (int)blockIdx.x;
    const int idx = nb % 8 ? b : (b & 7) * (nb >> 3) + (b >> 3);
    const int first = (int)((int64_t)idx * n_tiles / nb), n_mine = (int)((int64_t)(idx + 1) * n_tiles / nb) - first;

    auto out_of = [&](int r) {
        const ReqDesc *q = reqs + r;
        return AccOut{q->cand_ids, q->logits_out, q->scores_out, q->n_cand, q->row_base};
    };
    // ---- copies into LDS, all untracked: completion by the waits in the middle of a half
    // A stage's fragments: row tile t of layer 1, then layer 2's k-steps 2 kk, 2 kk + 1.  Wave w moves fragments w, w + 4, ..;
    // those of a matrix lie a fixed stride apart, which the lane offset takes.
    constexpr int N1 = KS1 / C::WAVES, N2 = 2 * NT2 / C::WAVES;
    uint32_t v1[N1], v2[N2];
#pragma unroll
    for (int j = 0; j < N1; ++j) v1[j] = lane16 + j * C::WAVES * 1024;
#pragma unroll
    for (int j = 0; j < N2; ++j) v2[j] = lane16 + j * (C::WAVES / 2) * C::KS2 * 1024;
    const char *w1p = pk.w[1] + (size_t)((wave >> 1) * C::KS2 + (wave & 1)) * 1024;
    auto send = [&](auto jc, uint32_t dst, const char *w0w, int t, int kk) {       // load J of a stage; w0w: layer 1's weights + 1 KB x wave
        constexpr int J = decltype(jc)::value;
        if constexpr (J < N1)
            dma_s<16>(w0w + t * KS1 * 1024, v1[J], dst, J % LPW * C::WAVES * 1024);
        else
            dma_s<16>(w1p + kk * 2048, v2[J - N1], dst, J % LPW * C::WAVES * 1024);
    };
    const uint32_t xdst = L0 + C::o_x + wave * C::x_wave;
    auto send_x = [&](auto kc, const char *src) {               // fragment K of a wave's input rows; src: its first 32 rows
        constexpr int K = decltype(kc)::value;
        dma_s<16>(src + (K >= KS1 ? (size_t)xtile_bytes : 0) + K % KS1 * 1024, lane16, xdst, K * 1024);
    };
    auto x_of = [&](int tile) { return X + (size_t)(tile * (C::ROWS / X_TILE) + wave * 2) * xtile_bytes; };
    auto send_req = [&](int tile, const AccOut &rd, int slot, int par) {
        dma_s<16>((const char *)(bias1 + (size_t)slot * H1) + (wave & 1) * 1024, lane16, L0 + C::o_b1 + par * H1 * 4 + (wave & 1) * 1024, 0);
        int local = tile * C::ROWS - rd.row_base + wave * 64 + lane;      // a lane with no candidate reads the first id
        if (local >= rd.n_cand) local = 0;
        dma_s<4>(rd.cand_ids, 4 * local, L0 + C::o_id + par * C::ROWS * 4 + wave * 256, 0);
    };

    // ---- the first tile, and the request of the second (past the block's last tile: the batch's last, whose data is then
    // sent for and not used)
    int tile = first;
    auto at = [&](int t) { return t < n_tiles ? t : n_tiles - 1; };
    const int r0 = blk_req[tile], sl0 = blk_slot[tile];
    int nr = blk_req[at(tile + 1)], nslot = blk_slot[at(tile + 1)];
    {
        const char *src = x_of(tile);
        static_for<0, 2 * KS1>([&](auto kc) { send_x(kc, src); });
    }
    AccOut cur = out_of(r0), nxt = cur, prev = cur;
    prev.n_cand = INT32_MIN;                                    // no tile before the first
    const char *w0c = pk.w0_user + (size_t)sl0 * pk.w0_stride + wave * 1024, *w0n = w0c;
    static_for<0, 3 * 2 * LPW>([&](auto ic) {                   // (layer 2's part of stage 0 meets no operands yet)
        constexpr int T = decltype(ic)::value / (2 * LPW), J = decltype(ic)::value % (2 * LPW);
        send(IC<J>{}, L0 + wave * 1024 + (2 * T + J / LPW) * C::slot_bytes, w0c, T, T ? T - 1 : 0);
    });
    send_req(tile, cur, sl0, 0);
    {
        float *sb2 = (float *)(lds + C::o_b2), *swl = (float *)(lds + C::o_wl);
        if ((int)threadIdx.x < H2) {
            sb2[threadIdx.x] = pk.bias[1][threadIdx.x];
            swl[threadIdx.x] = pk.wlast[threadIdx.x];
        }
    }
    const float bl = pk.blast[0];
    wait_vmcnt<0>();
    __syncthreads();

    auto lds8 = [&](uint32_t a) -> bf16x8 { return *(const bf16x8 __attribute__((address_space(3))) *)(uintptr_t)a; };
    auto lds4 = [&](uint32_t a) -> f32x4 { return *(lds_f32x4_t)(uintptr_t)a; };
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    f32x16 acc1[2][2];                      // layer 1's accumulators [parity of the row tile][column tile]; layer 2's: a0 .. a255
    reserve_acc();
    bf16x8 x[2][KS1];
    u32x4 hb[2][2][2] = {};                 // hb[parity of the row tile][column tile][k-step]: eight bf16
    bf16x8 areg[RING];
    float z[2] = {0.f, 0.f};
    f32x4 wlv[2][4];
    // four of an accumulator's biases: features 8 q + 4 h + i
    auto preload_q = [&](uint32_t addr, int q, f32x16 &a) {
        const f32x4 v = lds4(addr + 32 * q);
        a[4 * q + 0] = v.x;
        a[4 * q + 1] = v.y;
        a[4 * q + 2] = v.z;
        a[4 * q + 3] = v.w;
    };
    const uint32_t h16 = L0 + 16 * h, rb_x = xdst + lane16;
    uint32_t b1c = h16 + C::o_b1, b1n = b1c + H1 * 4;           // this and the next tile's layer-1 biases
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        preload_q(b1c, q, acc1[0][0]);
        preload_q(b1c, q, acc1[0][1]);
    }
    // the ring: offset of the current stage's first half, this lane's place in both halves and in the two after them
    uint32_t ring = 0;
    auto past = [&](uint32_t r, int halves) {
        const uint32_t p = r + halves * C::slot_bytes;
        return p < (uint32_t)C::ring_bytes ? p : p - C::ring_bytes;
    };
    uint32_t rb[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) rb[k] = L0 + lane16 + k * C::slot_bytes;
    auto advance = [&]() {
        ring = past(ring, 2);
        rb[0] = rb[2];
        rb[1] = rb[3];
        rb[2] = L0 + lane16 + past(ring, 2);
        rb[3] = L0 + lane16 + past(ring, 3);
    };
    // The place of the fragment of step F of stage t (in the edge layer 2's fragments come first); F >= SF: of the next stage
    auto frag = [&](auto tc, auto fc) -> bf16x8 {
        constexpr int F = decltype(fc)::value, T = decltype(tc)::value + F / SF, P = F % SF;
        constexpr int pos = T % NT1 ? P : (P < 2 * NT2 ? P + KS1 : P - 2 * NT2);
        return lds8(rb[F / SF * 2 + pos / HF] + pos % HF * 1024);
    };
    static_for<0, RING - 1>([&](auto fc) { areg[decltype(fc)::value] = frag(IC<0>{}, fc); });
#define AIF_FENCE __builtin_amdgcn_sched_barrier(0)
    // Step P of a stage: one fragment, two products, each with a share of the other work behind it (`gap`): a wave has its
    // SIMD to itself, so whatever is issued hides behind a product or not at all -- seven instructions fit behind one.
    auto step = [&](auto tc, auto pc, auto &&gap) {
        constexpr int T = decltype(tc)::value, P = decltype(pc)::value, I = T ? P - KS1 : P, PAR = T ? (T & 1) ^ 1 : 1;
        constexpr bool first_layer = T ? P < KS1 : P >= 2 * NT2;
        areg[(P + RING - 1) % RING] = frag(tc, IC<P + RING - 1>{});
        if constexpr (first_layer) {
            constexpr int K = T ? P : P - 2 * NT2;
            mfma_v(acc1[T & 1][0], areg[P % RING], x[0][K]);
            AIF_FENCE;
            gap(IC<2 * P>{});
            AIF_FENCE;
            mfma_v(acc1[T & 1][1], areg[P % RING], x[1][K]);
        } else {
            mfma_a<16 * (I / 2)>(areg[P % RING], __builtin_bit_cast(bf16x8, hb[PAR][0][I % 2]));
            AIF_FENCE;
            gap(IC<2 * P>{});
            AIF_FENCE;
            mfma_a<16 * (NT2 + I / 2)>(areg[P % RING], __builtin_bit_cast(bf16x8, hb[PAR][1][I % 2]));
        }
        AIF_FENCE;
        gap(IC<2 * P + 1>{});
        AIF_FENCE;
    };
    // pair S = 0 .. 15 of acc1's features into operands: column tile S / 8, values 2 (S % 8) and the next
    auto convert = [&](auto sc, auto parc) {
        constexpr int c = decltype(sc)::value / 8, i = decltype(sc)::value % 8, PAR = decltype(parc)::value;
        hb[PAR][c][i / 4][i % 4] = relu_pair(acc1[PAR][c][2 * i], acc1[PAR][c][2 * i + 1]);
    };
    // The ->1 layer: unit V = 0 .. 8 NT2 - 1 takes four features (V / 2 % 4) of row tile V / 8 of column tile V % 2; one unit a
    // gap, from gap 6 of the edge on through the next stage (the accumulators of row tile T are complete behind gap
    // 4 T + 3 of the edge and needed again in gap 16 + 4 T of the stage after it).  Its weights are read four gaps ahead of a
    // row tile's first unit, the accumulators are loaded with the biases again four gaps behind each unit.
    auto dot_unit = [&](auto vc) {
        constexpr int V = decltype(vc)::value, T = V / 8, q = V / 2 % 4, c = V % 2, A = 16 * (c * NT2 + T) + 4 * q;
        z[c] = dot4(z[c], wlv[T & 1][q], acc_relu<A>(), acc_relu<A + 1>(), acc_relu<A + 2>(), acc_relu<A + 3>());
        asm volatile("" : "+v"(z[c]));
    };
    auto dot_gap = [&](auto gc, auto last) {                    // gap of the edge and, counted on, of the stage behind it
        constexpr int G = decltype(gc)::value;
        if constexpr (G % 8 == 2 && G / 8 < NT2) {
#pragma unroll
            for (int q = 0; q < 4; ++q) wlv[G / 8 & 1][q] = lds4(h16 + C::o_wl + (G / 8) * 128 + 32 * q);
        }
        if constexpr (G >= 6 && G - 6 < 8 * NT2) dot_unit(IC<G - 6>{});
        if constexpr (!decltype(last)::value && G >= 10 && G - 10 < 8 * NT2) {
            constexpr int V = G - 10, T = V / 8, q = V / 2 % 4, c = V % 2;
            acc_from_lds<16 * (c * NT2 + T) + 4 * q, T * 128 + 32 * q>(h16 + C::o_b2);
        }
    };
    auto finish = [&](int t, int par, const AccOut &rd) {        // logits and scores of a tile: lane = candidate
        const float z0 = z[0] + __shfl_xor(z[0], 32, 64), z1 = z[1] + __shfl_xor(z[1], 32, 64);
        float zz = (h ? z1 : z0) + bl;
        const int32_t id = *(const int32_t __attribute__((address_space(3))) *)(uintptr_t)(L0 + C::o_id + par * C::ROWS * 4 + wave * 256 + lane * 4);
        const int local = t * C::ROWS - rd.row_base + wave * 64 + lane;
        if (local < rd.n_cand) {
            if (id < 0 || id >= n_items) zz = __uint_as_float(0x7FC00000u);
            typedef float __attribute__((address_space(1))) *gfloat_t;
            ((gfloat_t)rd.logits_out)[local] = zz;
            if (rd.scores_out) ((gfloat_t)rd.scores_out)[local] = 1.0f / (1.0f + __expf(-zz));
        }
        z[0] = z[1] = 0.f;
    };
    // In the middle of half I: this wave's share of the half AHEAD on has landed; behind the barrier everyone's has, and
    // nobody reads the half before any more: its slot takes the half SLOTS - 1 on.
    auto turn = [&](auto ic, auto ac) {
        wait_vmcnt<C::left(decltype(ic)::value, decltype(ac)::value)>();
        asm volatile("s_barrier" ::: "memory");
    };
    // load J of the half sent in half HH of stage T, i.e. of stage T + 3
    auto refill = [&](auto tc, auto jc, uint32_t dst) {
        constexpr int Q = decltype(tc)::value + 3;
        send(jc, dst, Q < NT1 ? w0c : w0n, Q % NT1, Q % NT1 ? Q % NT1 - 1 : NT1 - 1);
    };

    for (int n = 0;; ++n) {
        // the next tile's request, found in the edge before, and the index of the one after
        const int next_tile = at(tile + 1);
        nxt = out_of(nr);
        w0n = pk.w0_user + (size_t)nslot * pk.w0_stride + wave * 1024;
        const int next_slot = nslot;
        nr = blk_req[at(tile + 2)];
        nslot = blk_slot[at(tile + 2)];
        // Stage 0.  The first tile's meets no tile to end and the last one's no tile to begin: what they compute there
        // is overwritten or never stored.
        {
            const uint32_t d0 = L0 + wave * 1024 + past(ring, C::SLOTS - 1), d1 = L0 + wave * 1024 + ring;
            constexpr int PT = SF - RING + 1, GT = 2 * PT;      // from there on the next stage's fragments are read
            static_for<0, SF>([&](auto pc) {
                constexpr int P = decltype(pc)::value;
                if constexpr (P == PT) {            // every fragment of the stage is in registers: layer 1's lie in the slot that is refilled
                    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
                    turn(IC<1>{}, IC<1>{});
                }
                step(IC<0>{}, pc, [&](auto gc) {
                    constexpr int G = decltype(gc)::value;
                    if constexpr (G == HF) turn(IC<0>{}, IC<1>{});
                    if constexpr (G > HF && G <= HF + LPW) refill(IC<0>{}, IC<G - HF - 1>{}, d0);
                    if constexpr (G >= GT && G < GT + LPW) refill(IC<0>{}, IC<LPW + G - GT>{}, d1);
                    if constexpr (G % 2 == 0 && P < 2 * KS1) x[P / KS1][P % KS1] = lds8(rb_x + P * 1024);
                    if constexpr (G >= 2 * SF - 9 && G < 2 * SF - 1) preload_q(b1c + 128, (G - 2 * SF + 9) / 2, acc1[1][(G - 2 * SF + 9) % 2]);
                    dot_gap(gc, IC<0>{});
                });
            });
            // the scalar loads above (a wait that the compiler sees: with scalar loads in flight it would empty the queue at
            // every fragment)
            __builtin_amdgcn_s_waitcnt(0xC07F);                 // lgkmcnt(0)
            asm volatile("" ::"s"(nxt.cand_ids), "s"(nxt.logits_out), "s"(nxt.scores_out), "s"(nxt.n_cand), "s"(nxt.row_base), "s"(nr), "s"(nslot));
            advance();
        }
        if (n == n_mine) break;
        const char *xsrc = x_of(next_tile);
        static_for<1, NT1>([&](auto tc) {
            constexpr int T = decltype(tc)::value;
            const uint32_t d0 = L0 + wave * 1024 + past(ring, C::SLOTS - 1), d1 = L0 + wave * 1024 + ring;
            // the biases of the row tile after this one: of the next tile behind the last
            const uint32_t bnext = T == NT1 - 1 ? b1n : b1c + 128 * (T + 1);
            static_for<0, SF>([&](auto pc) {
                constexpr int P = decltype(pc)::value;
                // layer 2's biases read in this stage (the last in gap 25) have landed: only fragments were asked for since
                if constexpr (T == 1 && P == 16) asm volatile("s_waitcnt lgkmcnt(3)" ::: "memory");
                step(tc, pc, [&](auto gc) {
                    constexpr int G = decltype(gc)::value, G1 = 3 * HF;
                    if constexpr (G == HF) turn(IC<2 * T>{}, IC<1>{});
                    if constexpr (G > HF && G <= HF + LPW) refill(tc, IC<G - HF - 1>{}, d0);
                    if constexpr (G == HF + LPW + 1) {
                        if constexpr (2 * T >= C::IX && 2 * T < C::IX + 2 * KS1) send_x(IC<2 * T - C::IX>{}, xsrc);
                        if constexpr (2 * T == C::IREQ) send_req(next_tile, nxt, next_slot, (n + 1) & 1);
                    }
                    if constexpr (G == G1) turn(IC<2 * T + 1>{}, IC<T == NT1 - 1 ? 2 : 1>{});       // the edge reads both its halves from the start
                    if constexpr (G > G1 && G <= G1 + LPW) refill(tc, IC<LPW + G - G1 - 1>{}, d1);
                    if constexpr (G == 2 * SF - 1 && 2 * T + 1 >= C::IX && 2 * T + 1 < C::IX + 2 * KS1) send_x(IC<2 * T + 1 - C::IX>{}, xsrc);
                    if constexpr (T == 1 && G < 16) convert(gc, IC<0>{});
                    if constexpr (T == 1) dot_gap(IC<2 * SF + G>{}, IC<0>{});
                    if constexpr (G >= 2 * KS1 + 4 && G < 2 * KS1 + 20) convert(IC<G - 2 * KS1 - 4>{}, IC<T & 1>{});
                    if constexpr (G >= 2 * SF - 9 && G < 2 * SF - 1) preload_q(bnext, (G - 2 * SF + 9) / 2, acc1[(T + 1) & 1][(G - 2 * SF + 9) % 2]);
                    if constexpr (T == 2 && G == 0) finish(tile - 1, (n - 1) & 1, prev);
                });
            });
            advance();
        });
        prev = cur;
        cur = nxt;
        w0c = w0n;
        const uint32_t bt = b1c;
        b1c = b1n;
        b1n = bt;
        ++tile;
    }
#undef AIF_FENCE
    static_for<2 * SF, 8 * NT2 + 6>([&](auto gc) { dot_gap(gc, IC<1>{}); });
    finish(tile - 1, (n_mine - 1) & 1, prev);
    wait_vmcnt<0>();                                            // what was sent for behind the last tile has landed
}

hipError_t mlp_acc_c3f(const Model &m, const Batch &b, const void *X, const MlpPack &pk, const float *bias1, hipStream_t s)
{
    using C = Acc<8, 16, 8>;
    auto kern = k_mlp_acc<8, 16, 8, 6>;
    if (!pk.w0_user || !m.x_tiled) return hipErrorInvalidValue;
    static bool attr_set = false;
    if (!attr_set) {
        hipError_t e = hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, C::lds_bytes);
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    const int blocks = b.n_blk < n_cu() ? b.n_blk : n_cu();
    hipLaunchKernelGGL(kern, dim3(blocks), dim3(256), C::lds_bytes, s, m.n_items, b.reqs, b.blk_req, b.blk_slot, (const char *)X,
                       x_layout(m).tile_bytes, pk, bias1, b.n_blk);
    return hipGetLastError();
}

}  // namespace aif
