// Eq. 6, 7, 9 with the similarity on the matrix cores.
//
// The number of equal bits of two d'-bit signatures is a contraction: with the bits written as signs their dot product
// is (equal - unequal), so 2 * equal = d' + dot.  The signs are fp4 values (+-1, four bits each), and one
// v_mfma_scale_f32_32x32x64_f8f6f4 forms 32 x 32 cells over 64 of them in two blocks of 32, each with a scale of its own:
// a row's first block is 32 bits of one history item, its second block the same 32 bits of another, the column holds the
// candidate's bits twice.  With scales 2^(8 - SH) and 2^(16 - SH) and a start of 2^23 + d' (2^(8 - SH) + 2^(16 - SH)) a
// cell's mantissa is, exactly, 2^(8 - SH) * 2 equal_1 + 2^(16 - SH) * 2 equal_2 -- two history items a cell at half the
// matrix time and half the operand bytes an item takes as int8.  The candidates are the columns (a lane owns one and
// gets 32 history items' values of it per tile), the history items the rows: written once per request by k_lsh_expand
// in the order the instruction reads them, streamed by every wave from L2.  Only the product over ALL bits matters, so
// any assignment of bits to the instruction's k index serves, as long as rows and columns use the same one.
//
// What is left per (candidate, history item) is Eq. 9's count into tiers, and the vector ALU is what binds, so it is
// done on four values at a time.  N divides 2 d' to a power of two here, so tier = (2 * equal) >> SH: the scales put the
// first item's tier into the low bits of the cell's second byte and the other's into its third.  One byte permute and a
// mask bring the tiers of two cells into one word, a second permute (a table of eight bytes) turns them into four
// one-hot bytes, and the words of one-hot bytes are summed bit position by bit position in a network of carry-save
// adders (two 3-input bit operations each) whose planes hold the counts in binary; the carries of two passes go through
// the upper planes in one trip.  At the end (or every 960 or 1,984 words) the planes are read out: the four bytes' counters
// are added plane by plane, then gathered.  1.3 vector instructions per value in the loop, 1.6 with the ends (1.75 and 2.1 with
// one item a cell, as +-1 int8 on v_mfma_i32_32x32x32_i8: 465 us for 64 x 10^4 candidates x 10^4 items of 64 bits, 836 for
// 8 x 10^4 x 10^5 of 128, against 345 and 542; the paired carries and the read-out by planes, where every plane and tier took a
// mask and a population count, took the two calls from 419 to 403 us and from 613 to 605).
// Two corrections at the end: the rows past the history's end are zero vectors, which count as d' / 2 equal bits and
// are taken off that tier again; a signature equal to the candidate's in every bit gives tier index N, whose one-hot
// byte is empty -- the last tier's count is the history length less all the others.
#include <algorithm>

#include "k_lsh_blocks.h"

namespace aif {

typedef int v8i __attribute__((ext_vector_type(8)));
typedef float v16f __attribute__((ext_vector_type(16)));

constexpr int SMT_PART_BLOCKS = 2048; // a batch of fewer blocks than this has its histories cut into parts, a block each
constexpr int SMT_MAX_PARTS = 16;
constexpr int SMT_GROUP = 4;         // row tiles per pass of the adder network: 32 words per column tile
// Column tiles of 32 candidates a wave keeps (a row tile's bytes serve them all; what the registers allow): the block's 256
// candidates are SMT_GROUPS groups of columns, and the SMT_SHARE waves that have a group in common halve the history.
constexpr int SMT_COLS = 4, SMT_GROUPS = LSH_BLOCK / (32 * SMT_COLS), SMT_SHARE = 4 / SMT_GROUPS;
// Planes of weight 32 .. above the network's ones .. sixteens, and the passes between read-outs that they can count (an
// even number, of 32 words each; + 24 of a ragged end).  Signatures of up to 64 bits keep to three waves a SIMD with one
// plane fewer: its registers hold the carry that waits for its partner.
constexpr int smt_planes(int ks) { return ks <= 2 ? 5 : 6; }
constexpr int smt_flush(int ks) { return ks <= 2 ? 30 : 62; }

__device__ __forceinline__ void csa(uint32_t &sum, uint32_t &carry, uint32_t a, uint32_t b, uint32_t c)
{
    sum = __builtin_amdgcn_bitop3_b32(a, b, c, 0x96);          // a ^ b ^ c
    carry = __builtin_amdgcn_bitop3_b32(a, b, c, 0xE8);        // majority
}

// KS: k-steps of 32 bits (d' = 32 KS); a wave's candidates' operands stay in registers, 16 KS of them.  gridDim.y > 1: the
// history is cut into that many parts as well, a block each, and the counts go to `parts` [part][candidate slot][tier] for
// k_lsh_simtier_finish -- for batches too small to fill the chip otherwise (a handful of users with long histories).
// Every wave reads its row tiles from L2 itself, two to four tiles in flight.
template <int KS>
__device__ __forceinline__ void lsh_simtier_block(const LshModel &m, const LshBatch &b, const uint8_t *__restrict__ sig_table,
                                                  const v4i *__restrict__ hist, size_t req_stride, int sh, int32_t *__restrict__ parts,
                                                  int blk, int part_no, int n_parts)
{
    constexpr int SMT_PLANES = smt_planes(KS), SMT_FLUSH = smt_flush(KS);
    static_assert(SMT_FLUSH % 2 == 0 && 32 * SMT_FLUSH + 24 < 32 << SMT_PLANES, "the planes count every word between read-outs");
    __shared__ int32_t cnt[LSH_MAX_TIERS][LSH_BLOCK];
    // as in the vector-ALU kernel: the blocks of one user go to one XCD, whose L2 then holds that user's history
    {
        const int per_xcd = b.n_blk >> 3;
        if (blk < 8 * per_xcd) blk = (blk & 7) * per_xcd + (blk >> 3);
    }
    const int r = b.blk_req[blk];
    if (r < 0) return;
    const LshReqDesc rd = b.reqs[r];
    const int tid = threadIdx.x, lane = tid & 63, col = lane & 31, h = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);             // the same in every lane: the loop's bounds are scalars
    const int cg = wave % SMT_GROUPS, hh = wave / SMT_GROUPS;   // which candidates of the block, which share of the history
    const int first = blk * LSH_BLOCK - rd.cand_base;

    // column operand: each k-step's 32 bits of this lane's candidate in each of the column tiles
    v4i bf[SMT_COLS][KS];
#pragma unroll
    for (int ct = 0; ct < SMT_COLS; ++ct) {
        const int local = first + cg * (SMT_COLS * 32) + ct * 32 + col;
        int64_t id = local < rd.n_cand ? rd.cand_ids[local] : 0;
        if (id < 0 || id >= m.n_items) id = 0;
        const uint32_t *p = (const uint32_t *)(sig_table + (size_t)id * (KS * 4));
#pragma unroll
        for (int s = 0; s < KS; ++s) bf[ct][s] = fp4_signs(p[s]);              // the same bits for both of a row's items
    }
#pragma unroll
    for (int t = 0; t < LSH_MAX_TIERS; ++t) cnt[t][tid] = 0;
    __syncthreads();

    const int nrt = (rd.seq_len + SMT_TILE - 1) / SMT_TILE;
    const int per_part = (nrt + n_parts - 1) / n_parts;          // row tiles of this block ...
    const int part_begin = min(nrt, part_no * per_part), part_end = min(nrt, part_begin + per_part);
    const int per_wave = (part_end - part_begin + SMT_SHARE - 1) / SMT_SHARE;           // ... and of this wave
    const int rt_begin = min(part_end, part_begin + hh * per_wave), rt_end = min(part_end, rt_begin + per_wave);
    const v4i *__restrict__ hrow = hist + (size_t)r * req_stride + lane;

    // one-hot byte of tier t: bit t; the permute's selectors 0..3 take the second operand's bytes, 4..7 the first's
    constexpr uint32_t HOT_LO = 0x08040201u, HOT_HI = 0x80402010u;
    uint32_t ones[SMT_COLS], twos[SMT_COLS], fours[SMT_COLS], eights[SMT_COLS], sixteens[SMT_COLS], plane[SMT_COLS][SMT_PLANES];
#pragma unroll
    for (int ct = 0; ct < SMT_COLS; ++ct) {
        ones[ct] = twos[ct] = fours[ct] = eights[ct] = sixteens[ct] = 0;
#pragma unroll
        for (int j = 0; j < SMT_PLANES; ++j) plane[ct][j] = 0;
    }
    // The planes' 32 counters, a byte's bit each, to eight counts: the bytes are added as the planes stand (a full adder
    // per plane, twice), then a counter's bits are gathered, tiers t and t + 4 side by side.  A count fits sixteen bits:
    // four bytes of at most 2,047 words.
    auto read_out = [&]() {
#pragma unroll
        for (int ct = 0; ct < SMT_COLS; ++ct) {
            const int cand = cg * (SMT_COLS * 32) + ct * 32 + col;
            constexpr int NP = 5 + SMT_PLANES;
            uint32_t p[NP + 2] = {ones[ct], twos[ct], fours[ct], eights[ct], sixteens[ct]};
#pragma unroll
            for (int j = 0; j < SMT_PLANES; ++j) p[5 + j] = plane[ct][j];
#pragma unroll
            for (int fold = 0; fold < 2; ++fold) {
                uint32_t carry = 0;
#pragma unroll
                for (int j = 0; j < NP + fold; ++j) csa(p[j], carry, carry, p[j], p[j] >> (fold ? 8 : 16));
                p[NP + fold] = carry;
            }
            uint32_t n[LSH_MAX_TIERS / 2] = {};
#pragma unroll
            for (int j = 0; j < NP + 2; ++j) {
                const uint32_t y = (p[j] & 0xFFFFu) | (p[j] << 12 & 0xFFFF0000u);               // tiers 4 .. 7 from bit 16 up
#pragma unroll
                for (int t = 0; t < LSH_MAX_TIERS / 2; ++t) n[t] |= (y & 0x00010001u << t) << j;
            }
#pragma unroll
            for (int t = 0; t < LSH_MAX_TIERS / 2; ++t) {
                const uint32_t lo = (n[t] & 0xFFFFu) >> t, hi = n[t] >> (16 + t);
                if (lo) atomicAdd(&cnt[t][cand], (int32_t)lo);
                if (hi) atomicAdd(&cnt[t + LSH_MAX_TIERS / 2][cand], (int32_t)hi);
            }
            ones[ct] = twos[ct] = fours[ct] = eights[ct] = sixteens[ct] = 0;
#pragma unroll
            for (int j = 0; j < SMT_PLANES; ++j) plane[ct][j] = 0;
        }
    };

    // The one-hot words of one row tile against column tile ct.  The cells' start value is kept in registers of its own
    // (it is no inline constant; formed anew it would cost an instruction per cell).
    const uint32_t tier_mask = (uint32_t)(2 * m.n_tiers - 1) * 0x01010101u;
    const int scale = 127 + (h ? 16 - sh : 8 - sh);             // this lane's block of the row: E8M0
    v16f start;
#pragma unroll
    for (int i = 0; i < 16; ++i) start[i] = (float)((1 << 23) + ((32 * KS) << (8 - sh)) + ((32 * KS) << (16 - sh)));
#pragma unroll
    for (int i = 0; i < 16; ++i) asm volatile("" : "+v"(start[i]));
    auto mfma_step = [&](const v16f &acc, const v4i &row, const v4i &cand) __attribute__((always_inline)) {
        const v8i a = {row[0], row[1], row[2], row[3], 0, 0, 0, 0};                        // fp4 operands take four registers
        const v8i c = {cand[0], cand[1], cand[2], cand[3], 0, 0, 0, 0};
        return __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a, c, acc, 4, 4, 0, scale, 0, 127);
    };
    auto word = [&](const v16f &acc, int q) __attribute__((always_inline)) {
        // second and third bytes of cells 2q and 2q + 1; the low bits of each are a tier, 0 .. N (above the second
        // byte's tier lies what the other item's count leaves below its own tier: 2^(17 - SH) and up)
        const uint32_t t = __builtin_amdgcn_perm(__float_as_uint(acc[2 * q + 1]), __float_as_uint(acc[2 * q]), 0x06050201u);
        return __builtin_amdgcn_perm(HOT_HI, HOT_LO, t & tier_mask);
    };
    auto tile_words = [&](const v4i(&af)[KS], int ct, uint32_t(&w)[8]) {
        v16f acc = start;
#pragma unroll
        for (int s = 0; s < KS; ++s) acc = mfma_step(acc, af[s], bf[ct][s]);
#pragma unroll
        for (int q = 0; q < 8; ++q) w[q] = word(acc, q);
    };
    auto load_rows = [&](int rt, v4i(&af)[KS]) {
#pragma unroll
        for (int s = 0; s < KS; ++s) af[s] = hrow[(size_t)(rt * KS + s) * 64];
    };

    int passes = 0, rt0 = rt_begin;
    // a row tile is asked for AHEAD tiles before its turn, into the registers of the tile just read (past the last
    // whole pass the last tile is asked for again)
    constexpr int AHEAD = KS >= 2 ? 2 : SMT_GROUP;              // what keeps 64-bit signatures at three waves a SIMD (2 % faster than four ahead at two)
    static_assert(SMT_GROUP % AHEAD == 0, "a tile's registers are the same in every pass");
    v4i rows[AHEAD][KS];
    const int rt_last = rt_begin + (rt_end - rt_begin) / SMT_GROUP * SMT_GROUP - 1;      // of the whole passes
    if (rt0 + SMT_GROUP <= rt_end)
#pragma unroll
        for (int u = 0; u < AHEAD; ++u) load_rows(rt0 + u, rows[u]);
    // one row tile's words into the ones, twos, fours of column tile ct; the carry has weight 8
    auto add_tile = [&](const v4i(&af)[KS], int ct) __attribute__((always_inline)) {
        uint32_t w[8], c[4], d[2], up;
        tile_words(af, ct, w);
#pragma unroll
        for (int q = 0; q < 4; ++q) csa(ones[ct], c[q], ones[ct], w[2 * q], w[2 * q + 1]);
        csa(twos[ct], d[0], twos[ct], c[0], c[1]);
        csa(twos[ct], d[1], twos[ct], c[2], c[3]);
        csa(fours[ct], up, fours[ct], d[0], d[1]);
        return up;
    };
    // The same with the matrix cores at work on the next (row tile, column tile), one product per share of this one's counting:
    // left to itself the compiler issues a chain of four products in one go and waits it out (8 x 10^4 candidates, 10^5 items
    // of 128 bits: 541 -> 510 us for the kernel, 605 -> 587 a call).  Not for shorter signatures: their chains are one or two
    // products, covered by a third wave a SIMD, for which a second set of cells would leave no room.
    constexpr bool BESIDE = KS == 4;
    v16f cells = start;
    if constexpr (BESIDE)
        if (rt0 + SMT_GROUP <= rt_end)
#pragma unroll
            for (int s = 0; s < KS; ++s) cells = mfma_step(cells, rows[0][s], bf[0][s]);
    auto add_beside = [&](const v4i(&next)[KS], int next_ct, int ct) __attribute__((always_inline)) {
        v16f acc = start;
        uint32_t c[4], d[2], up;
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            __builtin_amdgcn_sched_barrier(0);
            acc = mfma_step(acc, next[s % KS], bf[next_ct][s % KS]);
            csa(ones[ct], c[s], ones[ct], word(cells, 2 * s), word(cells, 2 * s + 1));
            if (s % 2) csa(twos[ct], d[s / 2], twos[ct], c[s - 1], c[s]);
        }
        csa(fours[ct], up, fours[ct], d[0], d[1]);
        cells = acc;
        return up;
    };
    auto ripple = [&](uint32_t up, uint32_t &p) {
        const uint32_t next = p & up;
        p ^= up;
        return next;
    };
    uint32_t wait[SMT_COLS];                                    // a pass's carry of weight 32, until the next pass brings its partner
#pragma unroll
    for (int ct = 0; ct < SMT_COLS; ++ct) wait[ct] = 0;
    for (; rt0 + SMT_GROUP <= rt_end; rt0 += SMT_GROUP) {
        uint32_t e[SMT_COLS], f[SMT_COLS];                      // carries of weight 8 and 16 waiting for their partner
#pragma unroll
        for (int u = 0; u < SMT_GROUP; ++u) {
#pragma unroll
            for (int ct = 0; ct < SMT_COLS; ++ct) {
                uint32_t eu;
                if constexpr (BESIDE) {
                    if (ct == SMT_COLS - 1) load_rows(min(rt0 + u + AHEAD, rt_last), rows[u % AHEAD]);     // its last product is under way
                    eu = add_beside(rows[(ct == SMT_COLS - 1 ? u + 1 : u) % AHEAD], (ct + 1) % SMT_COLS, ct);
                } else
                    eu = add_tile(rows[u % AHEAD], ct);
                if (u % 2 == 0)
                    e[ct] = eu;
                else {
                    uint32_t fu;
                    csa(eights[ct], fu, eights[ct], e[ct], eu);
                    if (u == 1)
                        f[ct] = fu;
                    else
                        csa(sixteens[ct], f[ct], sixteens[ct], f[ct], fu);
                }
            }
            if constexpr (!BESIDE) load_rows(min(rt0 + u + AHEAD, rt_last), rows[u % AHEAD]);
        }
        if (++passes & 1) {
#pragma unroll
            for (int ct = 0; ct < SMT_COLS; ++ct) wait[ct] = f[ct];
        } else {
#pragma unroll
            for (int ct = 0; ct < SMT_COLS; ++ct) {
                uint32_t up;
                csa(plane[ct][0], up, plane[ct][0], wait[ct], f[ct]);
#pragma unroll
                for (int j = 1; j < SMT_PLANES; ++j) up = ripple(up, plane[ct][j]);
            }
            if (passes == SMT_FLUSH) {
                read_out();
                passes = 0;
            }
        }
    }
    if (passes & 1)
#pragma unroll
        for (int ct = 0; ct < SMT_COLS; ++ct)
#pragma unroll
            for (int j = 0; j < SMT_PLANES; ++j) wait[ct] = ripple(wait[ct], plane[ct][j]);
    // the last one to three row tiles, their carries rippled from weight 8 up
    for (; rt0 < rt_end; ++rt0) {
        v4i af[KS];
        load_rows(rt0, af);
#pragma unroll
        for (int ct = 0; ct < SMT_COLS; ++ct) {
            uint32_t up = ripple(ripple(add_tile(af, ct), eights[ct]), sixteens[ct]);
#pragma unroll
            for (int j = 0; j < SMT_PLANES; ++j) up = ripple(up, plane[ct][j]);
        }
    }
    read_out();
    __syncthreads();

    const int local = first + tid;
    if (n_parts > 1) {              // raw counts; the slot exists whether or not a candidate sits in it
        int32_t *o = parts + ((size_t)part_no * b.n_blk * LSH_BLOCK + (size_t)blk * LSH_BLOCK + tid) * LSH_MAX_TIERS;
#pragma unroll
        for (int t = 0; t < LSH_MAX_TIERS; ++t) o[t] = cnt[t][tid];
        return;
    }
    if (local >= rd.n_cand) return;
    int32_t n[LSH_MAX_TIERS];
#pragma unroll
    for (int t = 0; t < LSH_MAX_TIERS; ++t) n[t] = cnt[t][tid];
    simtier_store(m, rd, local, sh, n);
}

template <int KS>
__global__ __launch_bounds__(256, KS <= 2 ? 3 : 2) void k_lsh_simtier_mfma(LshModel m, LshBatch b, const uint8_t *__restrict__ sig_table,
                                                                         const v4i *__restrict__ hist, size_t req_stride, int sh,
                                                                         int32_t *__restrict__ parts)
{
    lsh_simtier_block<KS>(m, b, sig_table, hist, req_stride, sh, parts, blockIdx.x, blockIdx.y, gridDim.y);
}

// The same beside the blocks that cut D into pieces (they come first: the shorter ones).
template <int KS>
__global__ __launch_bounds__(256, KS <= 2 ? 3 : 2) void k_lsh_count(LshModel m, LshBatch b, const uint8_t *__restrict__ sig_table, const v4i *__restrict__ hist,
                                                                  size_t req_stride, int sh, int32_t *__restrict__ parts, int n_parts, LshPiecesArgs p)
{
    const int n_pieces = p.per_req * b.n_req;
    int idx = blockIdx.x;
    if (idx < n_pieces) {
        const int r = idx / p.per_req;
        lsh_pieces_block<256>(m, b.reqs[r], r, idx - r * p.per_req, p.part_stride, p.part, p.A, (uint4 *)p.pieces, p.stride);
        return;
    }
    idx -= n_pieces;
    lsh_simtier_block<KS>(m, b, sig_table, hist, req_stride, sh, parts, idx % b.n_blk, idx / b.n_blk, n_parts);
}

template <int KS>
__global__ __launch_bounds__(256) void k_lsh_expand(LshBatch b, v4i *__restrict__ out, size_t req_stride)
{
    lsh_expand_block<KS, 1>(b.reqs[blockIdx.y], blockIdx.y, blockIdx.x, out, req_stride);
}

__global__ __launch_bounds__(256) void k_lsh_simtier_finish(LshModel m, LshBatch b, int sh, const int32_t *__restrict__ parts, int n_parts)
{
    lsh_finish_block(m, b, sh, parts, n_parts, blockIdx.x);
}

static int simtier_shift(const LshModel &m)                     // 2 d' / N = 2^shift, or -1
{
    int sh = 0;
    while (sh < 9 && (1 << sh) * m.n_tiers < 2 * m.d_bits) ++sh;
    return (1 << sh) * m.n_tiers == 2 * m.d_bits ? sh : -1;
}

// Parts a history is cut into: enough blocks to fill the chip a few times over, each with at least two passes of the adder network per wave
static int simtier_parts(int n_blk, int nrt)
{
    const int n = std::min(SMT_PART_BLOCKS / n_blk, nrt / (4 * SMT_GROUP));
    return std::max(1, std::min(n, SMT_MAX_PARTS));
}

bool lsh_simtier_on_mfma(const LshModel &m)
{
    static_assert(LSH_MAX_TIERS == 8, "eight one-hot bits a byte, eight counts a slot");
    const int sh = simtier_shift(m);
    // the first item's scale is 2^(8 - shift), an integer
    return (m.d_bits == 32 || m.d_bits == 64 || m.d_bits == 128) && sh >= 0 && sh <= 8;
}

size_t lsh_hist_stride(const LshModel &m, int max_seq_len)      // 16-byte pieces per request
{
    return (size_t)((max_seq_len + SMT_TILE - 1) / SMT_TILE) * (m.d_bits / 32) * 64;
}

size_t lsh_simtier_parts_bytes() { return (size_t)(SMT_PART_BLOCKS + SMT_MAX_PARTS) * LSH_BLOCK * LSH_MAX_TIERS * 4; }

hipError_t launch_lsh_simtier_mfma(const LshModel &m, const LshBatch &b, const uint8_t *sig_table, void *hist, size_t req_stride,
                                   int longest, void *parts, hipStream_t s)
{
    if (b.n_blk == 0) return hipSuccess;
    if (!lsh_simtier_on_mfma(m) || !hist || !parts) return hipErrorInvalidValue;
    const int sh = simtier_shift(m);
    const int ks = m.d_bits / 32;
    const int nrt = (longest + SMT_TILE - 1) / SMT_TILE, pieces = nrt * ks * 64;
    if (pieces > 0) {
        const dim3 grid((pieces + 255) / 256, b.n_req);
        switch (ks) {
        case 1: hipLaunchKernelGGL(k_lsh_expand<1>, grid, dim3(256), 0, s, b, (v4i *)hist, req_stride); break;
        case 2: hipLaunchKernelGGL(k_lsh_expand<2>, grid, dim3(256), 0, s, b, (v4i *)hist, req_stride); break;
        default: hipLaunchKernelGGL(k_lsh_expand<4>, grid, dim3(256), 0, s, b, (v4i *)hist, req_stride); break;
        }
    }
    const int n_parts = simtier_parts(b.n_blk, nrt);
    const dim3 grid(b.n_blk, n_parts);
    int32_t *pp = (int32_t *)parts;
    switch (ks) {
    case 1: hipLaunchKernelGGL(k_lsh_simtier_mfma<1>, grid, dim3(256), 0, s, m, b, sig_table, (const v4i *)hist, req_stride, sh, pp); break;
    case 2: hipLaunchKernelGGL(k_lsh_simtier_mfma<2>, grid, dim3(256), 0, s, m, b, sig_table, (const v4i *)hist, req_stride, sh, pp); break;
    default: hipLaunchKernelGGL(k_lsh_simtier_mfma<4>, grid, dim3(256), 0, s, m, b, sig_table, (const v4i *)hist, req_stride, sh, pp); break;
    }
    if (n_parts > 1) hipLaunchKernelGGL(k_lsh_simtier_finish, dim3(b.n_blk), dim3(256), 0, s, m, b, sh, (const int32_t *)pp, n_parts);
    return hipGetLastError();
}

// A small call's finish costs no launch: parts of one pass a wave, up to two blocks a compute unit (1 x 3,000 candidates x 3,000 items
// 32.2 -> 29.3 us, 3 x 1,495 x 1,330 of 128 bits 43.0 -> 38.6; of half a pass 29.1 and 37.6, but 8 x 1,000 x 2,000 50.0 -> 52.4)
int lsh_small_parts(int n_blk, int longest)
{
    const int nrt = (longest + SMT_TILE - 1) / SMT_TILE;
    const int n = std::min(SMT_PART_BLOCKS / 4 / n_blk, nrt / (2 * SMT_GROUP));
    return std::max(simtier_parts(n_blk, nrt), std::min(n, SMT_MAX_PARTS));
}

hipError_t launch_lsh_count(const LshModel &m, const LshBatch &b, const uint8_t *sig_table, const void *hist, size_t req_stride, void *parts,
                            int n_parts, const LshPiecesArgs &p, hipStream_t s)
{
    if (!lsh_simtier_on_mfma(m) || !hist || !parts || !p.pieces) return hipErrorInvalidValue;
    const int sh = simtier_shift(m);
    const dim3 grid(p.per_req * b.n_req + b.n_blk * n_parts);
    auto go = [&](auto kern) {
        hipLaunchKernelGGL(kern, grid, dim3(256), 0, s, m, b, sig_table, (const v4i *)hist, req_stride, sh, (int32_t *)parts, n_parts, p);
    };
    switch (m.d_bits / 32) {
    case 1: go(k_lsh_count<1>); break;
    case 2: go(k_lsh_count<2>); break;
    default: go(k_lsh_count<4>); break;
    }
    return hipGetLastError();
}

int lsh_simtier_shift(const LshModel &m) { return simtier_shift(m); }

}  // namespace aif
