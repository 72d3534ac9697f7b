// User-side network of AIF (Sec. 3.1, Eq. 1-3), the parts around the attention:
// the projections of Eq. 1, and FFN + pooling + combined vector of Eq. 2.  The
// attentions themselves (Eq. 2's self-attention over the sequence and Eq. 3's
// profile-to-sequence attention) run on the library's target-attention kernels:
// every sequence position, and the profile, is a query over the same projected
// sequence.
//
// fp32 arithmetic over the storage type, fixed summation order per output.
#include "aif_user_dev.h"
#include "k_stage.h"

#include <algorithm>
#include <type_traits>

namespace aif {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

// Where a block of the projection finds its user: in the call's device tables, or in the launch's own arguments (their first).
struct UserTables {
    const UserDesc *users;
    const int32_t *blk_req;
    __device__ __forceinline__ int user_of(int blk) const { return blk_req[blk]; }
    __device__ __forceinline__ UserDesc desc(int u) const { return users[u]; }
};
struct UserArguments {
    int n_users;
    __device__ __forceinline__ int user_of(int blk) const      // every user has a block: the last whose first is not past this one
    {
        const int i = threadIdx.x & 63;
        const int first = kernel_arg<UserFew>(0)->ud[i < n_users ? i : 0].row_base / ROW_BLOCK;
        return __popcll(__ballot(i < n_users && first <= blk)) - 1;
    }
    __device__ __forceinline__ UserDesc desc(int u) const { return arg_copy(&kernel_arg<UserFew>(0)->ud[__builtin_amdgcn_readfirstlane(u)]); }
};
static_assert(USER_FEW <= 64, "a lane a user");

// the tables of such a call, by its first blocks of 256 threads; room: USER_FILL_ROOM in LDS (the caller's: a widest projection's rows
// leave no other)
constexpr int USER_FILL_ROOM = 2 * USER_FEW;
__device__ __forceinline__ void user_fill(const UserFew &f, int i, int *room)
{
    int *const first_blk = room, *const first_group = room + USER_FEW;
    const auto args = kernel_arg<UserFew>(0);
    if (threadIdx.x < 64) {
        const int u = threadIdx.x < f.n_users ? threadIdx.x : 0, ng = threadIdx.x < f.n_users ? args->groups_of[u] : 0;
        int sum = ng;                                           // of the users up to this one
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int before = __shfl_up(sum, o, 64);
            sum += (int)threadIdx.x >= o ? before : 0;
        }
        if ((int)threadIdx.x < f.n_users) {
            first_blk[threadIdx.x] = args->ud[u].row_base / ROW_BLOCK;
            first_group[threadIdx.x] = sum - ng;
        }
    }
    __syncthreads();
    auto last_not_past = [&](const int *first, int x) {
        int r = 0;
        for (int u = 1; u < f.n_users; ++u) r = first[u] <= x ? u : r;
        return r;
    };
    if (i < f.n_users) {
        const UserDesc ud = arg_copy(&args->ud[i]);
        f.users[i] = ud;
        ReqDesc e{};                                            // (aif_user_precompute has the same)
        e.seq_keys = e.seq_vals = ud.seq_out;
        e.seq_len = ud.seq_len;
        e.n_cand = ud.seq_len + 1;
        e.row_base = ud.row_base;
        e.index = e.slot = i;
        f.reqs[i] = e;
    }
    if (i < f.n_blk) f.blk_req[i] = last_not_past(first_blk, i);
    if (i < f.n_groups) {
        // (a user without groups has its successor's first: the last one not past i is the one that has it)
        const int r = last_not_past(first_group, i), ng = args->groups_of[r], at = i - first_group[r], tiles = (args->ud[r].seq_len + 1 + 31) / 32;
        f.groups[i] = AttnGroup{r, (int)((long)tiles * at / ng), (int)((long)tiles * (at + 1) / ng), 0};
    }
}

// The projected profile: four adjacent lanes share an output feature, each takes a quarter of the input
// features (d_raw is a multiple of four), they meet in a fixed two-step butterfly.  All of a thread's loads are
// independent, U of them on their way, so the row costs about one round trip to memory.
template <typename T, int U>
__device__ __forceinline__ void project_profile(const UserWeights &w, const UserDesc &ud, T *X, int nthreads)
{
    const T *pr = (const T *)ud.profile;
    const int d = w.d, q = threadIdx.x & 3, chunk = w.d_raw >> 2;
    for (int n0 = 0; n0 < d; n0 += nthreads >> 2) {
        const int n = n0 + (threadIdx.x >> 2);
        float acc = 0.f;
        if (n < d) {
            const float *wr = w.wprof + (size_t)n * w.d_raw + q * chunk;
            const T *px = pr + q * chunk;
#pragma unroll U
            for (int m = 0; m < chunk; ++m) acc = fmaf(wr[m], ld_f<T>(px + m), acc);
        }
        acc += __shfl_xor(acc, 1, 64);
        acc += __shfl_xor(acc, 2, 64);
        if (n < d && q == 0) st_f<T>(X + (size_t)(ud.row_base + ud.seq_len) * (2 * d) + n, acc);
    }
}

// ---------------------------------------------------------------------------
// Eq. 1 on the matrix cores (bf16): U^_seq^T = W_seq U_seq^T, positions as the
// columns of the B operand.  A wave owns 32 positions; lane (position c, half h)
// reads eight consecutive input features of its position per k-step straight
// from the caller's row-major sequence and receives sixteen output features of
// that position per 32-feature tile (features 8 q + 4 h + i), which it writes as
// four 8-byte pieces to the workspace row and to the user's seq_out.
// ---------------------------------------------------------------------------
// The rows pass through LDS, so that they leave for the workspace and seq_out in whole lines.  PACK: they are two whole
// 64-key stages of the attention that follows, and the block packs them from LDS as keys and values as well (one launch
// where two were: 64 users of up to 500 positions 11.6 us instead of 12.2 + 5.9).  The blocks past the sequences' project the profiles, one user each, beside them instead of after a
// block's own rows.
template <int D, bool PACK, class Users>
__device__ __forceinline__ void user_project_mfma_block(int blk, const UserWeights &w, const Users &src, int n_row_blk, uint16_t *__restrict__ X, const UserPack &pk)
{
    constexpr int FT = D / 32, ROWS = 128, SUB = ROW_BLOCK / ROWS;
    if (blk >= n_row_blk) {
        project_profile<uint16_t, 32>(w, src.desc(blk - n_row_blk), X, 256);
        return;
    }
    const int u = src.user_of(blk / SUB);
    if (u < 0) return;
    const UserDesc ud = src.desc(u);
    const int row0 = blk * ROWS, local0 = row0 - ud.row_base, L = ud.seq_len;
    constexpr int LD = D + 8;                                   // LDS row: 16 bytes of padding
    __shared__ __align__(16) uint16_t rows[ROWS * LD];
    if (local0 >= L) return;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, col = lane & 31, h = lane >> 5;
    const int li = local0 + wave * 32 + col;
    const int KS = w.d_raw / 16;
    if (local0 + wave * 32 < L) {                               // wave-uniform: some position of this wave exists
        const uint16_t *src = (const uint16_t *)ud.seq + (size_t)(li < L ? li : 0) * w.d_raw + 8 * h;
        const bf16x8 *wf = (const bf16x8 *)w.wseq_frag + lane;
        f32x16 acc[FT];
#pragma unroll
        for (int ft = 0; ft < FT; ++ft)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[ft][i] = 0.f;
        // all of a group's input pieces are asked for before its first MFMA: the loads are independent, and one
        // round trip to memory per group instead of one per k-step is what this short kernel's time is made of
        constexpr int G = 8;
        for (int k0 = 0; k0 < KS; k0 += G) {
            // (and all of its weights: a k-step past the last reads the last again and multiplies it by zeros, so that no
            // load hangs on a condition)
            bf16x8 b[G], a[G][FT];
#pragma unroll
            for (int j = 0; j < G; ++j) {
                const int k = min(k0 + j, KS - 1);
                b[j] = *(const bf16x8 *)(src + 16 * k);
#pragma unroll
                for (int ft = 0; ft < FT; ++ft) a[j][ft] = wf[(size_t)(ft * KS + k) * 64];
            }
#pragma unroll
            for (int j = 0; j < G; ++j) {
                if (k0 + j >= KS)
#pragma unroll
                    for (int ft = 0; ft < FT; ++ft) a[j][ft] = b[j] = bf16x8{};
#pragma unroll
                for (int ft = 0; ft < FT; ++ft) acc[ft] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[j][ft], b[j], acc[ft], 0, 0, 0);
            }
        }
        uint16_t *dst = rows + (wave * 32 + col) * LD;
#pragma unroll
        for (int ft = 0; ft < FT; ++ft)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                bf16x4 o4;
#pragma unroll
                for (int i = 0; i < 4; ++i) o4[i] = (__bf16)acc[ft][4 * q + i];
                *(bf16x4 *)(dst + 32 * ft + 8 * q + 4 * h) = o4;
            }
    }
    __syncthreads();
    {
        constexpr int PR = D / 8;                               // 16-byte pieces of a row
        uint16_t *so = (uint16_t *)ud.seq_out + (size_t)local0 * D, *xr = X + (size_t)row0 * (2 * D);
#pragma unroll
        for (int it = 0; it < ROWS * PR / 256; ++it) {
            const int i = it * 256 + (int)threadIdx.x, row = i / PR, pc = i - row * PR;
            const uint4 v = *(const uint4 *)(rows + row * LD + 8 * pc);
            if (local0 + row < L) {
                *(uint4 *)(xr + (size_t)row * (2 * D) + 8 * pc) = v;
                *(uint4 *)(so + (size_t)row * D + 8 * pc) = v;
            }
        }
    }
    if constexpr (PACK) {
        auto key = [&](int t) { return rows + (t - local0) * LD; };
#pragma unroll
        for (int s = 0; s < ROWS / 64; ++s) pack_kv_stage<D>(u, 0, local0 / 64 + s, L, 1, key, key, pk.kvpack, pk.stride, pk.kmax, pk.nktp);
    }
}

template <int D, bool PACK>
__global__ __launch_bounds__(256) void k_user_project_mfma(UserWeights w, const UserDesc *__restrict__ users,
                                                           const int32_t *__restrict__ blk_req, int n_row_blk, uint16_t *__restrict__ X, UserPack pk)
{
    user_project_mfma_block<D, PACK>(blockIdx.x, w, UserTables{users, blk_req}, n_row_blk, X, pk);
}
// An upload of 2 - 3 us and its wait saved: 64 users of up to 500 positions 39.0 us a call -> 34.2, 6 of 60 positions 21.4 -> 15.7.
template <int D, bool PACK>
__global__ __launch_bounds__(256) void k_user_project_mfma_few(UserFew few /* first: kernel_arg */, UserWeights w, int n_row_blk, uint16_t *__restrict__ X, UserPack pk)
{
    if ((int)blockIdx.x < few.n_fill) {
        __shared__ int room[USER_FILL_ROOM];
        user_fill(few, blockIdx.x * 256 + threadIdx.x, room);
        return;
    }
    user_project_mfma_block<D, PACK>((int)blockIdx.x - few.n_fill, w, UserArguments{few.n_users}, n_row_blk, X, pk);
}

// ---------------------------------------------------------------------------
// FFN of Eq. 2 on the matrix cores (bf16) and the pooling share of 32 positions:
// Y^T = W_ffn A^T with the accumulators preloaded with the bias, ReLU, positions
// past the end zeroed, then the sum over the wave's 32 positions (the lanes of a
// half) by a fixed butterfly.
// ---------------------------------------------------------------------------
// y summed over the 32 lanes of a half: the butterfly xor 1, 2, 4, 8 on the vector ALU's own lane permutes (within four equal
// lanes a mirror is as good as an xor), 16 through the LDS crossbar
template <int CTRL> __device__ __forceinline__ float add_dpp(float y)
{
    return y + __uint_as_float((uint32_t)__builtin_amdgcn_update_dpp(0, (int)__float_as_uint(y), CTRL, 0xF, 0xF, true));
}
__device__ __forceinline__ float half_sum(float y)
{
    y = add_dpp<0xB1>(y);       // quad_perm 1,0,3,2
    y = add_dpp<0x4E>(y);       // quad_perm 2,3,0,1
    y = add_dpp<0x141>(y);      // row_half_mirror
    y = add_dpp<0x140>(y);      // row_mirror
    return y + __shfl_xor(y, 16, 64);
}

// The tile of 32 positions whose first workspace row is row0 (position local0 of L): dst[D] = the sum of its FFN outputs.
template <int D>
__device__ __forceinline__ void ffn_tile(const UserWeights &w, const uint16_t *__restrict__ X, int row0, int local0, int L, float *dst0)
{
    constexpr int FT = D / 32, KS = D / 16;
    const int lane = threadIdx.x & 63, col = lane & 31, h = lane >> 5;
    const uint16_t *src = X + (size_t)(row0 + col) * (2 * D) + D + 8 * h;      // rows past L are inside the workspace
    const bf16x8 *wf = (const bf16x8 *)w.wffn_frag + lane;
    bf16x8 b[KS];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) b[ks] = *(const bf16x8 *)(src + 16 * ks);
    const bool live = local0 + col < L;
#pragma unroll
    for (int ft = 0; ft < FT; ++ft) {
        f32x16 acc;
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int i = 0; i < 4; ++i) acc[4 * q + i] = w.b_ffn ? w.b_ffn[32 * ft + 8 * q + 4 * h + i] : 0.f;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[(size_t)(ft * KS + ks) * 64], b[ks], acc, 0, 0, 0);
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[v] = half_sum(live ? fmaxf(acc[v], 0.f) : 0.f);
        if (col == 0) {
            float *dst = dst0 + 32 * ft + 4 * h;
#pragma unroll
            for (int q = 0; q < 4; ++q) *(float4 *)(dst + 8 * q) = make_float4(acc[4 * q], acc[4 * q + 1], acc[4 * q + 2], acc[4 * q + 3]);
        }
    }
}

// a tile per wave, its sums to memory for k_user_combine: users of long sequences
template <int D>
__global__ __launch_bounds__(256) void k_user_ffn_mfma(UserWeights w, const UserDesc *__restrict__ users,
                                                       const int32_t *__restrict__ blk_req, const uint16_t *__restrict__ X,
                                                       float *__restrict__ part)
{
    constexpr int ROWS = 128, SUB = ROW_BLOCK / ROWS;
    const int u = blk_req[blockIdx.x / SUB];
    if (u < 0) return;
    const UserDesc ud = users[u];
    const int row0 = blockIdx.x * ROWS + (threadIdx.x >> 6) * 32, local0 = row0 - ud.row_base;
    if (local0 >= ud.seq_len) return;
    ffn_tile<D>(w, X, row0, local0, ud.seq_len, part + (size_t)(row0 / 32) * D);
}

// FFN, pooling and the combined vector of one user by one block of sixteen waves: the tiles' sums meet in LDS and are added
// in the order k_user_combine adds them (the same bits).  One launch where two were, and no trip of the sums through
// memory: 64 users of up to 500 positions 8 us instead of 6 + 8.  A user's tiles share one compute unit, which the launch
// saved outweighs up to USER_POOL_TILES tiles: one user of 512, 1,024 and 2,048 positions, d = 64, 32.8, 30.4 and 40.8 us a
// call against 34.4, 33.9 and 43.0 with two launches, d = 32 25.3, 34.1 and 26.5 against 30.8, 42.3 and 41.0; 64 users of
// 2,048, d = 64, 189 against 195.  Not for d = 128, where the 128 registers that sixteen waves leave a lane do not hold
// a tile's fragments (308 bytes spilled): 96, 157 and 279 against 80, 130 and 232, 64 users of 500 95 against 80.
template <int D>
__global__ __launch_bounds__(1024) void k_user_ffn_pool(UserWeights w, const UserDesc *__restrict__ users, const uint16_t *__restrict__ X)
{
    __shared__ float sums[USER_POOL_TILES][D];
    const UserDesc ud = users[blockIdx.x];
    const int L = ud.seq_len, nt = (L + 31) / 32;
    for (int t = threadIdx.x >> 6; t < nt; t += 16) ffn_tile<D>(w, X, ud.row_base + 32 * t, 32 * t, L, sums[t]);
    __syncthreads();
    const int n = threadIdx.x;
    if (n >= D) return;
    float sum = 0.f;
    for (int t = 0; t < nt; ++t) sum += sums[t][n];
    uint16_t *out = (uint16_t *)ud.user_vec_out;
    out[n] = f2bf(L > 0 ? sum / (float)L : 0.f);
    out[D + n] = X[(size_t)(ud.row_base + L) * (2 * D) + D + n];               // Eq. 3: the profile row's attention
}

// The two kernels of fp32 arithmetic below are chains of loads: rows into LDS and weights sixteen at a time.  32 weights at a time are
// more rows of them than a compute unit's L1 holds for four waves and several blocks.  us a call, one | 32 | 16 at a time, 1 user of
// 20 positions, 256 -> 128, fp32: 87 | 77 | 58, 200 of 60: 226 | 266 to 286 | 162, 65 of 250: 169 | 163 | 119; 1,000 of 30, 40 -> 72, bf16:
// 220 | 252 | 195.  (Rows of few features: no more passes than they have; 200 of 60, 12 -> 8: 28.9 | 28.9, with sixteen whatever the width 38.4.)
// A feature's rows lie in quads at 4 (quad ^ feature mod RT / 4): neighbouring lanes hold neighbouring features, and rows at one place would
// share a bank, all 64 of them.
template <int RT> __device__ __forceinline__ int user_row_at(int m, int r) { return m * RT + (r ^ 4 * (m & (RT / 4 - 1))); }
template <int RT, int U, class Get> __device__ __forceinline__ void user_stage_in(float *xs, int width, int &pass, int n, const Get &get)
{
    for (; pass + U <= n; pass += U) {
        float v[U];
#pragma unroll
        for (int q = 0; q < U; ++q) {
            const int idx = min(threadIdx.x + 256 * (pass + q), RT * width - 1), r = idx / width;
            v[q] = get(r, idx - r * width);
        }
#pragma unroll
        for (int q = 0; q < U; ++q) {
            const int idx = min(threadIdx.x + 256 * (pass + q), RT * width - 1), r = idx / width;
            xs[user_row_at<RT>(idx - r * width, r)] = v[q];              // (past the end: the last one again)
        }
    }
}
template <int RT, class Get> __device__ __forceinline__ void user_stage_rows(float *xs, int width, const Get &get)
{
    const int n = (RT * width + 255) / 256;
    int pass = 0;
    user_stage_in<RT, 16>(xs, width, pass, n, get);
    user_stage_in<RT, 4>(xs, width, pass, n, get);
    user_stage_in<RT, 1>(xs, width, pass, n, get);
}
template <int U, class Weight, class Use> __device__ __forceinline__ void user_walk_in(int &m, int n, const Weight &weight, const Use &use)
{
    for (; m + U <= n; m += U) {
        float wv[U];
#pragma unroll
        for (int q = 0; q < U; ++q) wv[q] = weight(m + q);
#pragma unroll
        for (int q = 0; q < U; ++q) use(m + q, wv[q]);
    }
}
template <class Weight, class Use> __device__ __forceinline__ void user_walk(int n, const Weight &weight, const Use &use)      // use(m, weight(m)) in order
{
    int m = 0;
    user_walk_in<16>(m, n, weight, use);
    user_walk_in<4>(m, n, weight, use);
    for (; m < n; ++m) use(m, weight(m));
}

// ---------------------------------------------------------------------------
// Eq. 1.  One block = USER_PROJ_ROWS rows of one user.  The rows are staged in
// LDS transposed (xs[m][row]) so that a thread reads the eight rows it owns for
// one input feature with two 16-byte reads; thread (column lane, row group) walks
// the transposed weights, one coalesced load per input feature reused for its
// eight rows.
// ---------------------------------------------------------------------------
template <typename T, class Users>
__device__ __forceinline__ void user_project_block(int blk, const UserWeights &w, const Users &src, int n_row_blk, T *__restrict__ X, float *xs)
{
    constexpr int RT = USER_PROJ_ROWS, SUB = ROW_BLOCK / RT;
    if (blk >= n_row_blk) {                                     // the profiles, a block each
        project_profile<T, 16>(w, src.desc(blk - n_row_blk), X, 256);
        return;
    }
    const int u = src.user_of(blk / SUB);
    if (u < 0) return;
    const UserDesc ud = src.desc(u);
    const int row0 = blk * RT;
    const int local0 = row0 - ud.row_base;
    const int L = ud.seq_len;
    if (local0 >= L) return;
    const int d_raw = w.d_raw, d = w.d;
    const T *seq = (const T *)ud.seq;
    user_stage_rows<RT>(xs, d_raw, [&](int r, int m) { return local0 + r < L ? ld_f<T>(seq + (size_t)(local0 + r) * d_raw + m) : 0.f; });
    __syncthreads();
    const int nl = threadIdx.x & 63, g = threadIdx.x >> 6;      // 4 row groups of 8
    T *so = (T *)ud.seq_out;
    for (int n = nl; n < d; n += 64) {
        float acc[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) acc[i] = 0.f;
        user_walk(d_raw, [&](int m) { return w.wseq_t[(size_t)m * d + n]; }, [&](int m, float wv) {
            const float4 a = *(const float4 *)(xs + user_row_at<RT>(m, g * 8)), b = *(const float4 *)(xs + user_row_at<RT>(m, g * 8 + 4));
            acc[0] = fmaf(wv, a.x, acc[0]);
            acc[1] = fmaf(wv, a.y, acc[1]);
            acc[2] = fmaf(wv, a.z, acc[2]);
            acc[3] = fmaf(wv, a.w, acc[3]);
            acc[4] = fmaf(wv, b.x, acc[4]);
            acc[5] = fmaf(wv, b.y, acc[5]);
            acc[6] = fmaf(wv, b.z, acc[6]);
            acc[7] = fmaf(wv, b.w, acc[7]);
        });
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int li = local0 + g * 8 + i;
            if (li < L) {
                st_f<T>(X + (size_t)(row0 + g * 8 + i) * (2 * d) + n, acc[i]);
                st_f<T>(so + (size_t)li * d + n, acc[i]);
            }
        }
    }
}
template <typename T>
__global__ __launch_bounds__(256) void k_user_project(UserWeights w, const UserDesc *__restrict__ users, const int32_t *__restrict__ blk_req, int n_row_blk, T *__restrict__ X)
{
    extern __shared__ __align__(16) float xs[];                 // [d_raw][USER_PROJ_ROWS]
    user_project_block<T>(blockIdx.x, w, UserTables{users, blk_req}, n_row_blk, X, xs);
}
template <typename T>
__global__ __launch_bounds__(256) void k_user_project_few(UserFew few /* first: kernel_arg */, UserWeights w, int n_row_blk, T *__restrict__ X)
{
    extern __shared__ __align__(16) float xs[];
    static_assert(USER_FILL_ROOM <= 4 * USER_PROJ_ROWS, "the narrowest rows are 16 bytes");
    if ((int)blockIdx.x < few.n_fill) {
        user_fill(few, blockIdx.x * 256 + threadIdx.x, (int *)xs);
        return;
    }
    user_project_block<T>((int)blockIdx.x - few.n_fill, w, UserArguments{few.n_users}, n_row_blk, X, xs);
}

size_t user_project_lds_bytes(int d_raw) { return (size_t)d_raw * USER_PROJ_ROWS * sizeof(float); }

hipError_t launch_user_project(const UserWeights &w, const UserDesc *users, const int32_t *blk_req, int n_blk, int n_users, void *X,
                               const UserPack *pack, UserFew *few, hipStream_t s)
{
    if (n_blk == 0) return hipSuccess;
    if (pack && !w.wseq_frag) return hipErrorInvalidValue;
    int n_fill = 0;
    if (few) {
        if (few->n_users != n_users || n_users > USER_FEW || few->n_blk != n_blk) return hipErrorInvalidValue;
        n_fill = few->n_fill = (std::max(std::max(n_users, n_blk), few->n_groups) + 255) / 256;
    }
    if (w.wseq_frag) {
        const int n_row_blk = n_blk * (ROW_BLOCK / 128);
        const UserPack pk = pack ? *pack : UserPack{};
        const dim3 grid(n_fill + n_row_blk + n_users);
        auto go = [&](auto d, auto packs) {
            constexpr int D = decltype(d)::value;
            constexpr bool PACK = decltype(packs)::value;
            if (few) hipLaunchKernelGGL((k_user_project_mfma_few<D, PACK>), grid, dim3(256), 0, s, *few, w, n_row_blk, (uint16_t *)X, pk);
            else hipLaunchKernelGGL((k_user_project_mfma<D, PACK>), grid, dim3(256), 0, s, w, users, blk_req, n_row_blk, (uint16_t *)X, pk);
        };
        using Yes = std::true_type;
        using No = std::false_type;
        switch (w.d) {
        case 32: pack ? go(std::integral_constant<int, 32>{}, Yes{}) : go(std::integral_constant<int, 32>{}, No{}); break;
        case 64: pack ? go(std::integral_constant<int, 64>{}, Yes{}) : go(std::integral_constant<int, 64>{}, No{}); break;
        case 128:
            if (pack) return hipErrorInvalidValue;
            go(std::integral_constant<int, 128>{}, No{});
            break;
        default: return hipErrorInvalidValue;
        }
        return hipGetLastError();
    }
    const size_t lds = user_project_lds_bytes(w.d_raw);
    const int n_row_blk = n_blk * (ROW_BLOCK / USER_PROJ_ROWS);
    const dim3 grid(n_fill + n_row_blk + n_users);
    hipError_t e = hipSuccess;
    auto go = [&](auto t) {
        using T = decltype(t);
        e = hipFuncSetAttribute(few ? (const void *)k_user_project_few<T> : (const void *)k_user_project<T>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return;
        if (few) hipLaunchKernelGGL(k_user_project_few<T>, grid, dim3(256), lds, s, *few, w, n_row_blk, (T *)X);
        else hipLaunchKernelGGL(k_user_project<T>, grid, dim3(256), lds, s, w, users, blk_req, n_row_blk, (T *)X);
    };
    if (w.dtype == 0) go(float{});
    else go(uint16_t{});
    return e != hipSuccess ? e : hipGetLastError();
}

// ---------------------------------------------------------------------------
// FFN of Eq. 2 (one layer with ReLU) on the attention outputs of USER_FFN_ROWS
// positions, summed over those positions in position order: the block's share
// of the pooling.  Same thread layout as the projection, sixteen rows a thread.
// ---------------------------------------------------------------------------
template <typename T>
__global__ __launch_bounds__(256) void k_user_ffn_partial(UserWeights w, const UserDesc *__restrict__ users,
                                                          const int32_t *__restrict__ blk_req, const T *__restrict__ X,
                                                          float *__restrict__ part)
{
    extern __shared__ __align__(16) float as[];                 // [d][USER_FFN_ROWS], then [4][d] group sums
    constexpr int RT = USER_FFN_ROWS, SUB = ROW_BLOCK / RT;
    const int u = blk_req[blockIdx.x / SUB];
    if (u < 0) return;
    const UserDesc ud = users[u];
    const int row0 = blockIdx.x * RT;
    const int local0 = row0 - ud.row_base;
    const int L = ud.seq_len;
    if (local0 >= L) return;
    const int d = w.d;
    float *gs = as + (size_t)d * RT;
    user_stage_rows<RT>(as, d, [&](int r, int m) { return local0 + r < L ? ld_f<T>(X + (size_t)(row0 + r) * (2 * d) + d + m) : 0.f; });
    __syncthreads();
    const int nl = threadIdx.x & 63, g = threadIdx.x >> 6;      // 4 row groups of 16
    for (int n = nl; n < d; n += 64) {
        float acc[16];
        const float b0 = w.b_ffn ? w.b_ffn[n] : 0.f;
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[i] = b0;
        user_walk(d, [&](int m) { return w.wffn_t[(size_t)m * d + n]; }, [&](int m, float wv) {
#pragma unroll
            for (int i4 = 0; i4 < 4; ++i4) {
                const float4 a = *(const float4 *)(as + user_row_at<RT>(m, g * 16 + 4 * i4));
                acc[4 * i4 + 0] = fmaf(wv, a.x, acc[4 * i4 + 0]);
                acc[4 * i4 + 1] = fmaf(wv, a.y, acc[4 * i4 + 1]);
                acc[4 * i4 + 2] = fmaf(wv, a.z, acc[4 * i4 + 2]);
                acc[4 * i4 + 3] = fmaf(wv, a.w, acc[4 * i4 + 3]);
            }
        });
        float sum = 0.f;
#pragma unroll
        for (int i = 0; i < 16; ++i)
            if (local0 + g * 16 + i < L) sum += fmaxf(acc[i], 0.f);
        gs[g * d + n] = sum;
    }
    __syncthreads();
    for (int n = threadIdx.x; n < d; n += 256)
        part[(size_t)blockIdx.x * d + n] = ((gs[n] + gs[d + n]) + gs[2 * d + n]) + gs[3 * d + n];
}

size_t user_ffn_lds_bytes(int d) { return (size_t)d * (USER_FFN_ROWS + 4) * sizeof(float); }

hipError_t launch_user_ffn_partial(const UserWeights &w, const UserDesc *users, const int32_t *blk_req, int n_blk,
                                   const void *X, float *part, hipStream_t s)
{
    if (n_blk == 0) return hipSuccess;
    if (w.wffn_frag) {
        const dim3 g(n_blk * (ROW_BLOCK / 128));
        switch (w.d) {
        case 32: hipLaunchKernelGGL(k_user_ffn_mfma<32>, g, dim3(256), 0, s, w, users, blk_req, (const uint16_t *)X, part); break;
        case 64: hipLaunchKernelGGL(k_user_ffn_mfma<64>, g, dim3(256), 0, s, w, users, blk_req, (const uint16_t *)X, part); break;
        case 128: hipLaunchKernelGGL(k_user_ffn_mfma<128>, g, dim3(256), 0, s, w, users, blk_req, (const uint16_t *)X, part); break;
        default: return hipErrorInvalidValue;
        }
        return hipGetLastError();
    }
    const size_t lds = user_ffn_lds_bytes(w.d);
    const dim3 grid(n_blk * (ROW_BLOCK / USER_FFN_ROWS));
    if (w.dtype == 0) {
        (void)hipFuncSetAttribute((const void *)k_user_ffn_partial<float>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        hipLaunchKernelGGL(k_user_ffn_partial<float>, grid, dim3(256), lds, s, w, users, blk_req, (const float *)X, part);
    } else {
        (void)hipFuncSetAttribute((const void *)k_user_ffn_partial<uint16_t>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        hipLaunchKernelGGL(k_user_ffn_partial<uint16_t>, grid, dim3(256), lds, s, w, users, blk_req, (const uint16_t *)X, part);
    }
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Pooling (mean) and the combined vector.  One block per user.
// ---------------------------------------------------------------------------
template <typename T>
__global__ __launch_bounds__(256) void k_user_combine(UserWeights w, const UserDesc *__restrict__ users,
                                                      const T *__restrict__ X, const float *__restrict__ part)
{
    const UserDesc ud = users[blockIdx.x];
    const int d = w.d, L = ud.seq_len;
    const int nb = (L + w.part_rows - 1) / w.part_rows;
    const size_t b0 = (size_t)ud.row_base / w.part_rows;
    T *out = (T *)ud.user_vec_out;
    for (int n = threadIdx.x; n < d; n += 256) {
        float sum = 0.f;
        for (int j = 0; j < nb; ++j) sum += part[(b0 + j) * d + n];
        st_f<T>(out + n, L > 0 ? sum / (float)L : 0.f);
        out[d + n] = X[(size_t)(ud.row_base + L) * (2 * d) + d + n];       // Eq. 3: the profile row's attention
    }
}

hipError_t launch_user_ffn_pool(const UserWeights &w, const UserDesc *users, int n_users, const void *X, hipStream_t s)
{
    if (n_users == 0) return hipSuccess;
    auto go = [&](auto kern) { hipLaunchKernelGGL(kern, dim3(n_users), dim3(1024), 0, s, w, users, (const uint16_t *)X); };
    switch (w.wffn_frag ? w.d : 0) {
    case 32: go(k_user_ffn_pool<32>); break;
    case 64: go(k_user_ffn_pool<64>); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_user_combine(const UserWeights &w, const UserDesc *users, int n_users, const void *X, const float *part,
                               hipStream_t s)
{
    if (n_users == 0) return hipSuccess;
    if (w.dtype == 0)
        hipLaunchKernelGGL(k_user_combine<float>, dim3(n_users), dim3(256), 0, s, w, users, (const float *)X, part);
    else
        hipLaunchKernelGGL(k_user_combine<uint16_t>, dim3(n_users), dim3(256), 0, s, w, users, (const uint16_t *)X, part);
    return hipGetLastError();
}

}  // namespace aif
