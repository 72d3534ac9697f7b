// Internal device-side types and launcher prototypes of the LSH path of libaif (gfx950 only).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace aif {

constexpr int LSH_BLOCK = 256;          // candidates per scheduling block
constexpr int LSH_TCHUNK = 1024;        // history items whose user-side sums one block forms (more for a long history)
constexpr int LSH_MAX_CHUNKS = 64;      // chunks of one history at most
// Chunk length of a history of L items, a multiple of 64: LSH_TCHUNK, or an even share of a history that would have more than
// LSH_MAX_CHUNKS chunks -- every chunk's partial sums ((d' + 2) d floats) are written to memory and read back, and a block walks its
// chunk in a chain of loads.  fine, contexts of at most LSH_FEW users: a tenth of the history instead, no shorter than LSH_TCHUNK_MIN, because
// there the chain is what a call waits for; with more users the blocks are enough and each one's start counts.  us a call, 1,024 | fine:
// 1 user x 1,000 candidates x 1,000 items 31.8 | 22.0, 8 x 1,000 x 2,000 (128 bits, fp32) 73.2 | 49.1, 16 x 2,000 x 1,000 48.5 | 40.0,
// 16 x 10^4 x 3,000 94.7 | 95.0; 24 x 10^4 x 3,000 112.3 | 115.8, 64 x 10^4 x 1,000 131.0 | 141.9, 200 x 4,000 x 1,000 163 | 188, 1,000 x 1,000 x 400 213 | 272.
// A function of the request's history, the model and the context's size alone, like everything that decides the order of its sums.
constexpr int LSH_FEW = 16, LSH_TCHUNK_MIN = 128, LSH_FEW_CHUNKS = 10;
__host__ __device__ inline int lsh_chunk_len(bool fine, int L)
{
    if (L > LSH_TCHUNK * LSH_MAX_CHUNKS) return ((L - 1) / LSH_MAX_CHUNKS + 64) / 64 * 64;
    const int share = ((L + LSH_FEW_CHUNKS - 1) / LSH_FEW_CHUNKS + 63) / 64 * 64;
    return !fine || share > LSH_TCHUNK ? LSH_TCHUNK : share < LSH_TCHUNK_MIN ? LSH_TCHUNK_MIN : share;
}
__host__ __device__ inline int lsh_chunks(bool fine, int L)
{
    const int len = lsh_chunk_len(fine, L);
    return (L + len - 1) / len;
}
// the most chunks a history of at most L items has
inline int lsh_most_chunks(bool fine, int L)
{
    const int shortest = (L + LSH_TCHUNK_MIN - 1) / LSH_TCHUNK_MIN, coarse = (L + LSH_TCHUNK - 1) / LSH_TCHUNK;
    const int few = !fine ? 0 : shortest < LSH_FEW_CHUNKS ? shortest : LSH_FEW_CHUNKS, most = few > coarse ? few : coarse;
    return most < LSH_MAX_CHUNKS ? most : LSH_MAX_CHUNKS;
}
constexpr int LSH_MAX_TIERS = 8;
// How many ways a block of k_lsh_user_sums shares out its chunk's items: its four waves take a row tile of 32 bits each,
// and signatures of 32 (64) bits have one (two).  Every share leaves partial sums of its own.
__host__ __device__ inline int lsh_user_split(int d_bits) { return d_bits == 32 ? 4 : d_bits == 64 ? 2 : 1; }
// Rows of d floats in a request's user-side sums: D's d', then total and `lowest` as hi + lo each, then the majority word
// (d' bits, in a row of their own).  An error in D[k] reaches a candidate divided by 2 d' and mixed with the others'; one
// in total or lowest reaches it whole, so these two are summed in 64 bits.
__host__ __device__ inline int lsh_rows(int d_bits) { return d_bits + 5; }
constexpr int LSH_TOTAL = 0, LSH_LOWEST = 2, LSH_MAJORITY = 4;      // rows past D's
// A candidate that has the history's majority bit in fewer than 5/16 of its places is served from `lowest` instead of
// total / 2 (k_lsh_user_mfma.hip).
__device__ __forceinline__ bool lsh_dissimilar(int n_majority_bits, int d_bits) { return 16 * n_majority_bits < 5 * d_bits; }
// the n partial sums at p, p + stride, .. added in order, eight loads in flight
__device__ __forceinline__ float lsh_sum_parts(const float *p, size_t stride, int n)
{
    float acc = 0.f;
    int c = 0;
    for (; c + 8 <= n; c += 8) {
        float v[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] = p[(size_t)(c + i) * stride];
#pragma unroll
        for (int i = 0; i < 8; ++i) acc += v[i];
    }
    for (; c < n; ++c) acc += p[(size_t)c * stride];
    return acc;
}
// two such sums at a time: sixteen loads in flight
__device__ __forceinline__ void lsh_sum_parts2(const float *p, const float *q, size_t stride, int n, float &a, float &b)
{
    a = b = 0.f;
    int c = 0;
    for (; c + 8 <= n; c += 8) {
        float v[8], w[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] = p[(size_t)(c + i) * stride];
#pragma unroll
        for (int i = 0; i < 8; ++i) w[i] = q[(size_t)(c + i) * stride];
#pragma unroll
        for (int i = 0; i < 8; ++i) a += v[i];
#pragma unroll
        for (int i = 0; i < 8; ++i) b += w[i];
    }
    for (; c < n; ++c) {
        a += p[(size_t)c * stride];
        b += q[(size_t)c * stride];
    }
}
// the same for a sum of 64 bits: each partial is p[0] + p[d]
__device__ __forceinline__ double lsh_sum_totals(const float *p, size_t stride, int d, int n)
{
    double acc = 0.0;
    int c = 0;
    for (; c + 4 <= n; c += 4) {
        float hi[4], lo[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            hi[i] = p[(size_t)(c + i) * stride];
            lo[i] = p[(size_t)(c + i) * stride + d];
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) acc += (double)hi[i] + (double)lo[i];
    }
    for (; c < n; ++c) acc += (double)p[(size_t)c * stride] + (double)p[(size_t)c * stride + d];
    return acc;
}

struct LshReqDesc {
    const uint8_t *seq_sigs;
    const void *seq_emb;
    const int32_t *cand_ids;
    float *din_out;
    int32_t *tier_out;
    int32_t seq_len;
    int32_t n_cand;
    int32_t cand_base;          // first candidate slot of this request in the batch (multiple of LSH_BLOCK)
    int32_t index;
};

struct LshBatch {
    const LshReqDesc *reqs;     // device, [n_req]
    const int32_t *blk_req;     // device, [n_blk]: request owning each block of LSH_BLOCK candidate slots
    int32_t n_req;
    int32_t n_blk;
};

// Descriptors of a batch of at most LSH_FEW requests in a kernel's arguments: its blocks read them there and the first of them write
// the batch's device tables, which the later kernels read.
struct LshFew {
    LshReqDesc rd[LSH_FEW];
    LshReqDesc *reqs;
    int32_t *blk_req;
    int32_t n_req, n_blk;
};

struct LshModel {
    int64_t n_items;
    int32_t d_bits, d_out, n_tiers;
    int32_t dtype;              // storage of U~: 0 fp32, 1 bf16
    int32_t fine;               // lsh_chunk_len
    int32_t tier_mul;           // ceil(2^20 / d_bits): (x * tier_mul) >> 20 == x / d_bits for x <= 2048
};

// a2 of this path (k_lsh_user_mfma.hip) -- per request and share of its history, lsh_rows(d') rows of d floats:
// part[r][share][k] = sum of c_tk U~_t (c = 1 where bit k of signature t is 0, else -1), then the sum of U~_t, the sum of w_t U~_t
// (w_t: places where signature t differs from the majority word; hi, lo each), and the majority word (share 0's alone)
// (grid_chunks: chunks of the longest history in the batch; part_stride: shares a request has room for)
hipError_t launch_lsh_user_sums(const LshModel &m, const LshBatch &b, int grid_chunks, int part_stride, float *part, hipStream_t s);
// A[r] = the shares of request r added up, in a fixed order: D [d'][d], total / 2 (hi, lo) [2][d], lowest = the weighted sum / d'
// (hi, lo) [2][d], the majority word
hipError_t launch_lsh_user_reduce(const LshModel &m, const LshBatch &b, int part_stride, const float *part, float *A, hipStream_t s);
// Eq. 8: din[i] = total / 2 + (1 / 2 d') sum_k c_ik D[k], or the same from `lowest`
hipError_t launch_lsh_din(const LshModel &m, const LshBatch &b, const uint8_t *sig_table, const float *A, int32_t *bad,
                          hipStream_t s);
// Eq. 8 on the matrix cores (d a multiple of 32 up to 128): the candidates' signs against D cut into three bf16 pieces.
// launch_lsh_din_pieces takes launch_lsh_user_reduce's place: it adds the shares up itself and leaves D as pieces
// (lsh_din_pieces_stride() 16-byte pieces per request) and the rest in A's last rows.
bool lsh_din_on_mfma(const LshModel &m);
size_t lsh_din_pieces_stride(const LshModel &m);
hipError_t launch_lsh_din_pieces(const LshModel &m, const LshBatch &b, int part_stride, const float *part, float *A, void *pieces, hipStream_t s);
hipError_t launch_lsh_din_mfma(const LshModel &m, const LshBatch &b, const uint8_t *sig_table, const float *A, const void *pieces,
                               int32_t *bad, hipStream_t s);
// Eq. 6, 7, 9: equal-bit counts against every history item, counted into tiers
hipError_t launch_lsh_simtier(const LshModel &m, const LshBatch &b, const uint8_t *sig_table, hipStream_t s);
// The same with the equal-bit counts formed on the matrix cores (signatures of 32, 64 or 128 bits; 2 d' / N a power of
// two up to 256).  hist: workspace of lsh_hist_stride() 16-byte pieces per request, written by the launch itself (the
// history signatures as the matrix instruction's operand); longest: the longest history of the batch; parts: workspace
// of lsh_simtier_parts_bytes() for the partial counts of a batch too small to fill the chip uncut.
bool lsh_simtier_on_mfma(const LshModel &m);
size_t lsh_hist_stride(const LshModel &m, int max_seq_len);
size_t lsh_simtier_parts_bytes();
hipError_t launch_lsh_simtier_mfma(const LshModel &m, const LshBatch &b, const uint8_t *sig_table, void *hist, size_t req_stride,
                                   int longest, void *parts, hipStream_t s);

// A small call in three launches instead of seven (SimTier and LSH-DIN both on the matrix cores): what the user's side needs
// (sums, the history expanded, the tables of a batch of few requests); SimTier beside D's pieces; LSH-DIN beside SimTier's finish.
// few: null, or the descriptors (nothing has been uploaded then).  n_parts: lsh_small_parts() for both launches that take it.
struct LshPiecesArgs {
    const float *part;
    float *A;
    void *pieces;
    size_t stride;              // lsh_din_pieces_stride()
    int32_t part_stride, per_req;       // per_req: lsh_pieces_blocks()
};
// Whether a call is small: its last launch takes a wave to a tile of 32 candidates and one of 32 features, and from 1,024 blocks of 256
// candidates x 32 features on (2,560 where the descriptors travel in the arguments) that costs more than the launches.  us a call, seven
// launches | three: 128 users x 1,000 candidates x 300 items (64 bits: 1,024) 66.8 | 66.6, 256 x 300 x 300 (1,024) 68.0 | 65.0,
// 128 x 100 x 300 (128 bits: 512) 74.4 | 68.1, 256 x 1,000 x 300 (32 bits: 1,024) 72.2 | 65.8; 64 x 3,000 x 500 (64 bits: 1,536) 72.8 | 73.9,
// 128 x 1,000 x 300 (128 bits: 2,048) 88.3 | 104.2, 600 x 100 x 300 (128 bits: 2,400) 153.8 | 179.4, 128 x 3,000 x 500 (6,144) 164.5 | 202.7;
// 16 x 10^4 x 500 (128 bits: 2,560) 110.2 | 96.4.
inline bool lsh_call_is_small(const LshModel &m, int n_req, int n_blk)
{
    return (int64_t)n_blk * (m.d_out / 32) <= (n_req <= LSH_FEW ? 2560 : 1024);
}
inline int lsh_pieces_blocks(const LshModel &m) { return (m.d_bits / 16 + 1) * (m.d_out / 32); }
int lsh_small_parts(int n_blk, int longest);
int lsh_simtier_shift(const LshModel &m);
hipError_t launch_lsh_stage(const LshModel &m, const LshBatch &b, const LshFew *few, int grid_chunks, int part_stride, float *part, void *hist,
                            size_t req_stride, int longest, hipStream_t s);
hipError_t launch_lsh_count(const LshModel &m, const LshBatch &b, const uint8_t *sig_table, const void *hist, size_t req_stride, void *parts,
                            int n_parts, const LshPiecesArgs &p, hipStream_t s);
hipError_t launch_lsh_result(const LshModel &m, const LshBatch &b, const uint8_t *sig_table, const float *A, const void *pieces, int32_t *bad,
                             int sh, const void *parts, int n_parts, hipStream_t s);

}  // namespace aif
