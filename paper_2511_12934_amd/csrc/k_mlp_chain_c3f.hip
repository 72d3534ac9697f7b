// The fused MLP chain (k_mlp_chain.h), shape of k_mlp_chain_c3.hip, with the Hadamard cross block folded into the user's layer-1
// weights (one set of layer-1 fragments per user slot, made by the staging launch): layer 1 contracts over [item | attention].
#include "k_mlp_chain.h"

namespace aif {

hipError_t mlp_acc_c3f(const Model &, const Batch &, const void *, const MlpPack &, const float *, hipStream_t);      // k_mlp_acc.hip

// k_mlp_acc gives every compute unit one block at a time and whole tiles of 256 candidates, so it takes as long as its fullest
// block: 18 us a round of one tile a unit, where the chain takes 20 us for as many and fills a last round in quarters.  It
// serves batches of two rounds and more that leave at most 15 % of the last one empty.  Whole calls, 10^4 candidates a user
// over 100 history items, us, chain / k_mlp_acc: 6 users (0.94 of one round) 47.3 / 48.7; 8 (0.63 of two) 58.6 / 64.7;
// 12 (0.94) 72.1 / 69.3; 16 (0.83 of three) 85.4 / 86.8; 20 (0.78 of four) 111.8 / 113.6; 26 (0.81 of five) 135.2 / 135.4;
// 32 (all of five) 144.3 / 135.6.
static bool fills_rounds(int n_blk)
{
    const int64_t cu = n_cu(), rounds = (n_blk + cu - 1) / cu;
    return rounds >= 2 && 100 * (int64_t)n_blk >= 85 * rounds * cu;
}

hipError_t mlp_chain_c3f(const Model &m, const Batch &b, const void *X, const MlpPack &pk, const float *bias1, hipStream_t s)
{
    if (m.x_tiled && fills_rounds(b.n_blk)) return mlp_acc_c3f(m, b, X, pk, bias1, s);
    return launch_spec<128, 512, 256, 0, 4, 16, 4, 2, 0, 1>(m, b, X, pk, bias1, s);
}

}  // namespace aif
