// The fused MLP chain (k_mlp_chain.h), shape of k_mlp_chain_c3.hip, with the Hadamard cross block folded into the user's layer-1
// weights (one set of layer-1 fragments per user slot, made by the staging launch): layer 1 contracts over [item | attention].
#include "k_mlp_chain.h"

namespace aif {

// k_mlp_acc (k_mlp_acc.hip) gives every compute unit one block at a time and whole tiles of 256 candidates, so it takes as long as
// its fullest block: 18 us a round of one tile a unit, where the chain takes 20 us for as many and fills a last round in quarters.
// It serves batches of two rounds and more that fill at least 85 % of their rounds.  Whole calls, 10^4 candidates a user over 100
// history items, us, chain / k_mlp_acc (how full): 6 users (0.94 of one round) 47.3 / 48.7; 8 (0.63 of two) 58.6 / 64.7;
// 16 (0.83 of three) 83.7 / 86.0; 27 (0.84 of five) 129.5 / 129.0; 22 (0.86 of four) 109.2 / 108.5; 11 (0.86 of two) 69.5 / 65.0;
// 28 (0.88 of five) 131.5 / 130.6; 17 (0.89 of three) 94.9 / 89.3; 45 (0.88 of eight) 200.3 / 194.5; 62 (0.97 of ten) 271.1 / 251.0.
// Over 400 items: 28 users 149.2 / 149.3, 17 105.8 / 99.5.  One request of 112,640 (0.86 of two): 265.4 / 262.6.
bool mlp_acc_c3f_serves(const Model &m, int n_blk)
{
    const int64_t cu = n_cu(), rounds = (n_blk + cu - 1) / cu;
    return m.x_tiled && rounds >= 2 && 100 * (int64_t)n_blk >= 85 * rounds * cu;
}

hipError_t mlp_chain_c3f(const Model &m, const Batch &b, const void *X, const MlpPack &pk, const float *bias1, hipStream_t s)
{
    return launch_spec<128, 512, 256, 0, 4, 16, 4, 2, 0, 1>(m, b, X, pk, bias1, s);
}

}  // namespace aif
