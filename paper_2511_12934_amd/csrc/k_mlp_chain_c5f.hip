// The fused MLP chain (k_mlp_chain.h), shape of k_mlp_chain_c5.hip, with the segment-dot cross block folded into the user's
// layer-1 weights (one set of layer-1 fragments per user slot): layer 1 contracts over [item | attention] = 384 columns.
#include "k_mlp_chain.h"

namespace aif {

// (10^4 candidates a user over 64 history items, whole calls, us, chain / k_mlp_acc3: 1 user 97.9 / 92.2, 3 112.3 / 110.0, 4 180.4 /
// 167.5, 8 237.6 / 221.9, 32 744.5 / 695.9; 1,000 candidates: 1 user 85.9 / 83.9, 8 98.6 / 94.3.  The chain is left the row-major workspace.)
bool mlp_acc_c5f_serves(const Model &m) { return m.x_tiled; }

hipError_t mlp_chain_c5f(const Model &m, const Batch &b, const void *X, const MlpPack &pk, const float *bias1, hipStream_t s)
{
    return launch_spec<384, 1024, 512, 256, 4, 16, 4, 1, 0, 1>(m, b, X, pk, bias1, s);
}

}  // namespace aif
