"""Shape-agnostic head: a hidden value whose sum of pieces overflows to minus infinity while the sum in fp32 does not.  The ReLU must not
hide it: the candidate is done again in plain fp32 arithmetic, as one whose sum overflows upwards is."""
import numpy as np
import pytest

from paper_2511_12934_amd import workloads as wl

from helpers import assert_logits_close, oracle_scores
from test_gpu_parity import R, _say, run_batch, small_cfg, torch  # noqa: F401  (fixtures)

pytestmark = pytest.mark.gpu

# the item value that does it: activations of (2 - 2^-9) 2^63, whose leading piece is 2^64; two of them times -2^63 make 2^128 out of
# the leading pieces and (2 - 2^-9) 2^127 in full; four of 1.375 2^63 in the next k-step bring the sum back up
BIG, W1_LOW, W1_UP, W2, W3 = 1.375 * 2.0 ** 31, 1.453125 * 2.0 ** 32, 2.0 ** 32, 2.0 ** 63, 2.0 ** -125
LOW, UP = [0, 1], [32, 33, 34, 35]


# 700 candidates in one launch and in two; 40,000: the blocks of 32 candidates (fp32), the head with its activations in registers (bf16)
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("n,tile", [(700, "1"), (700, "0"), (40_000, "1")])
def test_a_hidden_sum_of_minus_infinity_is_done_again(R, torch, monkeypatch, dtype, n, tile):  # noqa: F811
    monkeypatch.setenv("AIF_MLP_TILE", tile)
    if dtype == "bf16":
        monkeypatch.setenv("AIF_FORCE_GENERIC", "1")
    cfg = small_cfg(dtype, n_items=3000, seq_len=20, d_item=64, d_user=64, d_attn=32, use_wq=True, mlp_dims=(224, 128, 64, 1))
    _say(f"hidden sum of minus infinity, {dtype} n={n} tile={tile}")
    rng = np.random.default_rng(83)
    model = wl.make_model(cfg, seed=3, bias_scale=0.3)
    model.w_q[:, 0] = 0.0
    w1, w2, w3 = (w.reshape(o, i) for w, o, i in zip(model.weights, cfg.mlp_dims[1:], cfg.mlp_dims[:-1]))
    item0 = cfg.d_user                                      # the item row's first column of [user | item | attention | cross]
    w1[:, item0] = 0.0
    w1[LOW + UP, :] = 0.0
    w1[LOW, item0], w1[UP, item0] = W1_LOW, W1_UP
    w2[:, LOW + UP] = 0.0
    w2[5, LOW], w2[5, UP] = -W2, W2
    w3[0, 5] = W3
    table = wl.make_table_host(cfg, rng, n_items=3000, sigma=1.0)
    table[:, 0] = 0.0
    table[:2, 0] = BIG
    user = wl.make_user(cfg, rng, sigma=1.0, seq_len=20)
    user.user_vec[0] = 0.0
    ids = rng.integers(2, 3000, n).astype(np.int32)
    odd = [0, 17, 300, n - 1]
    ids[odd] = [0, 1, 0, 1]
    (z,), _, _, _ = run_batch(R, torch, cfg, model, R.to_device(table, dtype), [(user, ids)])
    look = np.unique(odd + list(range(40)) + list(range(n - 40, n)))
    ref = oracle_scores(cfg, model, table, user, ids[look]).logits
    assert np.all(np.abs(ref[np.isin(look, odd)]) > 1.0)    # 0.752 2^127 W3 = 3: what is lost if the sum counts as zero
    assert_logits_close(dtype, z[look], ref, "against the oracle")
