"""Few candidates on the shape-agnostic kernels, attention and head in one launch, against the two of larger batches; and keys that
stay resident in batches of nearly a full round of blocks."""
import numpy as np
import pytest

from paper_2511_12934_amd import binding as B
from paper_2511_12934_amd import workloads as wl

from helpers import assert_logits_close, oracle_scores
from test_gpu_parity import R, _say, run_batch, small_cfg, torch  # noqa: F401  (fixtures)

pytestmark = pytest.mark.gpu

SHAPES = {
    "c1": dict(d_item=64, d_user=64, d_attn=32, use_wq=True, mlp_dims=(224, 128, 64, 1)),
    "head_64": dict(d_item=64, d_user=64, d_attn=64, mlp_dims=(256, 512, 256, 1)),                   # two activation buffers
    "head_16_wide_row": dict(d_item=80, d_user=80, d_attn=16, n_heads=1, mlp_dims=(256, 24, 1)),     # ragged k-steps, one hidden layer
    "two_heads_of_72": dict(d_item=144, d_user=144, d_attn=144, n_heads=2, mlp_dims=(576, 40, 30, 20, 1)),
    "no_cross": dict(d_item=32, d_user=16, d_attn=32, cross_mode=wl.CROSS_NONE, mlp_dims=(80, 33, 1)),
}


def requests(cfg, rng, sizes, lens):
    out = []
    for r, (n, l) in enumerate(zip(sizes, lens)):
        ids = rng.integers(0, cfg.n_items, n).astype(np.int32)
        if r == 1:
            ids[[0, n // 2, n - 1]] = [-1, 2_000_000_000, cfg.n_items]
        out.append((wl.make_user(cfg, rng, sigma=1.0, seq_len=l), ids))
    return out


# tiles of 16 round their edges and a ROW_BLOCK's; histories of no, one, few and ragged chunks; `odd`: values that are not finite send
# candidates the plain way
@pytest.mark.parametrize("odd", [False, True])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("shape", list(SHAPES))
def test_one_launch_gives_the_bits_of_two(R, torch, monkeypatch, shape, dtype, odd):  # noqa: F811
    if dtype == "bf16":
        monkeypatch.setenv("AIF_FORCE_GENERIC", "1")
    cfg = small_cfg(dtype, n_items=3000, seq_len=70, **SHAPES[shape])
    _say(f"one launch, {shape} {dtype} odd={odd}")
    rng = np.random.default_rng(59)
    model = wl.make_model(cfg, seed=9, bias_scale=0.3)
    table = wl.make_table_host(cfg, rng, n_items=3000, sigma=1.0)
    # (three pieces of two heads of 72: the keys of 32 items fit LDS beside the head)
    lens = (30, 0, 1, 32, 17, 32) if dtype == "f32" and shape == "two_heads_of_72" else (70, 0, 1, 32, 33, 64)
    users_ids = requests(cfg, rng, (1, 33, 16, 257, 15, 256), lens)
    if odd:
        table[users_ids[3][1][[3, 200]], 5] = np.inf, np.nan
        users_ids[4][0].seq_vals[2, 3] = -np.inf
    table_dev = R.to_device(table, dtype)
    got, got_y, _, ctx = run_batch(R, torch, cfg, model, table_dev, users_ids, max_seq_len=70)
    assert ctx.aif_last_forms() == B.FORM_ONE_LAUNCH
    bad = ctx.aif_poll_device_errors()
    X = [R.peek_features(ctx, cfg, r, ids.size) for r, (_, ids) in enumerate(users_ids)]
    monkeypatch.setenv("AIF_MLP_TILE", "0")
    ref, ref_y, _, ctx0 = run_batch(R, torch, cfg, model, table_dev, users_ids, max_seq_len=70)
    assert ctx0.aif_last_forms() == 0
    assert bad == 3 and ctx0.aif_poll_device_errors() == 3
    for r, (u, ids) in enumerate(users_ids):
        assert np.array_equal(X[r], R.peek_features(ctx0, cfg, r, ids.size), equal_nan=True), r
        assert np.array_equal(got[r], ref[r], equal_nan=True) and np.array_equal(got_y[r], ref_y[r], equal_nan=True), r
    if dtype == "f32" and not odd:
        assert_logits_close("f32", got[3], oracle_scores(cfg, model, table, *users_ids[3]).logits, "against the oracle")


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("n_req,seq_len", [(440, 40), (960, 90)])
def test_resident_keys_give_the_bits_of_single_requests(R, torch, monkeypatch, dtype, n_req, seq_len):  # noqa: F811
    """Blocks that fill a round (440 of 512) over histories of two chunks, two rounds (960 of 1,024) over three."""
    if dtype == "bf16":
        monkeypatch.setenv("AIF_FORCE_GENERIC", "1")
    cfg = small_cfg(dtype, n_items=3000, seq_len=seq_len, d_item=32, d_user=32, d_attn=32, use_wq=True, mlp_dims=(128, 70, 20, 1))
    _say(f"resident keys {n_req} x {seq_len} {dtype}")
    rng = np.random.default_rng(61)
    model = wl.make_model(cfg, seed=5, bias_scale=0.3)
    table = wl.make_table_host(cfg, rng, sigma=1.0)
    users_ids = requests(cfg, rng, rng.integers(3, 257, n_req), [seq_len, *rng.integers(0, seq_len + 1, n_req - 1)])
    zs, _, _, ctx = run_batch(R, torch, cfg, model, R.to_device(table, dtype), users_ids, max_seq_len=seq_len)
    assert ctx.aif_last_forms() & B.FORM_KEYS_RESIDENT
    for r in (0, 1, 70, n_req - 1):
        alone = R.upload_request(cfg, *users_ids[r])
        ctx.aif_score_request(alone.req)
        torch.cuda.synchronize()
        assert ctx.aif_last_forms() == B.FORM_ONE_LAUNCH
        assert np.array_equal(alone.logits.cpu().numpy(), zs[r], equal_nan=True), r
