"""The shape-agnostic kernels of fp32 precision (bf16 pieces on the matrix cores) at the edges of their tiles, against the
oracle, and the plain route they take where an input is not finite."""
import numpy as np
import pytest

from paper_2511_12934_amd import workloads as wl

from helpers import assert_features_close, assert_logits_close, key_rounding_term, oracle_scores
from test_gpu_parity import R, _say, run_batch, small_cfg, torch  # noqa: F401  (fixtures)

pytestmark = pytest.mark.gpu

# head widths around the 16-feature tiles and 32-wide k-steps, item widths around a k-step, layer widths around the row
# tiles, several heads of a query projection at every tile count a head can have, and heads too wide for the matrix-core
# form (132) or layers for
# split activations in LDS (1280 -> 1280 takes all of a compute unit's for the plain form)
SHAPES = {
    "head_3": dict(d_item=12, d_user=12, d_attn=12, n_heads=4, mlp_dims=(48, 17, 1)),
    "head_16": dict(d_item=16, d_user=16, d_attn=16, mlp_dims=(64, 16, 15, 1)),
    "head_20_wq": dict(d_item=36, d_user=36, d_attn=40, n_heads=2, use_wq=True, mlp_dims=(148, 33, 1)),
    "head_64": dict(d_item=64, d_user=64, d_attn=64, mlp_dims=(256, 129, 65, 1)),
    "head_68_wq": dict(d_item=28, d_user=28, d_attn=68, use_wq=True, mlp_dims=(152, 1)),
    "head_128_none": dict(d_item=128, d_user=4, d_attn=128, cross_mode=wl.CROSS_NONE, mlp_dims=(260, 40, 1)),
    "heads_40_wq": dict(d_item=40, d_user=40, d_attn=160, n_heads=4, use_wq=True, mlp_dims=(280, 33, 1)),
    "heads_72_wq": dict(d_item=40, d_user=40, d_attn=144, n_heads=2, use_wq=True, mlp_dims=(264, 33, 1)),
    "heads_80_wq": dict(d_item=64, d_user=64, d_attn=240, n_heads=3, use_wq=True, mlp_dims=(432, 17, 1)),
    "heads_96_wq": dict(d_item=72, d_user=72, d_attn=384, n_heads=4, use_wq=True, mlp_dims=(600, 1)),
    "head_132": dict(d_item=132, d_user=132, d_attn=132, mlp_dims=(528, 64, 1)),
    "wide_layers": dict(mlp_dims=(56, 1280, 1280, 1)),
    "segdot": dict(d_item=48, d_user=12, d_attn=32, use_wq=True, cross_mode=wl.CROSS_SEGDOT, n_cross=8, d_cross_vec=24, mlp_dims=(108, 31, 1)),
}
SIZES = [(1, 65), (15, 1), (16, 0), (17, 31), (63, 32), (65, 33), (256, 64), (257, 63), (300, 65)]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("shape", list(SHAPES))
def test_pieces_kernels_at_tile_edges(R, torch, monkeypatch, dtype, shape):  # noqa: F811
    kw = dict(SHAPES[shape])
    if dtype == "bf16":
        if any(kw.get(k, 16) % 8 for k in ("d_item", "d_attn")):
            pytest.skip("widths are multiples of eight in bf16")
        monkeypatch.setenv("AIF_FORCE_GENERIC", "1")
    cfg = small_cfg(dtype, seq_len=65, n_items=400, **kw)
    _say(f"pieces {shape} {dtype}")
    rng = np.random.default_rng(99)
    model = wl.make_model(cfg, seed=5, bias_scale=0.3)
    table = wl.make_table_host(cfg, rng, sigma=1.0)
    users_ids = [(wl.make_user(cfg, rng, sigma=1.0, seq_len=L), rng.integers(0, cfg.n_items, n).astype(np.int32)) for n, L in SIZES]
    zs, _, drs, ctx = run_batch(R, torch, cfg, model, R.to_device(table, dtype), users_ids, max_seq_len=65)
    assert ctx.aif_stage_kind("attention") == 0 and ctx.aif_stage_kind("mlp") == 0
    for r, ((u, ids), z) in enumerate(zip(users_ids, zs)):
        ref = oracle_scores(cfg, model, table, u, ids)
        X = R.peek_features(ctx, cfg, r, ids.size)
        assert np.array_equal(X[:, :cfg.d_item], table[ids])
        assert_features_close(dtype, X[:, cfg.d_item:cfg.d_item + cfg.d_attn], ref.attn, f"req {r} attention", key_rounding_term(cfg, model, table[ids], u))
        if dtype == "f32":
            assert_logits_close(dtype, z, ref.logits, f"req {r}")
        else:
            assert np.abs(z - ref.logits).max() <= 2e-2 * max(1.0, float(np.abs(ref.logits).max())), f"req {r}"


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("seq_len,n_heads", [(40, 1), (700, 1), (40, 2), (30, 4)])
def test_large_batches_give_the_bits_of_single_requests(R, torch, monkeypatch, dtype, seq_len, n_heads):  # noqa: F811
    """520 requests take the kernels with 32 candidates a block (MLP) and all keys of every head resident or, of 700, 32 at a
    time in blocks of eight waves (attention); one alone those with 16 candidates and four waves."""
    if dtype == "bf16":
        monkeypatch.setenv("AIF_FORCE_GENERIC", "1")
    cfg = small_cfg(dtype, seq_len=seq_len, n_items=3000, d_item=32, d_user=32, d_attn=32, n_heads=n_heads, use_wq=True, mlp_dims=(128, 70, 20, 1))
    rng = np.random.default_rng(3)
    model = wl.make_model(cfg, seed=5, bias_scale=0.3)
    table = wl.make_table_host(cfg, rng, sigma=1.0)
    users_ids = [(wl.make_user(cfg, rng, sigma=1.0, seq_len=int(rng.integers(0, seq_len + 1))), rng.integers(0, 3000, int(rng.integers(1, 257))).astype(np.int32))
                 for _ in range(520)]
    zs, _, drs, ctx = run_batch(R, torch, cfg, model, R.to_device(table, dtype), users_ids, max_seq_len=seq_len)
    for r in (0, 1, 70, 519):
        alone = R.upload_request(cfg, *users_ids[r])
        ctx.aif_score_request(alone.req)
        torch.cuda.synchronize()
        assert np.array_equal(alone.logits.cpu().numpy(), zs[r]), r
        if n_heads > 1:
            ref = oracle_scores(cfg, model, table, *users_ids[r])
            cols = slice(cfg.d_item, cfg.d_item + cfg.d_attn)
            X = R.peek_features(ctx, cfg, 0, users_ids[r][1].size)
            assert_features_close(dtype, X[:, cols], ref.attn, f"req {r} attention", key_rounding_term(cfg, model, table[users_ids[r][1]], users_ids[r][0]))


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("n_req,seq_len", [(3, 65), (520, 65), (130, 700)])
def test_keys_past_the_end_weigh_nothing_however_low_the_real_scores(R, torch, monkeypatch, dtype, n_req, seq_len):  # noqa: F811
    """Real scores of -1e32 and below, far enough apart that the softmax is one key's, whose value the attention then is:
    histories that end inside a chunk of 32 keys, at its first and last key, and one key alone, in the small, the resident
    and the streamed form."""
    if dtype == "bf16":
        monkeypatch.setenv("AIF_FORCE_GENERIC", "1")
    cfg = small_cfg(dtype, seq_len=seq_len, n_items=300, d_item=32, d_user=32, d_attn=32, mlp_dims=(128, 16, 1))
    _say(f"keys past the end {dtype} {n_req} x {seq_len}")
    rng = np.random.default_rng(6)
    model = wl.make_model(cfg, seed=5, bias_scale=0.3)
    table = wl.round_storage((1e16 * (1 + rng.random((300, 32)))).astype(np.float32), dtype)
    users_ids = []
    for r in range(n_req):
        L = (1, 31, 33, 40, 63, 64, 65, seq_len - 3)[r % 8] if n_req > 3 else (1, 33, 65)[r]
        u = wl.make_user(cfg, rng, sigma=1.0, seq_len=L)
        u.seq_keys[:] = wl.round_storage(-1e16 * (1 + rng.permutation(L)[:, None] / np.float32(L)) * np.ones((1, 32), np.float32), dtype)
        # several keys may round to the same low value in 16 bits: one of them is made the highest
        u.seq_keys[int(rng.integers(0, L))] *= 0.5
        users_ids.append((u, rng.integers(0, 300, int(rng.integers(1, 257))).astype(np.int32)))
    ctx = run_batch(R, torch, cfg, model, R.to_device(table, dtype), users_ids, max_seq_len=seq_len)[3]
    for r in range(min(n_req, 16)):
        u, ids = users_ids[r]
        X = R.peek_features(ctx, cfg, r, ids.size)
        want = u.seq_vals[np.argmax(u.seq_keys[:, 0])]
        assert np.array_equal(X[:, 32:64], np.broadcast_to(want, (ids.size, 32))), (r, u.seq_keys.shape[0])


@pytest.mark.parametrize("seq_len", [40, 64, 700])
@pytest.mark.parametrize("d_attn", [32, 64])
def test_large_scores_beside_a_value_that_is_not_finite(R, torch, seq_len, d_attn):  # noqa: F811
    """Scores around -1e12, one key's far above the rest: the attention is that key's value -- by the pieces, and by plain
    arithmetic where an infinite value elsewhere sends the candidate there: zero times infinity in its own feature only."""
    cfg = small_cfg("f32", seq_len=seq_len, n_items=300, d_item=64, d_user=64, d_attn=d_attn, mlp_dims=(192 + d_attn, 16, 1))
    _say(f"large scores {seq_len} x {d_attn}")
    rng = np.random.default_rng(7)
    model = wl.make_model(cfg, seed=5, bias_scale=0.3)
    table = (1e6 * (1 + rng.random((300, 64)))).astype(np.float32)
    u = wl.make_user(cfg, rng, sigma=1.0)
    u.seq_keys[:] = -1e6 * (1 + rng.permutation(seq_len)[:, None] / np.float32(seq_len)) * np.ones((1, d_attn), np.float32)
    top = int(np.argmax(u.seq_keys[:, 0]))
    ids = np.arange(100, dtype=np.int32)
    for odd in (False, True):
        if odd:
            u.seq_vals[(top + 1) % seq_len, 5] = np.inf
        ctx = run_batch(R, torch, cfg, model, R.to_device(table, "f32"), [(u, ids)])[3]
        got = R.peek_features(ctx, cfg, 0, ids.size)[:, 64:64 + d_attn]
        keep = np.arange(d_attn) != 5 if odd else np.ones(d_attn, bool)
        same = bool(np.all(got[:, keep] == u.seq_vals[top][keep]))
        assert same, odd
        assert not odd or np.isnan(got[:, 5]).all()


def plain_logits(cfg, model, rows, u):
    """The path in numpy, in 64 bits, with the kernels' maxima: fmax(NaN, x) = x (ReLU turns a NaN into zero)."""
    f = lambda a: np.asarray(a, np.float64)  # noqa: E731
    e, K, V = f(rows), f(u.seq_keys), f(u.seq_vals)
    s = e[:, :cfg.d_attn] @ K.T / np.sqrt(cfg.d_attn)
    p = np.exp(s - np.fmax.reduce(s, axis=1, keepdims=True))
    a = (p @ V) / p.sum(1, keepdims=True)
    y = np.concatenate([np.broadcast_to(f(u.user_vec), e.shape), e, a, e * f(u.user_vec)], 1)
    for i, (w, b) in enumerate(zip(model.weights, model.biases)):
        y = (y[:, None, :] * f(w)).sum(2) + f(b)
        y = y if i + 1 == len(model.weights) else np.fmax(y, 0)
    return y[:, 0]


@pytest.mark.parametrize("where", ["row", "key", "value", "weight"])
def test_values_that_are_not_finite_propagate_as_in_plain_fp32(R, torch, where):  # noqa: F811
    """An infinity is no sum of bf16 pieces: such candidates take plain fp32 arithmetic, and the others are untouched."""
    cfg = small_cfg("f32", seq_len=40, n_items=300, d_item=32, d_user=32, d_attn=32, mlp_dims=(128, 40, 20, 1))
    rng = np.random.default_rng(4)
    model = wl.make_model(cfg, seed=5, bias_scale=0.3)
    table = wl.make_table_host(cfg, rng, sigma=1.0)
    u = wl.make_user(cfg, rng, sigma=1.0)
    ids = np.arange(200, dtype=np.int32)
    z0 = run_batch(R, torch, cfg, model, R.to_device(table, "f32"), [(u, ids)])[0][0]
    odd = np.zeros(ids.size, bool)
    if where == "row":
        odd[[5, 18, 40]] = True
        table[5, 3], table[18, 31], table[40, 0] = np.inf, -np.inf, np.nan
    elif where == "key":
        odd[:] = True
        u.seq_keys[33, 5] = np.inf
    elif where == "value":
        odd[:] = True
        u.seq_vals[2, 5] = -np.inf
    else:
        odd[:] = True
        model.weights[1][7, 3] = np.inf
    z = run_batch(R, torch, cfg, model, R.to_device(table, "f32"), [(u, ids)])[0][0]
    with np.errstate(all="ignore"):
        ref = plain_logits(cfg, model, table[ids], u)
    assert np.array_equal(z[~odd], z0[~odd])
    assert np.array_equal(np.isnan(z), np.isnan(ref)) and np.array_equal(np.isinf(z), np.isinf(ref))
    assert np.array_equal(np.sign(z[np.isinf(z)]), np.sign(ref[np.isinf(z)]))
    ok = np.isfinite(ref)
    if ok.any():
        assert_logits_close("f32", z[ok], ref[ok], where)
