"""Few candidates, a workgroup to a tile of 32: the head alone (the widest one) and attention and head in one launch, against the
kernels of larger batches (the chain; the widest head: the accumulating kernel; resident and key-split attention)."""
import numpy as np
import pytest

from paper_2511_12934_amd import binding as B
from paper_2511_12934_amd import workloads as wl

from helpers import assert_bf16_logits_tight, oracle_scores
from test_gpu_parity import MFMA_SHAPES, R, _say, run_batch, small_cfg, torch  # noqa: F401  (fixtures)

pytestmark = pytest.mark.gpu


def config(shape):
    if shape in ("B3", "C5"):
        return wl.CONFIGS[shape].scaled(n_items=20000, seq_len=24)
    return small_cfg("bf16", n_items=3000, seq_len=24, **MFMA_SHAPES[shape])


# sizes round a tile and round a block of 256 rows, tiles past a request's end, one request and several, up to the last batch it
# serves (a tile a compute unit) and the first it does not
@pytest.mark.parametrize("sizes", [(1,), (31, 32, 33), (255, 256, 257, 1, 100), "limit", "past the limit"])
@pytest.mark.parametrize("shape", [*MFMA_SHAPES, "B3", "C5"])
def test_few_candidates_give_the_bits_of_many(R, torch, monkeypatch, shape, sizes):  # noqa: F811
    cfg = config(shape)
    _say(f"head of few candidates {shape} {sizes}")
    rng = np.random.default_rng(47)
    model = wl.make_model(cfg, seed=9, bias_scale=0.05)
    table = wl.make_table_host(cfg, rng, n_items=cfg.n_items)
    table_dev = R.to_device(table, "bf16")
    n_cu = torch.cuda.get_device_properties(0).multi_processor_count
    if sizes == "limit":
        sizes = (32 * (n_cu - 3), 90)
    elif sizes == "past the limit":
        sizes = (32 * (n_cu - 3), 90, 1)
    users_ids = []
    for r, n in enumerate(sizes):
        ids = rng.integers(0, cfg.n_items, n).astype(np.int32)
        if r % 2 == 0:
            ids[[0, n // 2, n - 1]] = [-1, 2_000_000_000, cfg.n_items]
        users_ids.append((wl.make_user(cfg, rng, seq_len=int(rng.integers(0, 25))), ids))
    got, got_y, _, ctx = run_batch(R, torch, cfg, model, table_dev, users_ids, max_seq_len=24)
    few = sum(-(-n // 32) for n in sizes) <= n_cu               # (the others' one launch goes on to two tiles a unit)
    assert ctx.aif_last_forms() == ((B.FORM_HEAD_TILE if few else 0) if shape == "C5" else B.FORM_ONE_LAUNCH)
    monkeypatch.setenv("AIF_MLP_TILE", "0")
    ref, ref_y, _, ctx0 = run_batch(R, torch, cfg, model, table_dev, users_ids, max_seq_len=24)
    assert ctx0.aif_last_forms() == 0
    for r, (u, ids) in enumerate(users_ids):
        assert np.array_equal(got[r], ref[r], equal_nan=True) and np.array_equal(got_y[r], ref_y[r], equal_nan=True), r
        assert np.isnan(got[r]).sum() == np.sum((ids < 0) | (ids >= cfg.n_items))
    if len(sizes) > 2 and sizes[1] == 32:
        u, ids = users_ids[1]
        assert_bf16_logits_tight(got[1], oracle_scores(cfg, model, table, u, ids).logits, "against the oracle")


# a head of one run of keys (K/V that fit the resident kernel's LDS: 18 key tiles of 64 features) and of KEY_PARTS, alone and
# mixed; no history, ragged stages, a bound that needs the true maximum (sigma 4), more than one tile a unit
@pytest.mark.parametrize("sigma", [1.0, 4.0])
@pytest.mark.parametrize("lens", [(0, 1, 31), (64, 65, 576), (577, 1100, 700), (1100, 30, 0, 640)])
@pytest.mark.parametrize("shape", [*MFMA_SHAPES, "B3", "two_heads"])
def test_attention_and_head_in_one_launch_give_the_bits_of_two(R, torch, monkeypatch, shape, lens, sigma):  # noqa: F811
    if shape == "two_heads":
        cfg = small_cfg("bf16", n_items=3000, seq_len=24, d_item=64, d_user=64, d_attn=64, n_heads=2, mlp_dims=(256, 256, 128, 1))
    else:
        cfg = config(shape)
    _say(f"one launch {shape} {lens} sigma={sigma}")
    rng = np.random.default_rng(53)
    model = wl.make_model(cfg, seed=9, bias_scale=0.05)
    table = wl.make_table_host(cfg, rng, n_items=cfg.n_items, sigma=sigma)
    table_dev = R.to_device(table, "bf16")
    n_cu = torch.cuda.get_device_properties(0).multi_processor_count
    for big in (0, 32 * (n_cu + 9)):                            # past a tile a unit: workgroups of four waves
        users_ids = []
        for r, l in enumerate(lens):
            n = [33, 100, 257, 1][r] + (big if r == 0 else 0)
            ids = rng.integers(0, cfg.n_items, n).astype(np.int32)
            if r == 1:
                ids[[0, n // 2, n - 1]] = [-1, 2_000_000_000, cfg.n_items]
            users_ids.append((wl.make_user(cfg, rng, seq_len=l, sigma=sigma), ids))
        got, got_y, _, ctx = run_batch(R, torch, cfg, model, table_dev, users_ids, max_seq_len=1100)
        # several heads: one launch while all K/V fit the resident kernel's LDS, else the head alone, up to a tile a unit
        dh = cfg.d_attn // cfg.n_heads
        streamed = any(cfg.n_heads * ((-(-l // 32) + 1) // 2 * 2) * (dh // 8) > 152 for l in lens)
        assert ctx.aif_last_forms() == (B.FORM_ONE_LAUNCH if cfg.n_heads == 1 or not streamed else 0 if big else B.FORM_HEAD_TILE)
        bad = ctx.aif_poll_device_errors()
        X = [R.peek_features(ctx, cfg, r, ids.size) for r, (_, ids) in enumerate(users_ids)]
        with monkeypatch.context() as mp:
            mp.setenv("AIF_MLP_TILE", "0")
            ref, ref_y, _, ctx0 = run_batch(R, torch, cfg, model, table_dev, users_ids, max_seq_len=1100)
        assert ctx0.aif_last_forms() == 0
        assert bad == 3 and ctx0.aif_poll_device_errors() == 3
        assert ctx.aif_stage_kind("gather") == ctx0.aif_stage_kind("gather")
        for r, (u, ids) in enumerate(users_ids):
            assert np.array_equal(X[r], R.peek_features(ctx0, cfg, r, ids.size)), r
            assert np.array_equal(got[r], ref[r], equal_nan=True) and np.array_equal(got_y[r], ref_y[r], equal_nan=True), r
        if sigma == 1.0 and not big:
            u, ids = users_ids[2]
            assert_bf16_logits_tight(got[2], oracle_scores(cfg, model, table, u, ids).logits, "against the oracle")


# the last batch that is one launch and the first that is not: two tiles a unit, six where every history is streamed
@pytest.mark.parametrize("shape,seq_len,per_unit", [("c2_like", 20, 2), ("c3_like", 600, 6), ("c4_like", 20, 2)])
def test_where_one_launch_ends(R, torch, monkeypatch, shape, seq_len, per_unit):  # noqa: F811
    cfg = config(shape)
    _say(f"end of one launch {shape} L={seq_len}")
    rng = np.random.default_rng(57)
    model = wl.make_model(cfg, seed=9, bias_scale=0.05)
    table_dev = R.to_device(wl.make_table_host(cfg, rng, n_items=cfg.n_items), "bf16")
    n_cu = torch.cuda.get_device_properties(0).multi_processor_count
    users_ids = [(wl.make_user(cfg, rng, seq_len=seq_len), rng.integers(0, cfg.n_items, n).astype(np.int32)) for n in (32 * (per_unit * n_cu - 3), 90, 1)]
    for n, form in ((2, B.FORM_ONE_LAUNCH), (3, 0)):
        got, _, _, ctx = run_batch(R, torch, cfg, model, table_dev, users_ids[:n], max_seq_len=seq_len)
        assert ctx.aif_last_forms() == form
        with monkeypatch.context() as mp:
            mp.setenv("AIF_MLP_TILE", "0")
            ref, _, _, _ = run_batch(R, torch, cfg, model, table_dev, users_ids[:n], max_seq_len=seq_len)
        assert all(np.array_equal(a, b) for a, b in zip(got, ref))


def test_a_timed_call_keeps_the_stages_apart_that_it_times(R, torch):  # noqa: F811
    cfg = config("c3_like")
    rng = np.random.default_rng(58)
    model = wl.make_model(cfg, seed=9, bias_scale=0.05)
    table_dev = R.to_device(wl.make_table_host(cfg, rng, n_items=cfg.n_items), "bf16")
    ui = [(wl.make_user(cfg, rng, seq_len=24), rng.integers(0, cfg.n_items, 200).astype(np.int32))]
    z, _, drs, ctx = run_batch(R, torch, cfg, model, table_dev, ui, max_seq_len=24)
    for stages, form in ((("attention",), B.FORM_HEAD_TILE), (("mlp",), B.FORM_HEAD_TILE), (("user_fold",), B.FORM_ONE_LAUNCH), (("gather", "topk"), B.FORM_ONE_LAUNCH)):
        ctx.aif_profile_begin_stages(1, stages)
        drs[0].logits.fill_(float("nan"))
        ctx.aif_score_batch([drs[0].req])
        torch.cuda.synchronize()
        ctx.aif_profile_end()
        assert ctx.aif_last_forms() == form, stages
        assert np.array_equal(drs[0].logits.cpu().numpy(), z[0])
