"""Large batches on the shape-agnostic kernels of a bf16 model: the head that keeps its activations in registers against the one that
small requests take, bit for bit."""
import numpy as np
import pytest

from paper_2511_12934_amd import binding as B
from paper_2511_12934_amd import workloads as wl

from helpers import assert_bf16_logits_tight, oracle_scores
from test_gpu_parity import R, _say, run_batch, small_cfg, torch  # noqa: F401  (fixtures)

pytestmark = pytest.mark.gpu

SHAPES = {
    "five_k_steps_128_64": dict(d_item=64, d_user=64, d_attn=32, use_wq=True, mlp_dims=(224, 128, 64, 1)),
    "one_hidden_layer": dict(d_item=32, d_user=16, d_attn=32, cross_mode=wl.CROSS_NONE, mlp_dims=(80, 100, 1)),
    "ragged_k_steps_and_tiles": dict(d_item=72, d_user=72, d_attn=72, mlp_dims=(288, 36, 100, 1)),       # 216 columns, pairs past the widths
    "narrowest": dict(d_item=16, d_user=16, d_attn=16, cross_mode=wl.CROSS_NONE, mlp_dims=(48, 4, 4, 1)),
    "eight_k_steps": dict(d_item=80, d_user=80, d_attn=80, mlp_dims=(320, 68, 128, 1)),
    "width_not_of_fours": dict(d_item=64, d_user=64, d_attn=32, use_wq=True, mlp_dims=(224, 126, 1)),    # stays with the other kernel
}
SIZES = (12_000, 1, 255, 12_500, 12_600)         # 1,168 tiles of 32 candidates


# the ends of requests round a tile of 32 and a ROW_BLOCK; `odd`: values that are not finite send candidates the plain way, and
# their neighbours not
@pytest.mark.parametrize("odd", [False, True])
@pytest.mark.parametrize("shape", list(SHAPES))
def test_large_batch_gives_the_bits_of_small_requests(R, torch, monkeypatch, shape, odd):  # noqa: F811
    monkeypatch.setenv("AIF_FORCE_GENERIC", "1")
    cfg = small_cfg("bf16", n_items=3000, seq_len=40, **SHAPES[shape])
    _say(f"chain, {shape} odd={odd}")
    rng = np.random.default_rng(67)
    model = wl.make_model(cfg, seed=13, bias_scale=0.3)
    table = wl.make_table_host(cfg, rng, n_items=3000, sigma=1.0)
    users_ids = [(wl.make_user(cfg, rng, sigma=1.0, seq_len=l), rng.integers(10, 3000, n).astype(np.int32)) for n, l in zip(SIZES, (40, 7, 0, 33, 40))]
    users_ids[3][1][[0, 6000, 12_499]] = [-1, 2_000_000_000, 3000]
    if odd:
        table[:3, 5] = np.inf, np.nan, -np.inf
        users_ids[0][1][[17, 300, 301]] = 0, 1, 2
        users_ids[4][0].seq_vals[2, 3] = -np.inf
    zs, ys, _, ctx = run_batch(R, torch, cfg, model, R.to_device(table, "bf16"), users_ids, max_seq_len=40)
    assert ctx.aif_last_forms() & B.FORM_HEAD_REGISTERS == (0 if shape == "width_not_of_fours" else B.FORM_HEAD_REGISTERS)
    assert ctx.aif_poll_device_errors() == 3
    for r, (u, ids) in enumerate(users_ids):
        for lo in {0, max(0, ids.size - 700)}:
            alone = R.upload_request(cfg, u, ids[lo:lo + 700])
            ctx.aif_score_request(alone.req)
            torch.cuda.synchronize()
            assert ctx.aif_last_forms() & B.FORM_HEAD_REGISTERS == 0
            z = alone.logits.cpu().numpy()
            assert np.array_equal(z, zs[r][lo:lo + 700], equal_nan=True), (r, lo)
    assert np.isnan(zs[3][[0, 6000, 12_499]]).all()
    if not odd:
        assert_bf16_logits_tight(zs[4][:700], oracle_scores(cfg, model, table, users_ids[4][0], users_ids[4][1][:700]).logits, shape)


# 600 blocks of 256: a wave takes two or three tiles of 32, the next one's rows and descriptor on their way meanwhile; requests that
# end within them; values that are not finite in the first, second and third tile of a wave (2,048 tiles apart) and in neighbouring
# tiles of others
LOOP_SIZES = (40_000, 1, 255, 60_000, 300, 52_000)


@pytest.mark.parametrize("odd", [False, True])
@pytest.mark.parametrize("shape", ["five_k_steps_128_64", "one_hidden_layer", "ragged_k_steps_and_tiles"])
def test_waves_of_several_tiles_give_the_bits_of_small_requests(R, torch, monkeypatch, shape, odd):  # noqa: F811
    n_cu = torch.cuda.get_device_properties(0).multi_processor_count
    if n_cu != 256:
        pytest.skip("tiles of a wave are placed for 256 compute units")
    monkeypatch.setenv("AIF_FORCE_GENERIC", "1")
    cfg = small_cfg("bf16", n_items=3000, seq_len=20, **SHAPES[shape])
    _say(f"chain of several tiles, {shape} odd={odd}")
    rng = np.random.default_rng(71)
    model = wl.make_model(cfg, seed=13, bias_scale=0.3)
    table = wl.make_table_host(cfg, rng, n_items=3000, sigma=1.0)
    users_ids = [(wl.make_user(cfg, rng, sigma=1.0, seq_len=l), rng.integers(10, 3000, n).astype(np.int32)) for n, l in zip(LOOP_SIZES, (20, 7, 0, 13, 20, 3))]
    base = np.cumsum([0] + [-(-n // 256) * 256 for n in LOOP_SIZES])[:-1]
    look = [(r, lo) for r, n in enumerate(LOOP_SIZES) for lo in sorted({0, max(0, n // 2 - 300), max(0, n - 600)})]
    users_ids[3][1][[0, 30_000, 59_999]] = [-1, 2_000_000_000, 3000]
    if odd:
        table[:3, 5] = np.inf, np.nan, -np.inf
        for k, row in enumerate((1000, 1000 + 32 * 2048, 1000 + 32 * 4096, 1032, 1040 + 32 * 2048)):     # rows of the workspace
            r = int(np.searchsorted(base, row, side="right")) - 1
            at = row - int(base[r])
            assert at < LOOP_SIZES[r]
            users_ids[r][1][at] = k % 3
            look.append((r, max(0, min(at - 100, LOOP_SIZES[r] - 600))))
        users_ids[5][0].seq_vals[2, 3] = -np.inf
    zs, _, _, ctx = run_batch(R, torch, cfg, model, R.to_device(table, "bf16"), users_ids, max_seq_len=20)
    assert ctx.aif_last_forms() & B.FORM_HEAD_REGISTERS
    assert ctx.aif_poll_device_errors() == 3
    for r, lo in look:
        u, ids = users_ids[r]
        alone = R.upload_request(cfg, u, ids[lo:lo + 600])
        ctx.aif_score_request(alone.req)
        torch.cuda.synchronize()
        assert ctx.aif_last_forms() & B.FORM_HEAD_REGISTERS == 0
        assert np.array_equal(alone.logits.cpu().numpy(), zs[r][lo:lo + 600], equal_nan=True), (r, lo)
    assert all(np.isfinite(z).all() for r, z in enumerate(zs) if r not in (3, 5) and not odd)
