"""The head kernel of large batches (layer 2 accumulating while layer 1 is produced) against the chain that serves small ones."""
import numpy as np
import pytest

from paper_2511_12934_amd import workloads as wl

from helpers import assert_bf16_logits_tight, oracle_scores
from test_gpu_parity import MFMA_SHAPES, R, _say, run_batch, small_cfg, torch  # noqa: F401  (fixtures)

pytestmark = pytest.mark.gpu


CHAIN, ACCUMULATING = 1, 3      # aif_last_mlp_kind


def tiles_per_block(n_tiles, n_cu):
    return {(i + 1) * n_tiles // n_cu - i * n_tiles // n_cu for i in range(n_cu)}


# blocks of 256 candidates as multiples of the compute units: every block takes one tile more or fewer than its neighbour; 2.5
# rounds of 3 are the chain's (0.83); 5.9 reuse both halves of the double-buffered biases and ids
@pytest.mark.parametrize("rounds", [1.75, 2, 2.5, 2.9, 5.9])
def test_large_batches_give_the_bits_of_single_requests(R, torch, rounds):  # noqa: F811
    cfg = small_cfg("bf16", n_items=3000, seq_len=24, **MFMA_SHAPES["c3_like"])
    _say(f"head of large batches, {rounds} rounds")
    rng = np.random.default_rng(41)
    model = wl.make_model(cfg, seed=7, bias_scale=0.3)
    table = wl.make_table_host(cfg, rng, sigma=1.0)
    n_cu = torch.cuda.get_device_properties(0).multi_processor_count
    n_blk = int(rounds * n_cu)
    assert max(tiles_per_block(n_blk, n_cu)) == -(-n_blk // n_cu) == int(np.ceil(rounds))
    sizes = [256 * 39 - 1, 1, 256 * 17 + 33, 256 * 8, 256 * 64 + 255, 64]      # requests of many tiles: most tiles share a user with the next
    users_ids, left = [], n_blk
    while left:
        n = min(sizes[len(users_ids) % len(sizes)], 256 * left)
        ids = rng.integers(0, cfg.n_items, n).astype(np.int32)
        if len(users_ids) % 3 == 0:
            ids[[0, n // 2, n - 1]] = [-1, 2_000_000_000, cfg.n_items]
        users_ids.append((wl.make_user(cfg, rng, sigma=1.0, seq_len=int(rng.integers(0, 25))), ids))
        left -= (n + 255) // 256
    zs, ys, _, ctx = run_batch(R, torch, cfg, model, R.to_device(table, "bf16"), users_ids, max_seq_len=24)
    assert ctx.aif_stage_kind("mlp") == 1 and ctx.aif_last_mlp_kind() == (CHAIN if rounds == 2.5 else ACCUMULATING)
    for r, (u, ids) in enumerate(users_ids):
        alone = R.upload_request(cfg, u, ids)
        ctx.aif_score_request(alone.req)
        torch.cuda.synchronize()
        assert ctx.aif_last_mlp_kind() == CHAIN
        assert np.array_equal(alone.logits.cpu().numpy(), zs[r], equal_nan=True), r
        assert np.array_equal(alone.scores.cpu().numpy(), ys[r], equal_nan=True), r
        assert np.isnan(zs[r]).sum() == np.sum((ids < 0) | (ids >= cfg.n_items))
    u, ids = users_ids[2]
    assert_bf16_logits_tight(zs[2], oracle_scores(cfg, model, table, u, ids).logits, "against the oracle")


def test_widest_head_gives_the_bits_of_the_chain(R, torch, monkeypatch):  # noqa: F811
    """C5's head (tiles of 128 candidates; every block four or five of them) against the chain, which serves the row-major
    workspace, bit for bit: requests of sizes around a tile, several requests in a block's run, ids outside the table throughout."""
    cfg = wl.CONFIGS["C5"].scaled(n_items=20000, seq_len=24)
    _say("widest head against the chain")
    rng = np.random.default_rng(43)
    model = wl.make_model(cfg, seed=9, bias_scale=0.05)
    table = wl.make_table_host(cfg, rng, n_items=20000)
    table_dev = R.to_device(table, "bf16")
    n_cu = torch.cuda.get_device_properties(0).multi_processor_count
    sizes, big = [1, 127, 128, 129, 255, 257, 500, 31], [9973, 12000, 20000, 17000, 3001]
    while sum(-(-n // 256) for n in sizes) < 2.2 * n_cu:
        sizes.append(big[len(sizes) % len(big)])
    n_tiles = 2 * sum(-(-n // 256) for n in sizes)
    assert tiles_per_block(n_tiles, n_cu) == {4, 5}
    users_ids = []
    for r, n in enumerate(sizes):
        ids = rng.integers(0, cfg.n_items, n).astype(np.int32)
        if r % 3 == 0:
            ids[[0, n // 2, n - 1]] = [-1, 2_000_000_000, cfg.n_items]
        if n > 1000:
            ids[rng.integers(0, n, 50)] = rng.choice([-1, -2_000_000_000, cfg.n_items, 2_000_000_000], 50)
        users_ids.append((wl.make_user(cfg, rng, seq_len=int(rng.integers(0, 25))), ids))
    got, got_y, _, ctx = run_batch(R, torch, cfg, model, table_dev, users_ids, max_seq_len=24)
    assert ctx.aif_last_mlp_kind() == ACCUMULATING and ctx.aif_mlp_layer1_width() == cfg.d_item + cfg.d_attn
    few, _, _, ctx = run_batch(R, torch, cfg, model, table_dev, users_ids[:6], max_seq_len=24)      # fewer tiles than compute units
    assert ctx.aif_last_mlp_kind() == ACCUMULATING
    monkeypatch.setenv("AIF_X_ROW_MAJOR", "1")
    ref, ref_y, _, ctx = run_batch(R, torch, cfg, model, table_dev, users_ids, max_seq_len=24)
    assert ctx.aif_last_mlp_kind() == CHAIN
    for r, (u, ids) in enumerate(users_ids):
        assert np.array_equal(got[r], ref[r], equal_nan=True) and np.array_equal(got_y[r], ref_y[r], equal_nan=True), r
        assert np.isnan(got[r]).sum() == np.sum((ids < 0) | (ids >= cfg.n_items))
    for r in range(6):
        assert np.array_equal(got[r], few[r], equal_nan=True), r
    u, ids = users_ids[5]
    assert_bf16_logits_tight(got[5], oracle_scores(cfg, model, table, u, ids).logits, "against the oracle")
