"""How the resident attention kernel's work is cut into workgroups must not show: ragged batches, their tables written by
the staging launch (up to 16 requests) or uploaded, around one request per compute unit, against each request alone."""
import numpy as np
import pytest

from paper_2511_12934_amd import workloads as wl

from test_gpu_parity import MFMA_SHAPES, R, _say, run_batch, small_cfg, torch  # noqa: F401  (fixtures)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", ["c3_like", "c4_like"])
@pytest.mark.parametrize("n_req", [2, 16, 17, -1, 0, 1])        # the last three: one fewer than the compute units, as many, one more
def test_ragged_batches_give_the_bits_of_single_requests(R, torch, shape, n_req):  # noqa: F811
    cfg = small_cfg("bf16", n_items=3000, seq_len=300, **MFMA_SHAPES[shape])
    n = n_req if n_req > 1 else torch.cuda.get_device_properties(0).multi_processor_count + n_req
    _say(f"attention groups {shape}, {n} requests")
    rng = np.random.default_rng(17)
    model = wl.make_model(cfg, seed=3, bias_scale=0.2)
    table = wl.make_table_host(cfg, rng, sigma=1.0)
    sizes = [5000, 1, 127, 33, 0, 1600, 129, 32] if n < 100 else [40, 1, 129, 300, 0, 32]
    users_ids = [(wl.make_user(cfg, rng, sigma=1.0, seq_len=[300, 1, 65, 0, 200][r % 5]),
                  rng.integers(0, cfg.n_items, sizes[r % len(sizes)]).astype(np.int32)) for r in range(n)]
    zs, _, _, ctx = run_batch(R, torch, cfg, model, R.to_device(table, "bf16"), users_ids, max_seq_len=300)
    assert ctx.aif_stage_kind("attention") == 1
    for r in sorted({0, 1, 5, n // 2, n - 2, n - 1} & set(range(n))):
        alone = R.upload_request(cfg, *users_ids[r])
        ctx.aif_score_request(alone.req)
        torch.cuda.synchronize()
        assert np.array_equal(alone.logits.cpu().numpy(), zs[r]), r
