"""The user network's fused launches: keys packed by the projection, FFN and pooling as one launch up to 2,048 positions and
64 features."""
import numpy as np
import pytest

from paper_2511_12934_amd import workloads as wl

from test_gpu_user import R, _say, check_user, oracle_user, run_users, torch  # noqa: F401  (fixtures)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [32, 64, 128])
def test_one_launch_pooling_and_its_limit(R, torch, d):  # noqa: F811
    """Lengths around the 32-position tiles, 64-key stages and 128-row blocks and around the limit; a user beside one beyond
    the limit (two launches for the whole call) gets the bits it gets alone."""
    lens = (2048, 1, 31, 32, 33, 63, 65, 127, 129, 0)
    cfg = wl.UserNetConfig("T", 16, "bf16", len(lens) + 1, 2049, 64, d)
    _say(f"user net pooling d={d}")
    model = wl.make_user_net_model(cfg, bias_scale=0.05)
    rng = np.random.default_rng(7)
    users = [wl.make_raw_user(cfg, rng, seq_len=L) for L in lens]
    got, _, ctx = run_users(R, torch, cfg, model, users)
    for i, u in enumerate(users):
        check_user("bf16", got[i], oracle_user(model, u), d, f"user {i} (L={lens[i]})")
    long = users + [wl.make_raw_user(cfg, rng, seq_len=2049)]
    beside, _, _ = run_users(R, torch, cfg, model, long)
    check_user("bf16", beside[-1], oracle_user(model, long[-1]), d, "L=2049")
    for a, b in zip(got, beside):
        assert np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1])
