"""The user network of few users, whose descriptors travel in the projection's arguments, against the same with its tables uploaded."""
import numpy as np
import pytest

from paper_2511_12934_amd import workloads as wl

from test_gpu_user import R, _say, check_user, oracle_user, run_users, torch  # noqa: F401  (fixtures)

pytestmark = pytest.mark.gpu


# one user, several, as many as the arguments hold and one more; histories of none, a block and several; users that the resident
# attention does not serve (streamed: no groups) between others; the fp32 kernels, whose loads come eight at a time (ragged widths)
@pytest.mark.parametrize("n_users", [1, 3, 64, 65])
@pytest.mark.parametrize("dtype,d_raw,d,longest", [("bf16", 128, 64, 500), ("bf16", 48, 32, 300), ("bf16", 64, 128, 200), ("bf16", 64, 64, 1500),
                                                   ("bf16", 24, 16, 70), ("f32", 128, 64, 130), ("f32", 12, 8, 65)])
def test_descriptors_in_the_arguments_and_uploaded_give_the_same_bits(R, torch, monkeypatch, dtype, d_raw, d, longest, n_users):  # noqa: F811
    cfg = wl.UserNetConfig("T", 17, dtype, n_users, longest, d_raw, d)
    _say(f"few users {dtype} {d_raw} -> {d}, {n_users} of up to {longest}")
    model = wl.make_user_net_model(cfg, bias_scale=0.05)
    rng = np.random.default_rng(19)
    lens = [longest, 0, longest - 33, *rng.integers(0, longest + 1, n_users)][:n_users]
    users = [wl.make_raw_user(cfg, rng, seq_len=int(l)) for l in lens]
    got, dev, ctx = run_users(R, torch, cfg, model, users)
    assert ctx.aif_user_last_form() == (n_users <= 64)
    ctx.aif_user_precompute([v.req for v in dev[:1]])                   # a smaller call on the same context
    torch.cuda.synchronize()
    assert np.array_equal(R.from_device_f32(dev[0].user_vec), got[0][0])
    monkeypatch.setenv("AIF_USER_UPLOAD", "1")
    ref, _, ctx0 = run_users(R, torch, cfg, model, users)
    assert ctx0.aif_user_last_form() == 0
    for r, (a, b) in enumerate(zip(got, ref)):
        assert np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1]), r
    check_user(dtype, got[0], oracle_user(model, users[0]), d, f"L={lens[0]}")


# the widest rows that a context takes: 160 KB of LDS a block of the projection off the matrix cores
@pytest.mark.parametrize("n_users", [3, 65])
@pytest.mark.parametrize("dtype,d", [("f32", 8), ("bf16", 16)])
def test_few_users_of_the_widest_rows(R, torch, dtype, d, n_users):  # noqa: F811
    cfg = wl.UserNetConfig("T", 17, dtype, n_users, 40, 1280, d)
    _say(f"few users {dtype} 1280 -> {d}, {n_users}")
    model = wl.make_user_net_model(cfg, bias_scale=0.05)
    rng = np.random.default_rng(23)
    users = [wl.make_raw_user(cfg, rng, seq_len=int(l)) for l in [40, 0, 33, *rng.integers(0, 41, n_users)][:n_users]]
    got, _, _ = run_users(R, torch, cfg, model, users)
    for r in range(3):
        check_user(dtype, got[r], oracle_user(model, users[r]), d, f"user {r}")
