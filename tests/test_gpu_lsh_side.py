"""A call large enough to run LSH-DIN beside SimTier gives the bits of its pieces, on any stream, call after call."""
import numpy as np
import pytest

from paper_2511_12934_amd import workloads as wl

from test_gpu_lsh import R, _say, torch  # noqa: F401  (fixtures)

pytestmark = pytest.mark.gpu


def test_halves_side_by_side_give_the_bits_of_small_calls(R, torch):  # noqa: F811
    cfg = wl.LshConfig("S", 17, "bf16", 1, 10, 5000, 64, 64, 8, 50, n_clusters=16, flip=0.2)
    n, L = 9000, 32_000                                    # 2.9e8 pairs: over the line; a tenth of the list: under it
    _say(f"lsh {n} x {L}, halves side by side")
    rng = np.random.default_rng(11)
    table = torch.from_numpy(wl.make_sig_table_host(cfg)).cuda()
    u, ids = wl.make_lsh_user(cfg, rng, seq_len=L, sigma=1.0), rng.integers(0, cfg.n_items, n).astype(np.int32)
    ctx = R.make_lsh_context(cfg, table, max_users=1, max_candidates=n, max_seq_len=L)
    whole = R.upload_lsh_request(cfg, u, ids)
    parts = [R.slice_lsh_request(whole, lo, lo + n // 10) for lo in range(0, n, n // 10)]
    for p in parts:
        ctx.aif_lsh_batch([p.req])
    torch.cuda.synchronize()
    din, tiers = whole.din.clone(), whole.tiers.clone()
    side = torch.cuda.Stream()
    for stream in (torch.cuda.current_stream(), side, side):
        whole.din.fill_(float("nan"))
        whole.tiers.fill_(-3)
        stream.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(stream):
            ctx.aif_lsh_batch([whole.req])
            a, b = whole.din.clone(), whole.tiers.clone()  # on the caller's stream: both halves have to be in
        stream.synchronize()
        assert torch.equal(a, din) and torch.equal(b, tiers)
