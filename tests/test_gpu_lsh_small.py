"""Signature modelling of small calls, three launches, against the launches kept apart, and chunks of short histories against the oracle."""
import numpy as np
import pytest

from test_gpu_lsh import R, din_tolerance, torch  # noqa: F401  (fixtures)

from paper_2511_12934_amd import binding as B

import oracle

pytestmark = pytest.mark.gpu


# one request and several, more than the arguments hold; requests without candidates or history; blocks of 256 candidates and tiles of
# 32 round their edges; histories round a chunk of 128 items, a row tile of 64, and with parts of their own
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("bits,d", [(32, 32), (64, 64), (128, 128), (64, 96)])
@pytest.mark.parametrize("sizes", [[(207, 523)], [(1, 1), (31, 127), (0, 129), (33, 128), (256, 0), (257, 2049), (1495, 1330)],
                                   [(n, 60 + 37 * n) for n in range(1, 19)]])
def test_three_launches_give_the_results_of_seven(R, torch, monkeypatch, dtype, bits, d, sizes):  # noqa: F811
    rng = np.random.default_rng(71)
    t = torch.bfloat16 if dtype == "bf16" else torch.float32
    table = torch.from_numpy(rng.integers(0, 256, (5000, bits // 8), dtype=np.uint8)).cuda()
    users = []
    for n, L in sizes:
        sig = rng.integers(0, 256, (L, bits // 8), dtype=np.uint8)
        ids = rng.integers(0, 5000, n).astype(np.int32)
        if n > 30:
            ids[[0, n - 1]] = [-1, 5000]
            if L > 200:                                     # a history of like items, and candidates unlike them
                sig[:] = sig[0] ^ (rng.random(sig.shape) < 0.02)
                ids[3] = 17
                table[17] = torch.from_numpy(~sig[0]).cuda()
        emb = torch.from_numpy(rng.standard_normal((L, d)).astype(np.float32) * 0.1).to(t)
        users.append((sig, emb, ids))

    forms = []

    def run():
        din = [torch.full((n, d), 7.0, device="cuda") for n, _ in sizes]
        tier = [torch.full((n, 8), 7, dtype=torch.int32, device="cuda") for n, _ in sizes]
        reqs = [B.LshRequest(torch.from_numpy(s).cuda(), e.cuda(), torch.from_numpy(i).cuda(), a, b) for (s, e, i), a, b in zip(users, din, tier)]
        ctx = B.LshContext(sig_table=table, d_out=d, n_tiers=8, dtype=B.AIF_F32 if dtype == "f32" else B.AIF_BF16, max_seq_len=2500,
                           max_candidates=1500, max_users=len(sizes))
        for _ in range(2):
            ctx.aif_lsh_batch(reqs)
            torch.cuda.synchronize()
        forms.append(ctx.aif_lsh_last_form())
        assert ctx.aif_lsh_poll_device_errors() == 2 * 2 * sum(n > 30 for n, _ in sizes)
        return [a.cpu().numpy() for a in din], [b.cpu().numpy() for b in tier]

    din, tier = run()
    monkeypatch.setenv("AIF_LSH_SEPARATE", "1")
    din0, tier0 = run()
    assert forms == [3 if len(sizes) <= 16 else 2, 0]           # the launches that are compared
    for r, (sig, emb, ids) in enumerate(users):
        assert np.array_equal(din[r], din0[r], equal_nan=True) and np.array_equal(tier[r], tier0[r]), r
        if len(ids) == 0 or len(sig) == 0:
            continue
        ok = (ids >= 0) & (ids < 5000)
        ref = oracle.lsh_request(sig_table=table.cpu().numpy(), ids=np.where(ok, ids, 0), seq_sig=sig, u_seq=emb.float().numpy(), n_tiers=8)
        assert np.array_equal(tier[r][ok], ref.tiers[ok]), r
        assert np.all(np.abs(din[r][ok] - ref.din[ok]) <= din_tolerance(emb.float().numpy(), len(sig), bits)), r
