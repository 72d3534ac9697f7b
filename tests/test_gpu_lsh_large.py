"""Signature modelling of a large call, whose halves run side by side, against its requests alone, in the three launches of a small one or
(widths off the matrix cores) apart: the same bits, in a context of few users, whose chunks are short, and in one of more."""
import numpy as np
import pytest

from test_gpu_lsh import R, torch  # noqa: F401  (fixtures)

from paper_2511_12934_amd import binding as B

pytestmark = pytest.mark.gpu

# histories of no, one and several chunks of 128 to 1,024 items, their last one short or full; more than ten
LENS = (0, 1, 127, 128, 129, 640, 1000, 1024, 1025, 1280, 1281, 1330, 2049, 3000, 4100, 5120, 5121, 6000, 9000, 10_241)
N = 6000                                                   # 3e8 pairs together: over the line


@pytest.mark.parametrize("users", [16, 20])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("bits,d", [(32, 32), (64, 64), (64, 16), (128, 128), (96, 48), (256, 96)])
def test_a_large_call_gives_the_bits_of_its_requests(R, torch, dtype, bits, d, users):  # noqa: F811
    rng = np.random.default_rng(89)
    t = torch.bfloat16 if dtype == "bf16" else torch.float32
    table = torch.from_numpy(rng.integers(0, 256, (5000, bits // 8), dtype=np.uint8)).cuda()
    reqs, outs = [], []
    lens = (0, *LENS[1 - users:]) if users < len(LENS) else LENS
    for i, L in enumerate(lens):
        sig = rng.integers(0, 256, (L, bits // 8), dtype=np.uint8)
        if i % 2 and L:                                    # a history of like items, and a candidate unlike them
            sig[:] = sig[0] ^ (rng.random(sig.shape) < 0.02)
            table[i] = torch.from_numpy(~sig[0]).cuda()
        ids = rng.integers(0, 5000, N).astype(np.int32)
        ids[:users] = np.arange(users)
        emb = torch.from_numpy(rng.standard_normal((L, d)).astype(np.float32) * 0.1).to(t)
        outs.append((torch.full((N, d), 7.0, device="cuda"), torch.full((N, 8), 7, dtype=torch.int32, device="cuda")))
        reqs.append(B.LshRequest(torch.from_numpy(sig).cuda(), emb.cuda(), torch.from_numpy(ids).cuda(), *outs[-1]))
    ctx = B.LshContext(sig_table=table, d_out=d, n_tiers=8, dtype=B.AIF_F32 if dtype == "f32" else B.AIF_BF16, max_seq_len=max(lens),
                       max_candidates=N, max_users=users)
    ctx.aif_lsh_batch(reqs)
    torch.cuda.synchronize()
    assert ctx.aif_lsh_last_form() == 1
    whole = [(a.clone(), b.clone()) for a, b in outs]
    for r, (a, b) in enumerate(outs):
        a.fill_(7.0)
        b.fill_(7)
        ctx.aif_lsh_batch([reqs[r]])
        torch.cuda.synchronize()
        assert ctx.aif_lsh_last_form() == (3 if ctx.aif_lsh_simtier_kind() == ctx.aif_lsh_din_kind() == 1 else 0)
        assert torch.equal(a, whole[r][0]) and torch.equal(b, whole[r][1]), lens[r]
