"""The user-side sums of LSH-DIN at the edges of their steps, chunks and shares, against the oracle."""
import numpy as np
import pytest

from paper_2511_12934_amd import workloads as wl

from test_gpu_lsh import R, _say, check, din_tolerance, torch  # noqa: F401  (fixtures)

pytestmark = pytest.mark.gpu


# steps of 16 items, 64 signatures at a time, chunks of 1,024, even shares of a history of more than 64 chunks (65,536)
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("d_bits,d_out,lens", [(64, 64, (1, 15, 63, 1023, 1024, 1025, 2049)), (32, 128, (31, 65, 4097)),
                                               (256, 48, (17, 1041)), (128, 32, (65_536, 65_537, 70_001))])
def test_user_sums_at_chunk_edges(R, torch, dtype, d_bits, d_out, lens):  # noqa: F811
    cfg = wl.LshConfig("S", 14, dtype, 1, 10, 2000, d_bits, d_out, 8, 50, n_clusters=16, flip=0.2)
    _say(f"lsh user sums {dtype} d'={d_bits} d={d_out} L={lens}")
    table = wl.make_sig_table_host(cfg)
    rng = np.random.default_rng(8)
    check(R, torch, cfg, table, [(wl.make_lsh_user(cfg, rng, seq_len=L, sigma=1.0), rng.integers(0, cfg.n_items, 40).astype(np.int32)) for L in lens])


SIZES = [(64, 64), (128, 128), (32, 16), (96, 48), (256, 256), (160, 32)]       # both kernels of the candidates' side


def serve(R, torch, cfg, sigs, emb, cands):
    ctx = R.make_lsh_context(cfg, torch.from_numpy(cands).cuda(), max_users=1, max_candidates=len(cands), max_seq_len=len(sigs))
    d = R.upload_lsh_request(cfg, wl.LshUser(sigs, emb), np.arange(len(cands), dtype=np.int32))
    ctx.aif_lsh_batch([d.req])
    torch.cuda.synchronize()
    return d.din.cpu().numpy()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("d_bits,d_out", SIZES)
def test_a_signature_opposite_to_the_whole_history_gets_zero(R, torch, dtype, d_bits, d_out):  # noqa: F811
    """No place matches: Eq. 8 is a sum of zeros, whatever the embeddings."""
    cfg = wl.LshConfig("S", 18, dtype, 1, 10, 2, d_bits, d_out, 1, 50)
    rng = np.random.default_rng(9)
    for L in (1, 7, 64, 2500):
        sig = rng.integers(0, 256, d_bits // 8).astype(np.uint8)
        emb = wl.round_storage(rng.standard_normal((L, d_out)).astype(np.float32) + 0.3, dtype)
        din = serve(R, torch, cfg, np.tile(sig, (L, 1)), emb, np.stack([~sig, sig]))
        worst = float(np.abs(din[0]).max())
        assert worst == 0.0, L
        used = float((np.abs(din[1] - emb.astype(np.float64).sum(0)) / din_tolerance(emb, L, d_bits)).max())
        assert used <= 1, (L, used)                            # the signature itself: the sum of all


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("mean", [0.0, 1.0])
@pytest.mark.parametrize("d_bits,d_out", SIZES)
def test_dissimilar_candidates_keep_fp32_precision(R, torch, dtype, mean, d_bits, d_out):  # noqa: F811
    """A history within 2 % of a prototype, candidates that have the prototype's bit in a share p of their places, p from 0
    to 1: the error is measured against the result itself, small as it is where p is.  Bound, of 2-norms: the roundings
    counted in din_tolerance, 64 steps of a share and d' bits, independent, each of rms 2^-24 / sqrt(3) of a sum no larger
    than the result's terms, of which none cancels: sqrt(64 + d') 2^-24 / sqrt(3)."""
    cfg = wl.LshConfig("S", 19, dtype, 1, 10, 2, d_bits, d_out, 1, 50)
    rng = np.random.default_rng(d_bits)
    L, proto = 2000, rng.integers(0, 2, d_bits).astype(np.uint8)
    hist = proto ^ (rng.random((L, d_bits)) < 0.02).astype(np.uint8)
    shares = (0.0, 0.01, 0.05, 0.15, 0.28, 0.31, 0.34, 0.5, 1.0)
    cands = np.concatenate([(1 - proto) ^ (rng.random((32, d_bits)) < p).astype(np.uint8) for p in shares])
    emb = wl.round_storage((0.1 * rng.standard_normal((L, d_out)) + mean).astype(np.float32), dtype)
    din = serve(R, torch, cfg, np.packbits(hist, axis=1), emb, np.packbits(cands, axis=1))
    ref = (cands[:, None, :] == hist[None]).mean(2) @ emb.astype(np.float64)
    for i, p in enumerate(shares):
        rows = slice(32 * i, 32 * i + 32)
        err = np.linalg.norm(din[rows] - ref[rows]) / np.linalg.norm(ref[rows])
        assert err <= np.sqrt((64 + d_bits) / 3) * 2.0 ** -24, (p, err)
