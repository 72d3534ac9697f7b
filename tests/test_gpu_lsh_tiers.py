"""SimTier with two history items a cell: every pair of equal-bit counts at the tiers' edges, tile remainders, every width
and tier count the matrix-core kernel serves.  Counts are whole numbers: equal to the oracle's."""
import numpy as np
import pytest

from paper_2511_12934_amd import workloads as wl

from test_gpu_lsh import R, _say, check, torch  # noqa: F401  (fixtures)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d_bits,n_tiers", [(32, 1), (32, 2), (32, 8), (64, 2), (64, 4), (64, 8), (128, 1), (128, 2), (128, 4), (128, 8)])
def test_counts_at_tier_edges_beside_every_neighbour(R, torch, d_bits, n_tiers):  # noqa: F811
    cfg = wl.LshConfig("S", 15, "bf16", 1, 10, 300, d_bits, 32, n_tiers, 50, n_clusters=4, flip=0.3)
    _say(f"lsh tiers d'={d_bits} N={n_tiers}")
    table = wl.make_sig_table_host(cfg)
    rng = np.random.default_rng(d_bits + n_tiers)
    base = np.unpackbits(table[0])
    users_ids = []
    for L in (1, 31, 33, 63, 64, 65, 127, 256, 257, 64 * 9 + 40, 40_000):
        u = wl.make_lsh_user(cfg, rng, seq_len=L, sigma=1.0)
        for t in range(L):                                     # equal bits with candidate 0: 0, all, and around the edges of tiers
            w = d_bits // n_tiers
            e = int(rng.choice([0, d_bits, d_bits - 1, 1, w * int(rng.integers(0, n_tiers + 1)), max(0, w * int(rng.integers(0, n_tiers + 1)) - 1)]))
            bits = base.copy()
            bits[rng.permutation(d_bits)[:d_bits - e]] ^= 1
            u.seq_sigs[t] = np.packbits(bits)
            if t >= 2000:                                      # a long history repeats
                u.seq_sigs[2000:] = np.resize(u.seq_sigs[:2000], (L - 2000, d_bits // 8))
                break
        users_ids.append((u, np.arange(70, dtype=np.int32)))
    ctx, _ = check(R, torch, cfg, table, users_ids)
    assert ctx.aif_lsh_simtier_kind() == 1


# a wave's share past the passes that its counters hold (30 of 256 items, 62 for 128 bits; 16 parts of two waves), even and
# odd numbers of passes, ragged ends; three items of four in ONE tier, so that the counters come close to full
@pytest.mark.parametrize("d_bits,passes", [(64, 30), (64, 31), (32, 62), (128, 62), (128, 63)])
def test_counts_of_histories_longer_than_the_counters_hold(R, torch, d_bits, passes):  # noqa: F811
    L = 32 * passes * 256 + 32 * 100 + 37
    cfg = wl.LshConfig("S", 16, "bf16", 1, 10, 300, d_bits, 32, 8, 50, n_clusters=4, flip=0.3)
    _say(f"lsh tiers d'={d_bits} L={L}")
    table = wl.make_sig_table_host(cfg)
    rng = np.random.default_rng(d_bits + passes)
    u = wl.make_lsh_user(cfg, rng, seq_len=1000, sigma=1.0)
    half = np.packbits(np.concatenate([np.ones(d_bits // 2, np.uint8), np.zeros(d_bits // 2, np.uint8)]))
    u.seq_sigs[np.arange(1000) % 4 != 0] = table[0] ^ half
    u.seq_sigs, u.seq_emb = np.resize(u.seq_sigs, (L, d_bits // 8)), np.resize(u.seq_emb, (L, u.seq_emb.shape[1]))
    ctx, _ = check(R, torch, cfg, table, [(u, np.array([0, 1, 2, 299], np.int32))])
    assert ctx.aif_lsh_simtier_kind() == 1
