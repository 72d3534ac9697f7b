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
