"""The user-side sums of LSH-DIN at the edges of their steps, chunks and shares, against the oracle."""
import numpy as np
import pytest

from paper_2511_12934_amd import workloads as wl

from test_gpu_lsh import R, _say, check, torch  # noqa: F401  (fixtures)

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
