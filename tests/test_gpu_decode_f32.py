"""fp32 decode attention from five query rows on (matrix cores): against the oracle at the edges of its tiles, and against
the vector-ALU kernel that took these calls before."""

import numpy as np
import pytest

from helpers import DeviceBatch
from test_gpu_parity import check_decode, switch_override, torch_sync, variant
from workloads import generate_unit

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D,G,W,lens,path", [
    (128, 5, 1, [32, 33, 63, 64, 65, 4100], None),       # one tile, one row more, one row less; a chunk of four rows
    (64, 4, 8, [95, 257, 2049], None),                   # a whole block of query rows
    (128, 8, 8, [1000, 20000], None),                    # two blocks
    (64, 3, 11, [300], None),                            # 33 rows: one row in the second block
    (128, 1, 1, [700, 32], "mfma"),
])
@pytest.mark.parametrize("base", ["tiny", "stream2560"])
def test_decode_f32_matches_oracle(base, D, G, W, lens, path):
    w = variant(base, dtype="f32", head_dim=D, group=G, window=W, n_seq=len(lens), n_kv_heads=1)
    w = w.scaled(fresh_tail=8, n_sink=2)
    check_decode([generate_unit(w, 0, s, 0, n=n) for s, n in enumerate(lens)], "f32", D, G, W, path)


@pytest.mark.parametrize("n", [64, 65, 300, 513])
def test_decode_f32_infinite_values_agree_with_the_vector_kernel(n):
    """A Value that is infinite, in a row that a moved-back last tile sees twice and in others."""
    import torch
    w = variant("tiny", dtype="f32", head_dim=128, group=6, window=1, n_seq=1, n_kv_heads=1).scaled(n_sink=2)
    u = generate_unit(w, 0, 0, 0, n=n)
    outs = []
    for path in (1, 2):
        batch = DeviceBatch([u], group=6, window=1, head_dim=128, dtype="f32", n_sink=0, budgets=[n])
        for row, ch in ((n - 33, 3), (n - 30, 7), (0, 11), (n - 1, 90)):
            batch.V[row, ch] = float("inf")
        out = torch.zeros((1, 6, 128), dtype=torch.float32, device="cuda")
        ws = torch.full((batch.kvs.kvs_decode_workspace_size(batch.problem),), 0xFF, dtype=torch.uint8, device="cuda")
        with switch_override("decode_path", path):
            batch.kvs.kvs_decode_attention(batch.problem, batch.Q, batch.K, batch.V, None, out, ws, stream=batch.stream())
            torch_sync()
        outs.append(out.cpu().numpy()[0])
    assert np.isposinf(outs[0][:, [3, 7, 11, 90]]).all()
    finite = np.isfinite(outs[0])
    assert (np.isposinf(outs[1]) == np.isposinf(outs[0])).all() and (np.isnan(outs[1]) == np.isnan(outs[0])).all()
    # two fp32 sums of at most 513 terms in different orders: 513 * 2^-24 of the sum of their magnitudes (unit variance)
    assert np.abs(outs[0][finite] - outs[1][finite]).max() <= 513 * 2.0 ** -24 * 4
