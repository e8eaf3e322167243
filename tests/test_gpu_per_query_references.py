"""Per-query norms whose kernels keep a reference of their own for every row and piece of a chunk: logits that climb far
above the first tile's (the sums and partial outputs so far are brought to a higher reference), rows that a causal window
hides from a whole piece, pieces that are empty or a single tile, and marked tokens at the ends of pieces."""

import numpy as np
import pytest

from workloads import bf16_bits_to_f32, f32_to_bf16_bits, generate_unit

from test_gpu_parity import variant
from test_gpu_per_query import check_sensitivity

pytestmark = pytest.mark.gpu


def _bf16(x):
    return bf16_bits_to_f32(f32_to_bf16_bits(np.ascontiguousarray(x, dtype=np.float32)))


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("D,G,W,lens", [
    (128, 4, 32, [3000, 64]),       # one pass of rows, chunks of several tiles
    (64, 3, 11, [700, 33]),         # 33 rows: a wavefront of one row
    (128, 7, 32, [1500]),           # 224 rows: two passes
])
def test_sensitivity_of_logits_that_climb(D, G, W, lens, causal):
    """The Keys grow from a thousandth of their size, up to logits of 20 (29 in base 2; a reference reaches 16 above the tile
    that it is set by, so it has to rise; the suite's bars are for logits up to 20)."""
    w = variant("llama8b_8k", dtype="bf16", head_dim=D, group=G, window=W, n_seq=len(lens), n_kv_heads=1)
    units = [generate_unit(w, 0, s, 0, n=n) for s, n in enumerate(lens)]
    for u in units:
        K = u.K.astype(np.float32) * np.geomspace(1e-3, 1.0, u.n, dtype=np.float32)[:, None]
        e = u.Q.reshape(-1, D).astype(np.float64) @ K.T.astype(np.float64) / np.sqrt(D)
        u.K = _bf16(K * (20.0 / np.abs(e).max()))
    check_sensitivity(w, units, lens, D, G, W, "bf16", causal)


def test_sensitivity_of_marked_tokens_at_the_ends_of_pieces():
    """Values that repeat around every multiple of 128 (the shortest piece) and at the unit's ends: with a row's weight on
    such a token its norms cancel, and the token, or the one before it, lies in another workgroup's piece."""
    D, G, W, n = 128, 4, 32, 1300
    w = variant("llama8b_8k", dtype="bf16", head_dim=D, group=G, window=W, n_seq=1, n_kv_heads=1)
    u = generate_unit(w, 0, 0, 0, n=n)
    Q, K = u.Q.reshape(-1, D).astype(np.float32), u.K.astype(np.float32) * 0.1
    for i, t in enumerate([0, 127, 128, 255, 256, 511, 512, 1023, 1024, n - 2, n - 1]):
        q = Q[7 * i % len(Q)]
        K[t] = q * (20.0 * np.sqrt(D) / np.dot(q, q))          # this row's logit of the token is 20, its other ones are small
    u.K = _bf16(K)
    check_sensitivity(w, [u], [n], D, G, W, "bf16", False)
