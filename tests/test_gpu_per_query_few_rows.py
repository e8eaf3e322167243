"""Per-query norms of windows of few bf16 rows, whose wavefronts take whole tiles in turn: unit lengths at the edges of tiles
and of rounds of four tiles, chunks cut into pieces, cardinalities, causal window, references that rise, marked tokens."""

import numpy as np
import pytest

from workloads import bf16_bits_to_f32, f32_to_bf16_bits, generate_unit

from test_gpu_parity import variant
from test_gpu_per_query import check_sensitivity

pytestmark = pytest.mark.gpu

SHAPES = [(64, 1, 4), (128, 1, 31), (128, 4, 8)]          # 4, 31 and 32 rows


def _bf16(x):
    return bf16_bits_to_f32(f32_to_bf16_bits(np.ascontiguousarray(x, dtype=np.float32)))


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("base", ["llama8b_8k", "stream2560"])         # plain tokens, slots of several tokens
@pytest.mark.parametrize("D,G,W", SHAPES)
def test_norms_of_few_rows(D, G, W, base, causal):
    lens = [32, 33, 62, 63, 64, 65, 125, 129, 257, 1500]
    w = variant(base, dtype="bf16", head_dim=D, group=G, window=W, n_seq=len(lens), n_kv_heads=1)
    if w.mean_count > 0:
        w = w.scaled(fresh_tail=max(W, 8), n_sink=2)
    units = [generate_unit(w, 0, s, 0, n=n) for s, n in enumerate(lens)]
    check_sensitivity(w, units, lens, D, G, W, "bf16", causal)


@pytest.mark.parametrize("D,G,W", SHAPES)
def test_few_rows_of_logits_that_climb(D, G, W):
    """The Keys grow from a thousandth of their size, up to logits of 20: a wavefront's references rise, and at the end the
    four wavefronts of a piece hold different ones."""
    lens = [700, 64, 40]
    w = variant("llama8b_8k", dtype="bf16", head_dim=D, group=G, window=W, n_seq=len(lens), n_kv_heads=1)
    units = [generate_unit(w, 0, s, 0, n=n) for s, n in enumerate(lens)]
    for u in units:
        K = u.K.astype(np.float32) * np.geomspace(1e-3, 1.0, u.n, dtype=np.float32)[:, None]
        e = u.Q.reshape(-1, D).astype(np.float64) @ K.T.astype(np.float64) / np.sqrt(D)
        u.K = _bf16(K * (20.0 / np.abs(e).max()))
    check_sensitivity(w, units, lens, D, G, W, "bf16", False)


@pytest.mark.parametrize("D,G,W", SHAPES)
def test_few_rows_with_marked_tokens(D, G, W):
    """A row's weight on one token, at the ends of tiles of 31, of pieces and of the unit: its norms cancel there."""
    n = 700
    w = variant("llama8b_8k", dtype="bf16", head_dim=D, group=G, window=W, n_seq=1, n_kv_heads=1)
    u = generate_unit(w, 0, 0, 0, n=n)
    Q, K = u.Q.reshape(-1, D).astype(np.float32), u.K.astype(np.float32) * 0.1
    for i, t in enumerate([0, 30, 31, 32, 127, 128, 255, 256, n - 2, n - 1]):
        q = Q[7 * i % len(Q)]
        K[t] = q * (20.0 * np.sqrt(D) / np.dot(q, q))
    u.K = _bf16(K)
    check_sensitivity(w, [u], [n], D, G, W, "bf16", False)
