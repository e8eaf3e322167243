"""Per-query norms of windows of few bf16 rows, whose wavefronts take whole tiles in turn: unit lengths at the edges of tiles
and of rounds of four tiles, chunks cut into pieces, cardinalities, causal window, references that rise, marked tokens."""

import numpy as np
import pytest

from workloads import bf16_bits_to_f32, f32_to_bf16_bits, generate_unit

from test_gpu_parity import variant
from test_gpu_per_query import check_sensitivity, check_unit_norms

pytestmark = pytest.mark.gpu

SHAPES = [(64, 1, 4), (128, 1, 31), (128, 4, 8), (64, 3, 11), (128, 4, 16)]          # 4, 31, 32, 33 and 64 rows


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


@pytest.mark.parametrize("base", ["llama8b_8k", "stream2560"])
@pytest.mark.parametrize("D,G,W", [(128, 1, 9), (128, 1, 31), (128, 4, 8)])
def test_norms_of_few_rows_in_a_larger_launch(D, G, W, base):
    """Above 8192 tokens windows of 9 to 32 rows of 128 channels have the outputs' kernel whose wavefronts take whole tiles, too."""
    lens = [33, 127, 257, 1500, 6500]
    w = variant(base, dtype="bf16", head_dim=D, group=G, window=W, n_seq=len(lens), n_kv_heads=1)
    if w.mean_count > 0:
        w = w.scaled(fresh_tail=max(W, 8), n_sink=2)
    units = [generate_unit(w, 0, s, 0, n=n) for s, n in enumerate(lens)]
    check_sensitivity(w, units, lens, D, G, W, "bf16", False)


@pytest.mark.parametrize("lens", [[700, 64, 40], [8000, 700, 64]])
@pytest.mark.parametrize("D,G,W", SHAPES)
def test_few_rows_of_logits_that_climb(D, G, W, lens):
    """The Keys grow from a thousandth of their size, up to logits of 20: a wavefront's references rise, and at the end the
    four wavefronts of a piece hold different ones."""
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


@pytest.mark.parametrize("base,causal,marked", [
    ("llama8b_8k", False, False), ("llama8b_8k", True, True), ("stream2560", False, True), ("stream2560", True, False)])
def test_norms_of_64_rows_over_many_tokens(base, causal, marked):
    """128 channels and 33 to 64 rows: only launches of 262144 tokens or more have the norms' kernel for them.  Units that are
    alike, two of them against the oracle and all of them against each other; marked: a row's weight on one token, at the ends
    of tiles and of the unit, so that its norms cancel there."""
    import torch
    import paper_2603_00907_amd as kvs
    n, copies, D, G, W = 2050, 128, 128, 3, 13
    w = variant(base, dtype="bf16", head_dim=D, group=G, window=W, n_seq=2, n_kv_heads=1)
    u = [generate_unit(w, 0, s, 0, n=n) for s in range(2)]
    for x in u if marked else []:
        q, K = x.Q.reshape(-1, D).astype(np.float32), x.K.astype(np.float32) * 0.1
        for i, t in enumerate([0, 30, 31, 61, 62, 92, 93, 128, 1023, n - 2, n - 1]):
            r = len(q) - 1 if t >= n - 2 else 7 * i % len(q)            # (the last row sees all tokens)
            K[t] = q[r] * (20.0 * np.sqrt(D) / np.dot(q[r], q[r]))
        x.K = _bf16(K)
    Q, K, V = (torch.from_numpy(np.stack([getattr(x, f).astype(np.float32).reshape(-1, D) for x in u])).to("cuda", torch.bfloat16)
               .repeat(copies // 2, 1, 1) for f in "QKV")
    c = None
    if u[0].counts is not None:
        c = torch.from_numpy(np.stack([x.counts for x in u])).to("cuda", torch.int32).repeat(copies // 2, 1)
    p = kvs.Problem(lens=[n] * copies, budgets=[n // 2] * copies, group=G, window=W, head_dim=D, dtype="bf16", causal=causal)
    assert p.rows_in >= 1 << 18
    alpha, a_tok, c_edge = (torch.full((copies, n), -7.0, device="cuda") for _ in range(3))
    ws = torch.full((kvs.kvs_per_query_workspace_size(p),), 0xFF, dtype=torch.uint8, device="cuda")
    kvs.kvs_sensitivity_counts(p, Q, K, V, c, alpha, a_tok, c_edge, ws, stream=torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    for x in (alpha, a_tok, c_edge):
        assert torch.equal(x.view(copies // 2, 2, n), x[:2].expand(copies // 2, 2, n))
    for i in range(2):
        check_unit_norms(u[i], D, W if causal else 0, *(x[i].cpu().numpy().astype(np.float64) for x in (alpha, a_tok)),
                         c_edge[i, :-1].cpu().numpy().astype(np.float64), i)
