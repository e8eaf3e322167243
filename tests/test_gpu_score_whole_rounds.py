"""Launches whose score chunks are cut for whole rounds of workgroups: one to four rounds, equal units and (above 128 rows)
ragged ones, chunks that end inside a stage of the kernel for more than 128 rows, wavefronts with one and with two blocks of
query rows, one launch per 512 rows.  And launches of few workgroups, whose chunks are shorter than a stage."""

import numpy as np
import pytest

from oracle import kvs_oracle as O

from test_gpu_parity import TOL_ALPHA, switches

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,shortest,longest,D,G,W,dtype,counts,causal", [
    (8, 17001, 17001, 128, 7, 32, "bf16", False, True),       # 224 rows: one round of 512, a wavefront with one block
    (9, 15000, 40000, 64, 5, 39, "bf16", True, False),        # 195 rows, ragged
    (8, 16390, 16390, 128, 8, 64, "bf16", False, False),      # 512 rows: one round of 256
    (3, 30011, 60000, 128, 9, 33, "bf16", True, False),       # 297 rows: eight wavefronts, two of them with two blocks
    (8, 16500, 16500, 64, 5, 106, "bf16", False, True),       # 530 rows: two launches per sweep
    (32, 9000, 9000, 64, 5, 32, "bf16", False, False),        # 160 rows of 64 channels: a round of 256
    (20, 20000, 24000, 128, 6, 32, "bf16", False, True),      # 192 rows, read past the caches, ragged: two rounds of 256
    (90, 12300, 12300, 128, 4, 20, "bf16", True, False),      # 80 rows: several rounds
    (100, 11000, 11000, 64, 3, 1, "bf16", True, False),       # 3 rows: a round of 768
    (64, 4000, 21000, 128, 1, 1, "f32", False, False),        # one row, ragged
    (90, 12000, 12000, 64, 2, 16, "bf16", True, False),       # 32 rows of 64 channels with cardinalities: rounds of 768
    (50, 20000, 24000, 64, 4, 16, "bf16", False, False),      # without, ragged: a round of 1024
    (64, 4111, 4111, 64, 1, 9, "bf16", False, False),         # 9 rows
    (40, 4111, 4111, 128, 2, 17, "f32", False, False),        # fp32, 34 rows
])
def test_score_in_whole_rounds(n, shortest, longest, D, G, W, dtype, counts, causal):
    rng = np.random.default_rng(n * D + G * W)
    lens = [int(x) for x in rng.integers(shortest, longest + 1, n)]
    at_once, total = (256 if G * W > 256 else 512), sum(lens)
    assert total >= at_once * max(256, total // (512 if total <= 1 << 20 else 1024))      # what the rule is for
    check(lens, D, G, W, dtype, counts, causal)


@pytest.mark.parametrize("lens,D,G,W,dtype,counts,causal", [
    ([700, 33, 129, 5000, 64, 1025], 128, 4, 32, "bf16", False, False),      # a tile per wavefront, last chunks of 1 to 127
    ([1000, 513, 4000], 64, 1, 8, "bf16", True, True),
    ([300, 2000, 1], 128, 1, 1, "bf16", False, False),                       # vector kernel
    ([1024, 200, 3333], 64, 2, 4, "f32", True, False),
    ([4000, 65, 129], 128, 5, 32, "bf16", True, False),                      # 160 rows, chunks of 128
    ([2000, 65, 700], 128, 8, 64, "bf16", False, True),                      # 512 rows, chunks of 64
    ([2000, 65, 32, 1999], 128, 4, 32, "f32", False, True),                  # fp32, 128 rows, chunks of 64
    ([6000] * 8, 64, 3, 67, "f32", True, False),                             # fp32, 201 rows, chunks of 192
    ([6100] * 16, 128, 4, 30, "f32", False, False),                          # fp32, a round of 512
])
def test_score_in_short_chunks(lens, D, G, W, dtype, counts, causal):
    check(lens, D, G, W, dtype, counts, causal)


def check(lens, D, G, W, dtype, counts, causal):
    import torch
    import paper_2603_00907_amd as kvs
    n, R = len(lens), G * W
    rows = np.cumsum([0] + [x + 3 for x in lens])
    io = torch.float32 if dtype == "f32" else torch.bfloat16
    p = kvs.Problem(lens=lens, budgets=[2048] * n, group=G, window=W, head_dim=D, dtype=dtype, n_sink=4,
                    in_rows=[int(r) for r in rows[:-1]], causal=causal)
    gen = torch.Generator(device="cuda").manual_seed(n)
    K, V = (torch.randn((int(rows[-1]), D), generator=gen, device="cuda").to(io) for _ in range(2))
    Q = torch.randn((n, R, D), generator=gen, device="cuda").to(io)
    c = torch.randint(1, 20, (int(rows[-1]),), generator=gen, device="cuda", dtype=torch.int32) if counts else None

    def score():
        alpha = torch.full((int(rows[-1]),), -7.0, device="cuda")
        o_bar = torch.full((n, D), -7.0, device="cuda")
        ws = torch.full((kvs.kvs_workspace_size(p),), 0xFF, dtype=torch.uint8, device="cuda")
        kvs.kvs_score_counts(p, Q, K, V, c, alpha, o_bar, ws, stream=torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
        return alpha.cpu().numpy(), o_bar.cpu().numpy()

    got, got_o = score()
    for i, (r0, length) in enumerate(zip(rows[:-1], lens)):
        assert (got[r0 + length:r0 + length + 3] == -7.0).all()          # rows between the units are never touched
        assert abs(got[r0:r0 + length].astype(np.float64).sum() - 1) < TOL_ALPHA, i      # TOL_ALPHA of every term
    for i in {0, n // 2, int(np.argmin(lens)), n - 1}:
        at = slice(rows[i], rows[i] + lens[i])
        k, v = (x[at].float().cpu().numpy() for x in (K, V))
        ci = c[at].cpu().numpy() if counts else None
        ref, ref_o = O.score(Q[i].float().cpu().numpy().reshape(G, W, D), k, v, counts=ci, causal_window=W if causal else 0)
        assert np.max(np.abs(got[at] - ref) / ref) < TOL_ALPHA, i
        values = O.slot_values(v, ci)
        assert (np.abs(got_o[i] - ref_o) <= TOL_ALPHA * (ref @ np.abs(values)) + 1e-7).all(), i
    with switches(score_chunk=640):                                      # chunks of another length: each within its own bar
        other, _ = score()
    seen = got > 0
    assert np.max(np.abs(got - other)[seen] / other[seen]) < 2 * TOL_ALPHA
