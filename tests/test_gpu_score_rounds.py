"""Launches whose score chunks are lengthened so that the last round of workgroups is not nearly empty (4 to 128 bf16 rows), ragged
units by up to a quarter and equal ones to whole rounds: every token is scored once, in one launch group and in two with chunk
lengths of their own, with cardinalities and in the per-query kernels."""

import numpy as np
import pytest

from oracle import kvs_oracle as O

from test_gpu_parity import TOL_ALPHA, switches
from test_gpu_score_whole_rounds import check

pytestmark = pytest.mark.gpu


def workgroups(lens, want):
    return sum(-(-n // (-(-max(want, -(-n // 64)) // 64) * 64)) for n in lens)


@pytest.mark.parametrize("n,longest,D,G,W,seed", [
    (64, 32768, 64, 3, 22, 2),                                          # 66 rows, 1049 workgroups
    (64, 32768, 128, 4, 32, 24),                                    # 128 rows, 1033 workgroups
    (64, 32768, 128, 1, 32, 24),                                    # 32 rows
    (80, 65536, 64, 4, 32, 3),                                          # a group of 64 units (1045 workgroups) and one of 16
])
def test_score_with_longer_chunks(n, longest, D, G, W, seed):
    import torch
    import paper_2603_00907_amd as kvs
    rng = np.random.default_rng(seed)
    lens = [int(x) for x in rng.integers(4096, longest, n)]
    first = lens[:64]
    want = min(sum(lens) // 1024, 2048)
    assert sum(lens) > 1 << 20 and 0 < workgroups(first, want) % 512 <= 128     # what the rule is for
    rows = np.cumsum([0] + [x + 3 for x in lens])
    p = kvs.Problem(lens=lens, budgets=[2048] * n, group=G, window=W, head_dim=D, dtype="bf16", n_sink=4,
                    in_rows=[int(r) for r in rows[:-1]])
    gen = torch.Generator(device="cuda").manual_seed(seed)
    K, V = (torch.randn((int(rows[-1]), D), generator=gen, device="cuda").to(torch.bfloat16) for _ in range(2))
    Q = torch.randn((n, G * W, D), generator=gen, device="cuda").to(torch.bfloat16)
    alpha = torch.full((int(rows[-1]),), -7.0, device="cuda")
    o_bar = torch.full((n, D), -7.0, device="cuda")
    ws = torch.full((kvs.kvs_workspace_size(p),), 0xFF, dtype=torch.uint8, device="cuda")
    kvs.kvs_score(p, Q, K, V, alpha, o_bar, ws, stream=torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    got, got_o = alpha.cpu().numpy(), o_bar.cpu().numpy()
    for i, (r0, length) in enumerate(zip(rows[:-1], lens)):
        assert (got[r0 + length:r0 + length + 3] == -7.0).all()         # rows between the units are never touched
        assert (got[r0:r0 + length] > 0).all(), i
        assert abs(got[r0:r0 + length].astype(np.float64).sum() - 1) < TOL_ALPHA, i     # TOL_ALPHA of every term
    for i in {0, int(np.argmin(lens)), int(np.argmax(first)), min(63, n - 1), n - 1}:
        k, v = (x[rows[i]:rows[i] + lens[i]].float().cpu().numpy() for x in (K, V))
        ref, ref_o = O.score(Q[i].float().cpu().numpy().reshape(G, W, D), k, v)
        assert np.max(np.abs(got[rows[i]:rows[i] + lens[i]] - ref) / ref) < TOL_ALPHA, i
        assert (np.abs(got_o[i] - ref_o) <= TOL_ALPHA * (ref @ np.abs(v)) + 1e-7).all(), i


@pytest.mark.parametrize("G,W,counts,causal", [(1, 4, False, True), (4, 32, True, False)])
def test_score_with_longer_chunks_in_one_round(G, W, counts, causal):
    """520 chunks of 1024 tokens become 463 of 1152; V is carried along by sweep 1."""
    check([20000 + 640 * i for i in range(20)], 128, G, W, "bf16", counts, causal)


@pytest.mark.parametrize("counts", [False, True])
@pytest.mark.parametrize("D,G,W", [(64, 3, 22), (128, 4, 32)])
def test_equal_units_with_longer_chunks(D, G, W, counts):
    """100 units of 11000 tokens: 1100 chunks of 1088 tokens become 500 of 2304, one round, or of 2240 for the per-query
    kernels (tests/host/abi_driver.cpp asks the library for its numbers)."""
    import torch
    import paper_2603_00907_amd as kvs
    n, length = 100, 11000
    want = n * length // 1024
    assert n * length > 1 << 20 and workgroups([length] * n, want) == 1100
    assert workgroups([length] * n, 2304) == workgroups([length] * n, 2240) == 500 <= 512
    p = kvs.Problem(lens=[length] * n, budgets=[2048] * n, group=G, window=W, head_dim=D, dtype="bf16", n_sink=4)
    gen = torch.Generator(device="cuda").manual_seed(D)
    K, V = (torch.randn((n * length, D), generator=gen, device="cuda").to(torch.bfloat16) for _ in range(2))
    Q = torch.randn((n, G * W, D), generator=gen, device="cuda").to(torch.bfloat16)
    c = torch.randint(1, 20, (n * length,), generator=gen, device="cuda", dtype=torch.int32) if counts else None
    s = torch.cuda.current_stream().cuda_stream

    def calls():
        ws = torch.full((kvs.kvs_per_query_workspace_size(p),), 0xFF, dtype=torch.uint8, device="cuda")
        out = [torch.full((n * length,), -7.0, device="cuda") for _ in range(4)] + [torch.full((n, D), -7.0, device="cuda")]
        if counts:
            kvs.kvs_score_counts(p, Q, K, V, c, out[0], out[4], ws, stream=s)
            kvs.kvs_sensitivity_counts(p, Q, K, V, c, out[1], out[2], out[3], ws, stream=s)
        else:
            kvs.kvs_score(p, Q, K, V, out[0], out[4], ws, stream=s)
            kvs.kvs_sensitivity(p, Q, K, V, out[1], out[2], out[3], ws, stream=s)
        torch.cuda.synchronize()
        return [x.cpu().numpy() for x in out]

    alpha, alpha_pq, a_tok, c_edge, o_bar = calls()
    for i in (0, 63, 64, n - 1):
        rows = slice(i * length, (i + 1) * length)
        ref, ref_o = O.score(Q[i].float().cpu().numpy().reshape(G, W, D), K[rows].float().cpu().numpy(),
                             V[rows].float().cpu().numpy(), counts=c[rows].cpu().numpy() if counts else None)
        assert np.max(np.abs(alpha[rows] - ref) / ref) < TOL_ALPHA, i
        assert np.max(np.abs(alpha_pq[rows] - ref) / ref) < TOL_ALPHA, i
        values = O.slot_values(V[rows].float().cpu().numpy(), c[rows].cpu().numpy() if counts else None)
        assert (np.abs(o_bar[i] - ref_o) <= TOL_ALPHA * (ref @ np.abs(values)) + 1e-7).all(), i
    with switches(score_chunk=want):                                    # the same calls without the rule
        plain = calls()
    # (each within its own bar, TOL_ALPHA or test_gpu_per_query's TOL_NORMS: no row concentrates on these inputs)
    for got, other, tol in ((alpha, plain[0], TOL_ALPHA), (alpha_pq, plain[1], TOL_ALPHA), (a_tok, plain[2], 5e-5)):
        assert np.max(np.abs(got - other) / other) < 2 * tol
    inner = np.arange(n * length) % length != length - 1                # (a unit's last token has no edge)
    assert (c_edge[~inner] == 0).all()
    assert np.max(np.abs(c_edge - plain[3])[inner] / plain[3][inner]) < 2 * 5e-5


def test_launches_that_hold_units_of_two_groups():
    """164 units of 21000 tokens are planned as groups of 100, with chunks of 2176 tokens, and 64, with chunks of 2688; with the
    selection spread on request, launches take 64 units each, and one of them has units of both: the same edges, the same
    sums of Values."""
    import torch
    import paper_2603_00907_amd as kvs
    n, length, D = 164, 21000, 64
    assert workgroups([length] * 100, 2176) == 1000 and workgroups([length] * 64, 2688) == 512
    p = kvs.Problem(lens=[length] * n, budgets=[5000] * n, group=3, window=22, head_dim=D, dtype="bf16", n_sink=4)
    gen = torch.Generator(device="cuda").manual_seed(7)
    K, V = (torch.randn((n * length, D), generator=gen, device="cuda").to(torch.bfloat16) for _ in range(2))
    Q = torch.randn((n, 66, D), generator=gen, device="cuda").to(torch.bfloat16)

    def step():
        ws = torch.full((kvs.kvs_workspace_size(p),), 0xFF, dtype=torch.uint8, device="cuda")
        Ko, Vo = (torch.full((p.rows_out, D), -7.0, dtype=torch.bfloat16, device="cuda") for _ in range(2))
        co = torch.full((p.rows_out,), -7, dtype=torch.int32, device="cuda")
        slot = torch.full((n * length,), -7, dtype=torch.int32, device="cuda")
        kvs.kvs_step(p, Q, K, V, Ko, Vo, co, ws, slot_of_token_out=slot, stream=torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
        return slot, co, Vo, Ko

    ref = step()
    assert (ref[1].view(n, -1).sum(dim=1) == length).all()
    with switches(select_split=2):
        got = step()
    assert all(torch.equal(a, b) for a, b in zip(got[:3], ref[:3]))
    off = (got[3].float() - ref[3].float()).norm(dim=1) / ref[3].float().norm(dim=1)     # (o_bar's partials are others)
    assert off.max() < 1e-2
