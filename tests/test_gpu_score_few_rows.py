"""Windows of at most 64 bf16 rows in the wide score kernel: one and two blocks of 32 rows, the pass over V carried along by
sweep 1 or apart, unit lengths at the edges of its tiles, cardinalities, causal window."""

import numpy as np
import pytest

from oracle import kvs_oracle as O

from test_gpu_parity import TOL_ALPHA, switches

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("counts,causal", [(False, False), (True, False), (False, True)])
@pytest.mark.parametrize("D,G,W", [(64, 1, 4), (128, 1, 31), (128, 4, 8), (64, 3, 11), (128, 4, 16)])
@pytest.mark.parametrize("ride", [1, 2])                              # never, always
def test_score_of_few_rows(D, G, W, counts, causal, ride):
    import torch
    import paper_2603_00907_amd as kvs
    lens = [32, 33, 63, 65, 257, 1023, 2049]
    n, R = len(lens), G * W
    rows = np.cumsum([0] + [x + 3 for x in lens])
    p = kvs.Problem(lens=lens, budgets=[x // 2 + 5 for x in lens], group=G, window=W, head_dim=D, dtype="bf16", n_sink=4,
                    in_rows=[int(r) for r in rows[:-1]], causal=causal)
    gen = torch.Generator(device="cuda").manual_seed(R + D)
    K, V = (torch.randn((int(rows[-1]), D), generator=gen, device="cuda").to(torch.bfloat16) for _ in range(2))
    Q = torch.randn((n, R, D), generator=gen, device="cuda").to(torch.bfloat16)
    c = torch.randint(1, 5000, (int(rows[-1]),), generator=gen, device="cuda", dtype=torch.int32) if counts else None
    alpha = torch.full((int(rows[-1]),), -7.0, device="cuda")
    o_bar = torch.full((n, D), -7.0, device="cuda")
    ws = torch.full((kvs.kvs_workspace_size(p),), 0xFF, dtype=torch.uint8, device="cuda")
    with switches(fuse_obar=ride):
        kvs.kvs_score_counts(p, Q, K, V, c, alpha, o_bar, ws, stream=torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
    got, got_o = alpha.cpu().numpy(), o_bar.cpu().numpy()
    for i, (r0, length) in enumerate(zip(rows[:-1], lens)):
        assert (got[r0 + length:r0 + length + 3] == -7.0).all()
        at = slice(r0, r0 + length)
        k, v = (x[at].float().cpu().numpy() for x in (K, V))
        ci = c[at].cpu().numpy() if counts else None
        ref, ref_o = O.score(Q[i].float().cpu().numpy().reshape(G, W, D), k, v, counts=ci, causal_window=W if causal else 0)
        assert np.max(np.abs(got[at] - ref) / ref) < TOL_ALPHA, i
        values = O.slot_values(v, ci)
        assert (np.abs(got_o[i] - ref_o) <= TOL_ALPHA * (ref @ np.abs(values)) + 1e-7).all(), i


@pytest.mark.parametrize("G,W,counts,causal", [(1, 16, False, False), (4, 8, True, True), (4, 16, False, True)])
def test_score_of_few_rows_past_the_caches(G, W, counts, causal):
    """128 channels, K and V above 192 MB: read past the caches, the pass over V carried along by sweep 1."""
    import torch
    import paper_2603_00907_amd as kvs
    lens, D = [32000 - 777 * i for i in range(18)], 128
    n, R = len(lens), G * W
    rows = np.cumsum([0] + lens)
    assert 4 * int(rows[-1]) * D > 192 << 20
    p = kvs.Problem(lens=lens, budgets=[2048] * n, group=G, window=W, head_dim=D, dtype="bf16", n_sink=4, causal=causal)
    gen = torch.Generator(device="cuda").manual_seed(R)
    K, V = (torch.randn((int(rows[-1]), D), generator=gen, device="cuda").to(torch.bfloat16) for _ in range(2))
    Q = torch.randn((n, R, D), generator=gen, device="cuda").to(torch.bfloat16)
    c = torch.randint(1, 50, (int(rows[-1]),), generator=gen, device="cuda", dtype=torch.int32) if counts else None
    alpha = torch.full((int(rows[-1]),), -7.0, device="cuda")
    o_bar = torch.full((n, D), -7.0, device="cuda")
    ws = torch.full((kvs.kvs_workspace_size(p),), 0xFF, dtype=torch.uint8, device="cuda")
    kvs.kvs_score_counts(p, Q, K, V, c, alpha, o_bar, ws, stream=torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    got, got_o = alpha.cpu().numpy(), o_bar.cpu().numpy()
    for i in range(n):
        assert abs(got[rows[i]:rows[i + 1]].astype(np.float64).sum() - 1) < TOL_ALPHA, i      # TOL_ALPHA of every term
    for i in (0, 9, n - 1):
        at = slice(rows[i], rows[i + 1])
        k, v = (x[at].float().cpu().numpy() for x in (K, V))
        ci = c[at].cpu().numpy() if counts else None
        ref, ref_o = O.score(Q[i].float().cpu().numpy().reshape(G, W, D), k, v, counts=ci, causal_window=W if causal else 0)
        assert np.max(np.abs(got[at] - ref) / ref) < TOL_ALPHA, i
        values = O.slot_values(v, ci)
        assert (np.abs(got_o[i] - ref_o) <= TOL_ALPHA * (ref @ np.abs(values)) + 1e-7).all(), i
