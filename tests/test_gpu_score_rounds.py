"""Launches of ragged units whose score chunks are lengthened so that the last round of workgroups is not nearly empty (65 to
128 bf16 rows): every token is scored once, in one launch group and in two with chunk lengths of their own."""

import numpy as np
import pytest

from oracle import kvs_oracle as O

from test_gpu_parity import TOL_ALPHA

pytestmark = pytest.mark.gpu


def workgroups(lens, want):
    return sum(-(-n // (-(-max(want, -(-n // 64)) // 64) * 64)) for n in lens)


@pytest.mark.parametrize("n,longest,D,G,W,seed", [
    (64, 32768, 64, 3, 22, 2),                                          # 66 rows, 1049 workgroups
    (64, 32768, 128, 4, 32, 24),                                    # 128 rows, 1033 workgroups
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
