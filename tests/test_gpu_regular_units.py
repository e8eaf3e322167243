"""Units of one length at equal distances (a kernel forms their descriptors from the first two): the same results as the same
units in an order that is not regular, in groups of every table size, with rows between the units and steps of every sign."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def run(call, dtype, lens, in_rows, out_rows, Q, K, V, budget, counts=None, window=4):
    import torch
    import paper_2603_00907_amd as kvs
    n = len(lens)
    p = kvs.Problem(lens=lens, budgets=[budget] * n, group=2, window=window, head_dim=64, dtype=dtype, n_sink=4,
                    in_rows=in_rows, out_rows=out_rows)
    s = torch.cuda.current_stream().cuda_stream
    if call == "decode":
        ws = torch.full((kvs.kvs_decode_workspace_size(p),), 0xFF, dtype=torch.uint8, device="cuda")
        out = torch.zeros((n, 2 * window, 64), device="cuda")
        kvs.kvs_decode_attention(p, Q, K, V, counts, out, ws, stream=s)
        torch.cuda.synchronize()
        return [out[i].cpu().numpy() for i in range(n)]
    size = kvs.kvs_per_query_workspace_size if call == "per_query" else kvs.kvs_workspace_size
    ws = torch.full((size(p),), 0xFF, dtype=torch.uint8, device="cuda")
    Ko = torch.full((p.rows_out + 3, 64), -7.0, dtype=K.dtype, device="cuda")
    Vo = torch.full_like(Ko, -7.0)
    co = torch.full((p.rows_out + 3,), -7, dtype=torch.int32, device="cuda")
    if counts is None:
        f = kvs.kvs_step_per_query if call == "per_query" else kvs.kvs_step
        f(p, Q, K, V, Ko, Vo, co, ws, stream=s)
    else:
        f = kvs.kvs_step_per_query_counts if call == "per_query" else kvs.kvs_step_counts
        f(p, Q, K, V, counts, Ko, Vo, co, ws, stream=s)
    torch.cuda.synchronize()
    rest = np.ones(len(co), dtype=bool)
    for o in out_rows:
        rest[o:o + budget] = False
    assert (co.cpu().numpy()[rest] == -7).all()                     # rows between the units are never touched
    return [np.concatenate([x[o:o + budget].float().cpu().numpy().ravel() for x in (Ko, Vo, co)]) for o in out_rows]


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("call", ["step", "per_query", "decode"])
@pytest.mark.parametrize("n", [2, 8, 9, 64, 70])
def test_regular_units_give_what_they_give_in_any_order(n, call, dtype):
    check_orders(n, call, dtype, 97, 40, 4, False)


@pytest.mark.parametrize("counts", [False, True])
@pytest.mark.parametrize("call,dtype,window", [
    ("step", "bf16", 4), ("step", "bf16", 40), ("step", "bf16", 70), ("step", "bf16", 130), ("step", "f32", 4),
    ("step", "f32", 33), ("per_query", "bf16", 33), ("per_query", "f32", 4), ("decode", "bf16", 2), ("decode", "bf16", 16),
    ("decode", "f32", 4)])
def test_regular_units_of_several_workgroups(call, dtype, window, counts):
    """Units of several score chunks, merge ranges and chunks of the pass over V (and rows for every family of kernels): more
    than 64 of them, where the descriptors' steps are no longer one, and two launches of such groups."""
    from test_gpu_parity import switches
    check_orders(66, call, dtype, 2600, 700, window, counts)
    with switches(group_units=70):
        check_orders(140, call, dtype, 1100, 300, window, counts)


def check_orders(n, call, dtype, length, budget, window, with_counts):
    import torch
    rng = np.random.default_rng(n)
    gap = 5
    io = torch.float32 if dtype == "f32" else torch.bfloat16
    gen = torch.Generator(device="cuda").manual_seed(n)
    rows = n * (length + gap)
    K, V = (torch.randn((rows, 64), generator=gen, device="cuda").to(io) for _ in range(2))
    Q = torch.randn((n, 2 * window, 64), generator=gen, device="cuda").to(io)
    counts = torch.randint(1, 9, (rows,), generator=gen, device="cuda", dtype=torch.int32) if with_counts else None
    up = [i * (length + gap) for i in range(n)]
    out_up = [i * (budget + 1) for i in range(n)]
    base = run(call, dtype, [length] * n, up, out_up, Q, K, V, budget, counts, window)
    # backwards (a regular group with negative steps), and shuffled (not regular unless there are only two)
    for order in (np.arange(n)[::-1], rng.permutation(n)):
        got = run(call, dtype, [length] * n, [up[i] for i in order], [out_up[i] for i in order],
                  Q[torch.from_numpy(order.copy()).cuda()].contiguous(), K, V, budget, counts, window)
        for j, i in enumerate(order):
            assert np.array_equal(got[j], base[i]), (order[:4], int(i))
