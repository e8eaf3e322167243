"""Performance cases of the KV-cache merge library: what a program that uses it has it do.

Three calls, all through the public binding: `kvs_step` / `kvs_step_counts` (a layer's cache is merged back to its
budget, from plain tokens or from a cache that was merged before), `kvs_step_per_query` (the same with the per-query
norms) and `kvs_decode_attention` (attention over a merged cache).  Shapes and distributions are those of
`workloads/configs.py`: Keys AR(1) along the tokens with a few outlier channels, unit-variance Values (a slot of c
tokens: a sum of c draws), Gaussian Queries.  Inputs are drawn on the GPU.

The edges that a step merges are decided by comparing fp32 attention masses, whose relative errors are below 1e-6.
As in the repository's tests, a unit whose r-th and (r+1)-th smallest edge scores are too close (2e-5, relative) gets
other Queries: a tie that rounding decides would shift every slot after it, and two correct programs would then agree
in nothing.
"""

from __future__ import annotations

import math
import random

import torch

import paper_2603_00907_amd as kvs

GAP_MIN = 2e-5
MAX_REDRAWS = 60

_BASE = dict(call="step", dtype="bf16", head_dim=128, units=8, group=4, window=32, n_lo=8192, n_hi=8192, budget=2048,
             keep=0.0, heads=8, n_sink=32, n_recent=0, causal=False, rule="hessian", rho_lo=0.9, rho_hi=0.9,
             outliers=4, heavy=False, mean_count=0.0, fresh=0, length_seed=0)


def _case(name, **kw):
    return dict(_BASE, name=name, **kw)


def listed():
    return [
        # The smallest configuration: one head, fp32, 1024 tokens halved.  Launches and the host's share count.
        _case("tiny_f32", dtype="f32", head_dim=64, units=1, group=1, window=8, n_lo=1024, n_hi=1024, budget=512,
              outliers=0),
        # One attention layer (8 KV heads, 32 query heads) after a prompt of 8 K tokens: the call that an inference
        # loop makes once per layer.
        _case("layer_8k"),
        # The same layer after a long prompt.
        _case("layer_32k", n_lo=32768, n_hi=32768, budget=4096),
        # All 32 layers of that model handed over in one call (256 units): the headline workload.
        _case("model_32k", units=256, n_lo=32768, n_hi=32768, budget=4096),
        # A batch of 16 sequences of 4 K to 64 K tokens, a quarter of each kept: odd lengths, ragged units.
        _case("ragged_batch", units=128, n_lo=4096, n_hi=65536, budget=0, keep=0.25, rho_lo=0.7, rho_hi=0.98,
              outliers=0, length_seed=4),
        # One layer of a model with 64 query heads, 131072 tokens, a window of 64 (512 query rows), heavy-tailed
        # Values: the longest caches.
        _case("layer_128k_wide", group=8, window=64, n_lo=131072, n_hi=131072, budget=8192, rho_lo=0.95, rho_hi=0.95,
              outliers=0, heavy=True),
        # Streaming: every cache of a 32-layer model has grown from its budget by a chunk (2048 + 512 slots) and is
        # merged back; the old slots stand for 4 tokens on average.
        _case("stream_2560", units=256, n_lo=2560, n_hi=2560, budget=2048, mean_count=4.0, fresh=512),
        # 28 layers with 7 query heads per KV head (224 query rows), causal mask inside the window.
        _case("gqa7_32k_causal", units=112, group=7, heads=4, n_lo=32768, n_hi=32768, budget=4096, causal=True),
        # An fp32 layer.
        _case("layer_32k_f32", dtype="f32", n_lo=32768, n_hi=32768, budget=4096),
        # One layer with the norms kept apart per query row.
        _case("per_query_32k", call="per_query", n_lo=32768, n_hi=32768, budget=4096),
        # A decode step over the merged caches of all 32 layers (4 query heads per KV head, one token).
        _case("decode_model_4k", call="decode", units=256, window=1, n_lo=4096, n_hi=4096, budget=4096,
              mean_count=8.0),
        # The same for one layer: the smallest call of a serving loop, made once per layer and token.
        _case("decode_layer_4k", call="decode", units=8, window=1, n_lo=4096, n_hi=4096, budget=4096, mean_count=8.0),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng: random.Random):
    """One more call of the same ranges: 700 to 131072 rows, 1 to 256 units, 1 to 512 query rows."""
    c = dict(_BASE)
    c["call"] = rng.choice(["step"] * 5 + ["per_query"] * 2 + ["decode"] * 2)
    c["dtype"] = "f32" if c["call"] != "per_query" and rng.random() < 0.2 else "bf16"
    c["head_dim"] = rng.choice([64, 128, 128, 128])
    c["group"] = rng.choice([1, 4, 4, 7, 8])
    if c["call"] == "decode":
        c["window"] = rng.choice([1, 1, 1, 2, 4, 8])
    else:
        c["window"] = rng.choice([1, 8, 16, 32, 32, 32, 64])
    rows = c["group"] * c["window"]
    c["heads"] = rng.choice([1, 4, 8])
    c["units"] = c["heads"] * _log_uniform(rng, 1, 256 // c["heads"])
    n = _log_uniform(rng, 700, 131072)
    # bounds on the whole call: rows of the caches and, per kind of arithmetic, query rows times cache rows
    most = 2500000 if c["dtype"] == "f32" else 5000000
    per_row = {"f32": 1 << 25, "bf16": 1 << 29}[c["dtype"]] if c["call"] != "per_query" else 1 << 27
    total = min(most, per_row // max(rows, 16) if c["dtype"] == "bf16" else per_row // max(rows // 4, 4))
    n = max(700, min(n, total // c["units"]))
    c["n_lo"] = c["n_hi"] = n
    if c["units"] > c["heads"] and rng.random() < 0.4:      # several sequences, each of its own length
        c["n_lo"] = max(300, n // rng.choice([2, 4, 8]))
        c["length_seed"] = rng.randrange(1, 1 << 20)
    c["budget"], c["keep"] = 0, round(rng.uniform(0.125, 0.8), 3)
    c["n_sink"] = rng.choice([0, 4, 32, 32])
    c["n_recent"] = rng.choice([0, 0, 0, 16])
    c["outliers"] = rng.choice([0, 4])
    c["rho_lo"] = c["rho_hi"] = round(rng.uniform(0.7 if c["outliers"] else 0.85, 0.98), 3)
    c["heavy"] = rng.random() < 0.2
    if c["call"] == "decode":
        c["mean_count"] = rng.choice([0.0, 4.0, 8.0])
    elif rng.random() < 0.3:
        c["mean_count"], c["fresh"] = 4.0, rng.choice([128, 512])
    if c["call"] != "decode":
        c["causal"] = c["window"] > 1 and rng.random() < 0.3
        if c["call"] == "step":
            c["rule"] = rng.choice(["hessian", "hessian", "hessian", "diagonal", "mean"])
    return c


# ------------------------------------------------------------------------------------------------------- shapes
def _lengths(case):
    """Rows of every unit; the heads of one sequence have the same length."""
    n_seq = max(1, case["units"] // case["heads"])
    if case["n_lo"] == case["n_hi"]:
        per_seq = [case["n_hi"]] * n_seq
    else:
        r = random.Random(case["length_seed"])
        per_seq = [r.randint(case["n_lo"], case["n_hi"]) for _ in range(n_seq)]
    return [per_seq[min(u // case["heads"], n_seq - 1)] for u in range(case["units"])]


def _budgets(case, lens):
    if case["call"] == "decode":
        return list(lens)
    if case["budget"]:
        return [case["budget"]] * len(lens)
    return [max(int(n * case["keep"]), case["n_sink"] + 1 + case["n_recent"]) for n in lens]


# ------------------------------------------------------------------------------------------------------- inputs
def _keys(case, gen, n, rho):
    """AR(1) along the rows, started in its stationary law: x_t = rho x_{t-1} + eps_t by recursive doubling."""
    x = torch.randn((n, case["head_dim"]), generator=gen, device="cuda")
    x[0] /= math.sqrt(1.0 - rho * rho)
    step, factor = 1, rho
    while step < n and factor > 1e-8:
        x[step:] = x[step:] + factor * x[:-step]
        step, factor = 2 * step, factor * factor
    if case["outliers"]:
        ch = torch.randperm(case["head_dim"], generator=gen, device="cuda")[:case["outliers"]]
        x[:, ch] *= 8.0
    return x


def _values(case, gen, n):
    v = torch.randn((n, case["head_dim"]), generator=gen, device="cuda")
    if case["heavy"]:                                   # Student t with 4 degrees of freedom, unit variance
        chi2 = torch.zeros((n, case["head_dim"]), device="cuda")
        for _ in range(4):
            chi2 += torch.randn((n, case["head_dim"]), generator=gen, device="cuda").square()
        v = v / torch.sqrt(chi2 / 4.0) / math.sqrt(2.0)
    return v


def _cardinalities(case, gen, n):
    """1 for the sink rows and the fresh tail, geometric with the given mean between them."""
    c = torch.ones(n, dtype=torch.int32, device="cuda")
    lo, hi = min(case["n_sink"], n), n - case["fresh"]
    if hi > lo:
        u = torch.rand(hi - lo, generator=gen, device="cuda", dtype=torch.float64).clamp_min(1e-12)
        c[lo:hi] = (1 + torch.floor(torch.log(u) / math.log1p(-1.0 / case["mean_count"]))).int()
    return c


def _attention(case, Q, K, counts):
    """alpha [R, n] in 64 bits for one unit: softmax of the scaled logits, a slot of c tokens counting c times."""
    n, W = K.shape[0], case["window"]
    e = (Q.double() @ K.double().T) / math.sqrt(case["head_dim"])
    if counts is not None:
        e += torch.log(counts.double())
    if case["causal"]:
        last = n - W + torch.arange(Q.shape[0], device="cuda") % W
        e.masked_fill_(torch.arange(n, device="cuda") > last[:, None], -math.inf)
    return torch.softmax(e, dim=1)


def _edge_scores(case, alpha_bar):
    lo, hi = case["n_sink"], alpha_bar.shape[0] - 2 - case["n_recent"]
    return alpha_bar[lo:hi + 1] + alpha_bar[lo + 1:hi + 2]


def _gap(case, alpha_bar, budget):
    sigma = _edge_scores(case, alpha_bar)
    r = alpha_bar.shape[0] - budget
    if r <= 0 or r >= sigma.shape[0]:
        return math.inf
    s = torch.sort(sigma).values[r - 1:r + 1].tolist()
    return (s[1] - s[0]) / s[1]


def _inputs(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    pick = random.Random(seed)
    io = torch.float32 if case["dtype"] == "f32" else torch.bfloat16
    lens = _lengths(case)
    budgets = _budgets(case, lens)
    rows, R, D = sum(lens), case["group"] * case["window"], case["head_dim"]
    K = torch.empty((rows, D), dtype=io, device="cuda")
    V = torch.empty((rows, D), dtype=io, device="cuda")
    Q = torch.empty((len(lens), R, D), dtype=io, device="cuda")
    counts = torch.ones(rows, dtype=torch.int32, device="cuda") if case["mean_count"] else None
    r0 = 0
    for u, n in enumerate(lens):
        c = None
        K[r0:r0 + n] = _keys(case, gen, n, pick.uniform(case["rho_lo"], case["rho_hi"]))
        v = _values(case, gen, n)
        if counts is not None:
            c = counts[r0:r0 + n] = _cardinalities(case, gen, n)
            v = v * torch.sqrt(c.float())[:, None]
        V[r0:r0 + n] = v
        widest = -1.0
        for _ in range(MAX_REDRAWS):
            q = torch.randn((R, D), generator=gen, device="cuda").to(io)
            gap = math.inf
            if case["call"] != "decode":
                gap = _gap(case, _attention(case, q, K[r0:r0 + n], c).mean(dim=0), budgets[u])
            if gap > widest:
                widest, Q[u] = gap, q
            if gap >= GAP_MIN:
                break
        r0 += n
    return lens, budgets, Q, K, V, counts


def prepare(case, seed):
    lens, budgets, Q, K, V, counts = _inputs(case, seed)
    p = kvs.Problem(lens=lens, budgets=budgets, group=case["group"], window=case["window"],
                    head_dim=case["head_dim"], dtype=case["dtype"], n_sink=case["n_sink"],
                    n_recent=case["n_recent"], key_rule=case["rule"], causal=case["causal"])
    size = {"step": kvs.kvs_workspace_size, "per_query": kvs.kvs_per_query_workspace_size,
            "decode": kvs.kvs_decode_workspace_size}[case["call"]](p)
    state = dict(call=case["call"], p=p, Q=Q, K=K, V=V, counts=counts,
                 ws=torch.empty(size, dtype=torch.uint8, device="cuda"))
    if case["call"] == "decode":
        state["out"] = torch.empty((len(lens), Q.shape[1], Q.shape[2]), dtype=torch.float32, device="cuda")
    else:
        state["K_out"] = torch.empty((p.rows_out, Q.shape[2]), dtype=K.dtype, device="cuda")
        state["V_out"] = torch.empty((p.rows_out, Q.shape[2]), dtype=K.dtype, device="cuda")
        state["counts_out"] = torch.empty(p.rows_out, dtype=torch.int32, device="cuda")
    return state


def run(state):
    s, stream = state, torch.cuda.current_stream().cuda_stream
    if s["call"] == "decode":
        kvs.kvs_decode_attention(s["p"], s["Q"], s["K"], s["V"], s["counts"], s["out"], s["ws"], stream=stream)
        return {"out": s["out"]}
    if s["call"] == "per_query":
        kvs.kvs_step_per_query_counts(s["p"], s["Q"], s["K"], s["V"], s["counts"], s["K_out"], s["V_out"],
                                      s["counts_out"], s["ws"], stream=stream)
    else:
        kvs.kvs_step_counts(s["p"], s["Q"], s["K"], s["V"], s["counts"], s["K_out"], s["V_out"], s["counts_out"],
                            s["ws"], stream=stream)
    return {"K": s["K_out"], "V": s["V_out"], "counts": s["counts_out"]}


def work(case):
    lens = _lengths(case)
    out = sum(min(n, b) for n, b in zip(lens, _budgets(case, lens)))
    rows, R, D = sum(lens), case["group"] * case["window"], case["head_dim"]
    elt = 4 if case["dtype"] == "f32" else 2
    b = 2 * rows * D * elt + len(lens) * R * D * elt + (4 * rows if case["mean_count"] else 0)
    if case["call"] == "decode":
        return {"bytes": b + 4 * len(lens) * R * D, "flops": 4 * rows * R * D}
    products = 3 if case["call"] == "per_query" else 1      # Q.K; with per-query norms also alpha.V and o.V
    return {"bytes": b + out * (2 * D * elt + 4), "flops": 2 * products * rows * R * D + 10 * rows * D}


def tolerance(case):
    # Seen against 64 bits: decode (fp32 sums) up to 1.7e-6; a step's outputs 1e-7 in fp32 and 1.6e-3, the rounding of
    # the result, in bf16.  About four times that; fp32 Keys are weighted means, whose error the weights can raise.
    if case["call"] == "decode":
        return {"rel": 6e-6}
    return {"rel": 2e-6} if case["dtype"] == "f32" else {"rel": 7e-3}


# ------------------------------------------------------------------------------------------- in 64 bits, plain torch
def _norms(case, alpha, values):
    """A_t and C_t of the Key rule, averaged over the rows of alpha (one row: the mean attention)."""
    R, n = alpha.shape
    o = alpha @ values
    A, C = values.new_zeros(n), values.new_zeros(n - 1)
    for q in range(R):
        r = values - o[q]
        A += (alpha[q] * (1 - 2 * alpha[q])).abs() * r.norm(dim=1)
        C += alpha[q, :-1] * alpha[q, 1:] * (r[:-1] + r[1:]).norm(dim=1)
    return A / R, C / R


def _merge(case, Q, K, V, counts, budget):
    K, V = K.double(), V.double()
    n = K.shape[0]
    alpha = _attention(case, Q, K, counts)
    alpha_bar = alpha.mean(dim=0)
    c = torch.ones(n, dtype=torch.float64, device="cuda") if counts is None else counts.double()
    mask = torch.zeros(n, dtype=torch.bool, device="cuda")
    if n > budget:
        order = torch.sort(_edge_scores(case, alpha_bar), stable=True).indices[:n - budget]
        mask[case["n_sink"] + order] = True
    slot = torch.zeros(n, dtype=torch.int64, device="cuda")
    slot[1:] = torch.cumsum((~mask[:-1]).long(), 0)
    n_out = n - int(mask.sum())
    if case["rule"] == "mean":
        u = c.clone()
    else:
        A, C = _norms(case, alpha if case["call"] == "per_query" else alpha_bar[None], V / c[:, None])
        u = A
        if case["rule"] == "hessian":
            inner = torch.where(mask[:-1], C, torch.zeros_like(C))
            u = A.clone()
            u[:-1] -= inner
            u[1:] -= inner

    def sums(x):
        return x.new_zeros((n_out,) + x.shape[1:]).index_add_(0, slot, x)

    rows, U = sums(torch.ones_like(c)), sums(u)
    w = torch.where((U > 0)[slot], u, c)
    K_out = sums(w[:, None] * K) / sums(w)[:, None]
    K_out = torch.where((rows == 1)[:, None], sums(K), K_out)
    return K_out, sums(V), sums(c).round().int()


def exact(case, seed):
    lens, budgets, Q, K, V, counts = _inputs(case, seed)
    if case["call"] == "per_query" and sum(lens) * Q.shape[1] * case["head_dim"] > 1 << 36:
        return None
    got, r0 = [], 0
    for u, (n, b) in enumerate(zip(lens, budgets)):
        k, v, c = K[r0:r0 + n], V[r0:r0 + n], None if counts is None else counts[r0:r0 + n]
        if case["call"] == "decode":
            alpha = _attention(case, Q[u], k, c)
            got.append((alpha @ (v.double() if c is None else v.double() / c.double()[:, None]),))
        else:
            got.append(_merge(case, Q[u], k, v, c, b))
        r0 += n
    if case["call"] == "decode":
        return {"out": torch.stack([g[0] for g in got])}
    return {"K": torch.cat([g[0] for g in got]), "V": torch.cat([g[1] for g in got]),
            "counts": torch.cat([g[2] for g in got])}
