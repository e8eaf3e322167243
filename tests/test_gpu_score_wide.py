"""The score kernels whose running sums have a fixed reference (windows of more than 64 rows): logits that climb far above
the first stage's, the rounding of the terms against a low reference, blocks of query rows that are missing or partial, and
numbers that have no split into bf16 parts."""

import numpy as np
import pytest

from oracle import kvs_oracle as O
from workloads import bf16_bits_to_f32, f32_to_bf16_bits, generate_unit

from helpers import DeviceBatch, from_device
from test_gpu_parity import TOL_ALPHA, score_path, switches, torch_sync, variant

pytestmark = pytest.mark.gpu


def score(units, dtype, D, G, W, causal=False):
    batch = DeviceBatch(units, group=G, window=W, head_dim=D, dtype=dtype, n_sink=32, gap_rows=3, causal=causal)
    batch.kvs.kvs_score_counts(batch.problem, batch.Q, batch.K, batch.V, batch.counts_in, batch.alpha_bar, batch.o_bar,
                               batch.ws, stream=batch.stream())
    torch_sync()
    batch.check_guards()
    alpha, o_bar = from_device(batch.alpha_bar), from_device(batch.o_bar)
    return [alpha[r0:r0 + u.n] for u, r0 in zip(units, batch.problem.in_rows)], o_bar


@pytest.mark.parametrize("base,dtype,D,G,W,lens,causal", [
    ("llama8b_8k", "bf16", 128, 5, 32, [33, 64, 65, 1500], False),    # 160 rows: three blocks of 64, the last half empty
    ("llama8b_8k", "bf16", 64, 7, 32, [2000, 127], True),             # 224 rows: four
    ("llama8b_8k", "bf16", 128, 9, 31, [700, 129], True),             # 279 rows: nine blocks on eight, the last of 23
    ("stream2560", "bf16", 128, 8, 64, [1300], False),                # 512 rows, cardinalities
    ("llama8b_8k", "bf16", 64, 13, 40, [300], False),                 # 520 rows: a second launch of eight rows
    ("llama8b_8k", "bf16", 128, 5, 32, [45000] * 6, False),           # more workgroups than compute units: the shared tiles
    ("llama8b_8k", "bf16", 64, 5, 32, [20011] * 8, True),             # ... and tiles of their own, in three blocks of 64 rows
    ("llama8b_8k", "bf16", 128, 7, 32, [29003] * 14, True),           # ... 208 MB: K read past the caches, V carried along
    ("tiny", "f32", 128, 5, 13, [32, 33, 1000], False),               # 65 rows: a block of one row, a wavefront without
    ("tiny", "f32", 64, 4, 32, [511, 64], True),
    ("tiny", "f32", 128, 3, 43, [600], False),                        # 129 rows: eight wavefronts, three without rows
    ("stream2560", "f32", 64, 8, 33, [900, 40], True),                # 264 rows: a second launch of eight
])
def test_score_wide_windows(base, dtype, D, G, W, lens, causal):
    w = variant(base, dtype=dtype, head_dim=D, group=G, window=W, n_seq=len(lens), n_kv_heads=1).scaled(fresh_tail=16)
    lens = [max(n, W) for n in lens]
    units = [generate_unit(w, 0, s, 0, n=n) for s, n in enumerate(lens)]
    alphas, o_bar = score(units, dtype, D, G, W, causal)
    for i, (u, got) in enumerate(zip(units, alphas)):
        ref, ref_o = O.score(u.Q, u.K, u.V, counts=u.counts, causal_window=W if causal else 0)
        assert np.max(np.abs(got - ref) / ref) < TOL_ALPHA, i
        bound = TOL_ALPHA * (ref @ np.abs(O.slot_values(u.V, u.counts))) + 1e-7
        assert (np.abs(o_bar[i] - ref_o) <= bound).all(), i


CLIMB_CASES = [
    ("bf16", 128, 8, 64, 2000, "tiny", False), ("bf16", 64, 9, 32, 1100, "tiny", False),
    ("f32", 128, 4, 32, 2000, "tiny", False), ("f32", 64, 8, 40, 1100, "tiny", False),
    # every wavefront with tiles and a reference of its own: two, three and four blocks of 64 rows
    ("bf16", 128, 4, 25, 3000, "tiny", False), ("bf16", 128, 4, 32, 2000, "tiny", False),
    ("bf16", 64, 4, 32, 1100, "stream2560", False), ("bf16", 128, 4, 32, 1500, "stream2560", True),
    ("bf16", 128, 5, 32, 2000, "tiny", False), ("bf16", 64, 5, 32, 1500, "stream2560", True),
    ("bf16", 128, 7, 32, 2000, "stream2560", False), ("bf16", 128, 8, 32, 1100, "tiny", True),
    ("f32", 128, 4, 32, 1500, "stream2560", True), ("bf16", 128, 8, 64, 1500, "stream2560", True),
]


@pytest.mark.parametrize("dtype,D,G,W,n,base,causal,path", [c + (None,) for c in CLIMB_CASES] + [
    c + ("shared",) for c in CLIMB_CASES if c[0] == "bf16" and 128 < c[2] * c[3] <= 256])   # the kernel of larger launches
def test_score_logits_that_climb(dtype, D, G, W, n, base, causal, path):
    """Keys 25 times larger at the end than at the start: a later stage's terms exceed the first one's by far more than
    2^64, so its sums have to be formed again with a higher reference, several times per chunk; with cardinalities
    (stream2560) and a causal window, too."""
    w = variant(base, dtype=dtype, head_dim=D, group=G, window=W, n_seq=1, n_kv_heads=1).scaled(fresh_tail=16)
    u = generate_unit(w, 0, 0, 0, n=n)
    K = u.K * np.linspace(0.2, 5.0, n, dtype=np.float32)[:, None] ** 2
    u.K = bf16_bits_to_f32(f32_to_bf16_bits(K)) if dtype == "bf16" else K.astype(np.float32)
    e = (u.Q.reshape(-1, D).astype(np.float64) @ u.K.T.astype(np.float64)) / np.sqrt(D)
    assert e.max() > 100
    with score_path(path):
        got = score([u], dtype, D, G, W, causal)[0][0]
    ref, _ = O.score(u.Q, u.K, u.V, counts=u.counts, causal_window=W if causal else 0)
    # TOL_ALPHA is for logits up to 20: the error of a term grows with the logit.  Terms that underflow are left out.
    seen = ref > 1e-30
    assert seen.sum() > 100
    assert np.max(np.abs(got - ref)[seen] / ref[seen]) < TOL_ALPHA * np.abs(e).max() / 20


@pytest.mark.parametrize("dtype,G,W", [("bf16", 3, 32), ("bf16", 4, 32), ("bf16", 5, 32), ("bf16", 8, 32), ("bf16", 8, 64),
                                       ("f32", 4, 32), ("f32", 8, 32)])
def test_score_normaliser_of_rows_that_rise_far_above_their_first_tokens(dtype, G, W):
    """The first 256 tokens lie 2^61 below the one token on which a row puts nearly all its weight: formed against a
    reference from those first tokens, that term's exponent argument would be 61, rounded to 2^-19.

    Rows and dominating tokens: rows of a Hadamard matrix, so that every row has one token of its own (rows 128 apart share
    theirs) with a base-2 logit of 6 to 7.5; all others have -20.  What rounds, as base-2 exponents: the normaliser, 13 to
    17, by up to 2^-21 (2^-20 from 16 on); sweep 0's argument, up to 16 in size, 2^-21; sweep 1's, up to 9, 2^-21.  Each is
    uniform, so the tokens' relative errors are ln 2 sqrt(2^-40 + 2 * 2^-42) / sqrt 3 = 4.7e-7 in the root mean square,
    with an argument of 61 ln 2 sqrt(2^-38 + ...) / sqrt 3 = 8.6e-7."""
    D, n, R = 128, 2048, G * W
    H = np.array([[1.0]])
    while H.shape[0] < D:
        H = np.block([[H, H], [H, -H]])
    w = variant("tiny", dtype=dtype, head_dim=D, group=G, window=W, n_seq=1, n_kv_heads=1)
    u = generate_unit(w, 0, 0, 0, n=n)
    u.Q = H[np.arange(R) % D].reshape(G, W, D).astype(np.float32)
    rng = np.random.default_rng(R)
    K = np.zeros((n, D))
    K[:, 0] = -157.0
    K[:256, 0] = -424.0
    tokens = 300 + rng.permutation(n - 300)[:D]
    gain = (210.0 + rng.integers(0, 5, D)) / 128.0             # (numbers that bf16 has)
    K[tokens] += gain[:, None] * H
    K[tokens, 0] = np.round(rng.uniform(-158.0, -154.0, D))
    u.K = bf16_bits_to_f32(f32_to_bf16_bits(K.astype(np.float32)))
    with switches(score_chunk=2048):
        got = score([u], dtype, D, G, W)[0][0]
    ref, _ = O.score(u.Q, u.K, u.V)
    mine = tokens[:min(R, D)]
    assert (ref[mine] > 0.9 / R).all()
    err = (got[mine] - ref[mine]) / ref[mine]
    assert np.sqrt(np.mean(err ** 2)) < 6e-7


@pytest.mark.parametrize("G,W", [(3, 32), (4, 32), (5, 32), (8, 32), (8, 64)])
@pytest.mark.parametrize("count,first", [(1 << 22, -292.0), (1 << 10, -196.0)])
def test_score_normaliser_of_rows_that_small_cardinalities_dominate(count, first, G, W):
    """As above, with first tokens that stand for 2^22 (2^10) tokens each and lie 2^44 (2^32) below: in a sum in units of
    their cardinality the one token on which a row puts its weight has a term that many times smaller than its exponential,
    whose argument would be 37 (25), rounded to 2^-19 (2^-20), before the sum meets a limit of 2^16.  The same rounding
    as above, the same bound."""
    D, n, R = 128, 2048, G * W
    H = np.array([[1.0]])
    while H.shape[0] < D:
        H = np.block([[H, H], [H, -H]])
    w = variant("stream2560", dtype="bf16", head_dim=D, group=G, window=W, n_seq=1, n_kv_heads=1).scaled(fresh_tail=16)
    u = generate_unit(w, 0, 0, 0, n=n)
    u.Q = H[np.arange(R) % D].reshape(G, W, D).astype(np.float32)
    rng = np.random.default_rng(R)
    u.counts = np.ones(n, dtype=np.int32)
    u.counts[:256] = count
    K = np.zeros((n, D))
    K[:, 0] = -157.0
    K[:256, 0] = first
    tokens = 300 + rng.permutation(n - 300)[:D]
    gain = (210.0 + rng.integers(0, 5, D)) / 128.0             # (numbers that bf16 has)
    K[tokens] += gain[:, None] * H
    K[tokens, 0] = np.round(rng.uniform(-158.0, -154.0, D))
    u.K = bf16_bits_to_f32(f32_to_bf16_bits(K.astype(np.float32)))
    with switches(score_chunk=2048):
        got = score([u], "bf16", D, G, W)[0][0]
    ref, _ = O.score(u.Q, u.K, u.V, counts=u.counts)
    mine = tokens[:min(R, D)]
    assert (ref[mine] > 0.9 / R).all()
    err = (got[mine] - ref[mine]) / ref[mine]
    assert np.sqrt(np.mean(err ** 2)) < 6e-7


@pytest.mark.parametrize("exponent", [-122, 100])
@pytest.mark.parametrize("D,G,W", [(128, 4, 32), (64, 8, 32)])
def test_score_f32_numbers_whose_parts_are_too_small(D, G, W, exponent):
    """One channel of the queries of about 2^exponent in a third of the rows, and of the keys of about 2^-exponent: the
    products are ordinary numbers, but the second and third bf16 parts of the small factors are not normal numbers."""
    w = variant("tiny", dtype="f32", head_dim=D, group=G, window=W, n_seq=1, n_kv_heads=1)
    u = generate_unit(w, 0, 0, 0, n=700)
    rng = np.random.default_rng(exponent + 200)
    Q = u.Q.reshape(G * W, D).copy()
    Q[:, 5] = 0.0
    Q[::3, 5] = np.float32(2.0 ** exponent) * (1 + rng.random(len(Q[::3]), dtype=np.float32))
    u.Q = Q.reshape(u.Q.shape)
    u.K = u.K.copy()
    u.K[:, 5] = np.float32(2.0 ** -exponent) * (1 + rng.random(u.n, dtype=np.float32)) * np.sqrt(D)
    got = score([u], "f32", D, G, W)[0][0]
    ref, _ = O.score(u.Q, u.K, u.V)
    assert np.max(np.abs(got - ref) / ref) < TOL_ALPHA


@pytest.mark.parametrize("D,G,W", [(128, 4, 32), (64, 8, 32)])
def test_score_f32_numbers_without_a_split(D, G, W):
    """fp32 Keys that are minus infinity, or that round to infinity as bf16, in rows of a tile's beginning, middle and end:
    a row all of whose logits are minus infinity has no mass and changes nothing for the others."""
    n = 700
    w = variant("tiny", dtype="f32", head_dim=D, group=G, window=W, n_seq=1, n_kv_heads=1)
    u = generate_unit(w, 0, 0, 0, n=n)
    u.Q[..., 5] = np.abs(u.Q[..., 5]) + np.float32(0.1)
    u.Q[..., 6] = np.float32(1e-38)
    u.K[[0, 100, 255, 640, 699], 5] = -np.inf
    u.K[[31, 333], 6] = np.float32(3.4e38)
    got = score([u], "f32", D, G, W)[0][0]
    with np.errstate(invalid="ignore"):
        ref, _ = O.score(u.Q, u.K, u.V)
    assert (got[[0, 100, 255, 640, 699]] == 0).all() and np.isfinite(got).all()
    keep = ref > 0
    assert keep.sum() == n - 5
    assert np.max(np.abs(got - ref)[keep] / ref[keep]) < TOL_ALPHA
