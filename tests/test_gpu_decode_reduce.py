"""The combination of decode partials: caches of one chunk up to the most there are, at the borders of the batches of eight and
of the kernel's four parts, side by side with shorter ones."""

import pytest

from test_gpu_parity import check_decode, variant
from workloads import generate_unit

pytestmark = pytest.mark.gpu


# few rows in all: chunks of 64 rows on the vector ALU, so a cache of 64 c rows has c chunks (at most 64)
@pytest.mark.parametrize("dtype,D,G", [("bf16", 128, 4), ("f32", 64, 1)])
@pytest.mark.parametrize("chunks", [[1], [8, 1], [9], [32, 3, 33], [36, 37], [63, 1, 64]])
def test_decode_chunk_counts(dtype, D, G, chunks):
    w = variant("stream2560", dtype=dtype, head_dim=D, group=G, window=1, n_seq=len(chunks), n_kv_heads=1)
    w = w.scaled(fresh_tail=8, n_sink=2)
    check_decode([generate_unit(w, 0, s, 0, n=64 * c - 5 * (c % 3)) for s, c in enumerate(chunks)], dtype, D, G, 1, None)
