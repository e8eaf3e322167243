"""Merge launches of 129 to 256 ranges of 256 tokens (128 channels; bf16 units of unequal lengths: 145), which take workgroups of
eight wavefronts: the ends of that range, ranges that end short, cardinalities, a run longer than a workgroup looks ahead at
once, norms from memory."""

import pytest

from test_gpu_parity import check_merge_compact
from test_gpu_per_query import test_merge_compact_norms_matches_oracle as check_merge_norms

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("base,dtype,lens,budgets", [
    ("llama8b_8k", "bf16", [32769, 32], [6000, 32]),              # 130 ranges, one of a single token: four wavefronts still,
    ("llama8b_8k", "f32", [32769, 32], [6000, 32]),               # eight
    ("llama8b_8k", "bf16", [36609, 32], [6000, 32]),              # 145 ranges: eight
    ("llama8b_8k", "bf16", [33000, 32536], None),                 # 256
    ("llama8b_8k", "bf16", [32800], [40]),                        # 129; one run swallows nearly everything
    ("tiny", "f32", [20000, 257, 13000], [15000, 200, 2000]),
    ("stream2560", "bf16", [33000], [9000]),
])
def test_merge_of_a_range_per_compute_unit(base, dtype, lens, budgets):
    check_merge_compact(base, dtype, 128, lens, budgets, "hessian")


def test_merge_with_norms_of_a_range_per_compute_unit():
    check_merge_norms("stream2560", "bf16", 128, [20000, 13500], [9000, 3000], "hessian")
