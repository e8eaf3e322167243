"""The kernel for more than 128 bf16 rows with long and with short stages of K: in both sweeps and both channel counts, chunks that
end inside a stage and inside a tile, cardinalities, causal window, reads past the caches."""

import pytest

from test_gpu_score_whole_rounds import check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lens,D,G,W,counts,causal", [
    ([4000 + 431 * i for i in range(24)], 128, 7, 32, False, False),     # long in sweep 0, short in sweep 1
    ([4000 + 431 * i for i in range(24)], 128, 7, 32, True, True),       # short in both
    ([300 + 37 * i for i in range(72)], 128, 8, 32, False, True),        # chunks of two long stages: short ones
    ([4000 + 431 * i for i in range(24)], 64, 8, 32, False, True),       # long in both
    ([4000 + 431 * i for i in range(24)], 64, 9, 32, False, True),       # short in sweep 0, long in sweep 1
    ([300 + 37 * i for i in range(72)], 64, 7, 32, False, False),        # the same with chunks of two long stages
    ([4000 + 431 * i for i in range(24)], 64, 7, 32, True, False),
    ([2900 + 431 * i for i in range(30)], 64, 9, 32, True, False),       # the same with eight wavefronts
    ([2900 + 431 * i for i in range(30)], 128, 8, 64, False, False),
    ([2900 + 431 * i for i in range(30)], 128, 9, 32, True, True),
    ([33000 + 97 * i for i in range(24)], 64, 9, 32, False, True),       # read past the caches: long in sweep 0, V in sweep 1
    ([20000 + 97 * i for i in range(40)], 64, 7, 32, False, False),
    ([20000 + 97 * i for i in range(40)], 64, 8, 32, True, True),        # with cardinalities
    ([20000 + 97 * i for i in range(40)], 64, 9, 32, True, False),
])
def test_score_in_stages(lens, D, G, W, counts, causal):
    check(lens, D, G, W, "bf16", counts, causal)
