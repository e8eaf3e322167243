"""Selection with the keys in registers: numbers of edges at the borders of a group of four, a wavefront, a slice of 4096 and
the kernel's sizes, rows that do not begin on a multiple of four, and workgroups that share a unit, against the oracle bit
for bit."""

import numpy as np
import pytest

from test_gpu_parity import check_select

pytestmark = pytest.mark.gpu


def masses(kind, n, rng):
    if kind == "ties":
        a = rng.integers(1, 4, size=n).astype(np.float64)
    elif kind == "crowded":                      # a handful of values in one bin of a wide range: the list overflows
        a = 1.0 + 1e-6 * rng.integers(0, 40, size=n)
        a[n // 2] = 1e6
    else:
        a = np.exp(2.0 * rng.standard_normal(n))
    return a / a.sum()


# (tokens, sinks, recent): the eligible edges are tokens - 1 - sinks - recent
@pytest.mark.parametrize("kind", ["lognormal", "ties", "crowded"])
@pytest.mark.parametrize("shapes", [
    [(5, 3, 0), (6, 0, 3), (7, 3, 0), (9, 1, 3), (12, 3, 2)],                        # 1 to 6 edges
    [(259, 1, 0), (4096, 0, 0), (4100, 2, 1), (4105, 3, 5), (8190, 1, 0)],           # a wavefront, one slice, two
    [(8193, 0, 0), (8200, 1, 2), (12289, 0, 0), (32760, 3, 1), (32767, 0, 0)],       # two, three, eight slices
    [(32770, 0, 0), (36871, 5, 2), (65530, 2, 1), (65536, 0, 0), (65537, 1, 0)],     # nine to sixteen, seventeen
])
def test_select_at_the_borders_of_slices(shapes, kind):
    rng = np.random.default_rng(len(kind) + shapes[0][0])
    for sinks, recent in sorted({(s, r) for _, s, r in shapes}):
        lens = [n for n, s, r in shapes if (s, r) == (sinks, recent)]
        for first in range(4):                   # a unit in front: the others begin at every remainder of four
            pads = [first + 1] if first else []
            alphas = [masses(kind, n, rng) for n in pads + lens]
            for share in (0.25, 0.9):
                budgets = [n for n in pads] + [min(n - 1, max(int(n * share), sinks + recent + 1)) for n in lens]
                check_select(alphas, budgets, sinks, recent)
                check_select(alphas, budgets, sinks, recent, "one")


def test_select_a_launch_of_many_units_that_share_workgroups():
    """Sixty-four units, four workgroups to each: one to eight slices side by side."""
    rng = np.random.default_rng(3)
    lens = [int(x) for x in rng.integers(700, 33000, size=64)]
    alphas = [masses("ties" if i % 5 == 0 else "lognormal", n, rng) for i, n in enumerate(lens)]
    check_select(alphas, [max(40, n // 3) for n in lens], 32, 0)
