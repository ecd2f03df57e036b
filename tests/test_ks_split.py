"""The rows that the workgroups of a split key switch leave their sums in
(csrc/ks_split.h): no two share one and all lie in the workspace, for every
ring, digit size, number of special primes, level, number of integer rows and
batch that the parameters allow.  On the CPU."""

import pytest

from .ks_split_host import walk
from .test_gpu_ks_early import CASES, split_of


@pytest.mark.parametrize("log_n", range(12, 17))
def test_sums_are_disjoint(log_n):
    layouts, early_whole, overlapping = walk(log_n)
    assert layouts > 1000 and early_whole > 100
    assert overlapping == 0


def test_shapes_pinned_on_the_gpu():
    """The cases that are compared with the oracle on the GPU take early rows
    beside whole special rows, all but one where the rows of acc would overlap
    if the special rows' sums stayed in their own."""
    crowded = 0
    for c in CASES.values():
        parts, _, early = split_of(c)
        assert early and parts == 1
        crowded += len(c["p"]) + sum(q >= 2 ** 50 for q in c["q"][:c["level"]]) > c["level"]
    assert crowded == len(CASES) - 1
