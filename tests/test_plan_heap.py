"""The host planner's least-filled assignment on both sides of the line between
its two forms (a ring of lists by load; a heap for few, heavy items: more than
16 nonzeros per item and 65536), bit for bit against the oracle's linear scan.
"""
import numpy as np
import pytest

import oracle
from test_plan_ring import _degrees

S = pytest.importorskip("paper_2405_08470_amd.spmttkrp")

# (four items, so the line lies at 4 * 16 + 65536 nonzeros)
CASES = [(4 * 16 + 65536, 30_000, 7, 1), (4 * 16 + 65536 + 1, 30_000, 7, 1), (200_000, 150_000, 100_000, 0)]


@pytest.mark.parametrize("deg", CASES, ids=lambda d: str(d[0]))
@pytest.mark.parametrize("kappa", [1, 3, 9])
def test_least_filled_equals_the_oracle(deg, kappa):
    dims, idx = _degrees(*deg)
    got = S.plan_coo(dims, idx, kappa=kappa, split_cap=0)
    ref = oracle.plan(dims, idx, kappa, split_cap=0)
    for d in range(2):
        assert np.array_equal(got["remap"][d], ref["b"][d]) and np.array_equal(got["ptr"][d], ref["ptr"][d])
