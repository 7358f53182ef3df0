"""The host planner's least-filled assignment at the edges of its two forms (a
ring of lists by load; a heap for items above 2^20 nonzeros) and of its two
sorts by size, bit for bit against the oracle's linear scan.
"""
import numpy as np
import pytest

import oracle

S = pytest.importorskip("paper_2405_08470_amd.spmttkrp")


def _degrees(*deg):
    """One mode with the given row degrees, and a mode of 5 rows."""
    rows = np.repeat(np.arange(len(deg)), deg)
    return (len(deg), 5), np.stack([rows, np.arange(rows.size) % 5]).astype(np.int32)


_RNG = np.random.default_rng(3)
CASES = [
    ("equal_sizes", _degrees(*[7] * 100), 9, None),
    ("ones_and_empty_rows", _degrees(*([1] * 50 + [0] * 40 + [1] * 30)), 16, None),
    ("ring_wraps", _degrees(*_RNG.integers(0, 60, 400)), 13, 0),
    ("more_blocks_than_items", _degrees(5, 3, 3, 1), 40, None),
    ("one_block", _degrees(5, 3, 3, 1), 1, None),
    ("pieces", _degrees(1000, 900, 3, 2, 2), 17, 50),
    ("sort_by_comparison", _degrees(80_000, 70_001, 3, 1), 3, 0),
    ("largest_of_the_ring", _degrees(1 << 20, 1 << 19, 7, 7, 1), 3, 0),
    ("heap", _degrees((1 << 20) + 1, 1 << 19, 7, 7, 1), 3, 0),
]


@pytest.mark.parametrize("name,shape,kappa,cap", CASES, ids=[c[0] for c in CASES])
def test_least_filled_equals_the_oracle(name, shape, kappa, cap):
    dims, idx = shape
    got = S.plan_coo(dims, idx, kappa=kappa, split_cap=cap)
    ref = oracle.plan(dims, idx, kappa, split_cap=cap)
    for d in range(2):
        assert np.array_equal(got["remap"][d], ref["b"][d]), f"{name}: remap ids of mode {d}"
        assert np.array_equal(got["ptr"][d], ref["ptr"][d]), f"{name}: partitions of mode {d}"
