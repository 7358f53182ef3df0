"""The reuse form of the elementwise kernel against the plain form on the CPU
build of the kernels (tests/cpuhip; no GPU needed), each forced by the build
option: the same bits, for 2 to 8 modes and partitions on both sides of the lines
between steps of one, two and four records per lane (a nonzero of four lanes:
R 16, or R 32 with BF16 factors).
"""
import numpy as np
import pytest

import oracle
import test_cpu_kernels as K
from paper_2405_08470_amd import synth
from paper_2405_08470_amd.spmttkrp import LAYOUTS
from parity import check_elementwise, mttkrp_abs
from test_cpu_kernels import T, bf16_bits, lib  # noqa: F401 (lib: the fixture that builds the objects)
from test_cpu_split import _build


@pytest.fixture(scope="module")
def forms(lib, tmp_path_factory):  # noqa: F811
    return [_build(lib, tmp_path_factory, [f"SPT_EC_FORM={f}"]) for f in (0, 1)]


SHAPES = [(c[0], c[1], c[2], c[4], c[5], c[6], c[7], c[8]) for c in K.CASES if c[2] <= 30_000] + [
    # name, dims, nnz, zipf_s, R, kappa, split_cap, layout
    ("short_255", (40, 30, 20), 7 * 255, 1.2, 16, 7, None, "auto"),
    ("short_256", (40, 30, 20), 7 * 256, 1.2, 16, 7, None, "auto"),
    ("short_8_modes", (9, 8, 7, 6, 5, 4, 3, 2), 40 * 30, 1.1, 16, 40, None, "auto"),
    ("long_4095", (40, 30, 20, 9), 2 * 4095, 1.2, 16, 2, None, "auto"),
    ("long_4096", (40, 30, 20, 9), 2 * 4096, 1.2, 16, 2, None, "auto"),
    ("two_modes_runs", (400, 6), 9_000, 1.1, 64, 9, None, "auto"),
]


@pytest.mark.parametrize("lib", ["chosen"], indirect=True)  # (only its objects are used)
@pytest.mark.parametrize("shape", SHAPES, ids=[s[0] for s in SHAPES])
@pytest.mark.parametrize("bf16", [False, True], ids=["f32", "bf16"])
def test_both_forms_give_the_same_bits(lib, forms, shape, bf16):  # noqa: F811
    name, dims, nnz, s, R, kappa, cap, layout = shape
    R = 32 if bf16 and R == 16 else R
    idx, val = synth.random_coo(dims, nnz, seed=17, dist="zipf", zipf_s=s)
    Y = synth.random_factors(dims, R, seed=18)
    given, exact = (([bf16_bits(y) for y in Y], [oracle.bf16_round(y) for y in Y]) if bf16 else (Y, Y))
    outs = []
    for L in forms:
        t = T(L, dims, idx, val, kappa=kappa, split_cap=cap, layout=LAYOUTS[layout])
        outs.append([t.mttkrp(d, given, R, bf16=bf16) for d in range(len(dims))])
        t.free()
    for d, (plain, reuse) in enumerate(zip(*outs)):
        assert np.array_equal(plain.view(np.uint32), reuse.view(np.uint32)), f"{name} mode {d}"
        check_elementwise(plain, oracle.mttkrp(dims, idx, val, exact, d), mttkrp_abs(dims, idx, val, exact, d),
                          label=f"{name} mode {d}")
