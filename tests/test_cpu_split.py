"""The elementwise kernel with 1, 4 and 8 waves per partition on the CPU build
of the kernels (tests/cpuhip), against the oracle (no GPU needed).

A workgroup splits its partition among the lane groups of all its waves, and a
row that crosses groups is finished by a walk over them, so the cases are the
edges of that split: fewer nonzeros than groups, one more, a single row over
every group, rows that end exactly where a group ends, split rows, and ranks
with 1 to 64 groups per wave.  Tolerance: 1e-5 of M_abs, as everywhere.
"""
import os

import numpy as np
import pytest

import oracle
import test_cpu_kernels as K
from parity import check_elementwise, mttkrp_abs
from paper_2405_08470_amd import synth
from test_cpu_kernels import T, bf16_bits, lib  # noqa: F401 (lib: the fixture that builds the objects)


def _one_row(nnz):
    idx = np.zeros((3, nnz), np.int32)
    idx[1] = np.arange(nnz) % 7
    idx[2] = np.arange(nnz) % 5
    return (3, 7, 5), idx


def _equal_rows(rows, each):
    e = np.arange(rows * each)
    return (rows, 7, 5), np.stack([e // each, e % 7, e % 5]).astype(np.int32)


# name, (dims, indices), R, kappa
SHAPES = [
    ("one_row_r8", _one_row(3001), 8, 1),
    ("one_row_r128", _one_row(700), 128, 1),
    ("one_row_split", _one_row(2000), 16, 6),
    ("fewer_than_groups", _equal_rows(20, 3), 8, 1),
    ("groups_plus_one", _equal_rows(257, 1), 8, 1),
    ("rows_end_with_groups", _equal_rows(64, 16), 32, 1),
    ("short_rows", _equal_rows(300, 5), 64, 2),
]


def _build(lib, tmp_path_factory, defines):  # noqa: F811
    import ctypes
    import subprocess
    out = tmp_path_factory.mktemp("split")
    flags = ["-std=c++17", "-O1", "-g", "-fPIC", "-I", K.HERE, "-I", os.path.join(K.ROOT, "include"), "-I", K.CSRC]
    o, so = str(out / "ec_kernel.o"), str(out / "lib.so")
    subprocess.run([K.CXX, *flags, *[f"-D{d}" for d in defines], "-x", "c++", "-c",
                    os.path.join(K.CSRC, "ec_kernel.hip"), "-o", o], check=True, capture_output=True)
    objs = dict(K._OBJS, **{"ec_kernel.o": o})
    subprocess.run([K.CXX, "-shared", "-o", so, *objs.values(), "-pthread"], check=True, capture_output=True)
    L = ctypes.CDLL(so)
    for name in ("spt_tensor_load_coo", "spt_mttkrp", "spt_tensor_info", "spt_tensor_free"):
        getattr(L, name).argtypes = getattr(lib, name).argtypes
    L.spt_last_error.restype = ctypes.c_char_p
    return L


@pytest.fixture(scope="module", params=[(1, 1), (4, 0), (8, 1)], ids=lambda p: f"waves{p[0]}form{p[1]}")
def split_lib(request, lib, tmp_path_factory):  # noqa: F811
    return _build(lib, tmp_path_factory, [f"SPT_EC_WAVES={request.param[0]}", f"SPT_EC_FORM={request.param[1]}"])


@pytest.fixture(scope="module")
def order_libs(lib, tmp_path_factory):  # noqa: F811
    """The order of one wave: by one wave, and by the ordered form's turns."""
    return [_build(lib, tmp_path_factory, ["SPT_EC_ONE_WAVE", f"SPT_EC_ORDERED={below}"]) for below in (0, 1 << 30)]


@pytest.mark.parametrize("lib", ["chosen"], indirect=True)  # (only its objects are used)
@pytest.mark.parametrize("shape", SHAPES, ids=[s[0] for s in SHAPES])
@pytest.mark.parametrize("bf16", [False, True], ids=["f32", "bf16"])
def test_split_of_a_partition(lib, split_lib, shape, bf16):  # noqa: F811
    name, (dims, idx), R, kappa = shape
    val = synth.normal(3, 1, idx.shape[1]).astype(np.float32)
    Y = synth.random_factors(dims, R, seed=18)
    given, exact = (([bf16_bits(y) for y in Y], [oracle.bf16_round(y) for y in Y]) if bf16 else (Y, Y))
    t = T(split_lib, dims, idx, val, kappa=kappa)
    for d in range(3):
        out = t.mttkrp(d, given, R, bf16=bf16)
        ref = oracle.mttkrp(dims, idx, val, exact, d)
        check_elementwise(out, ref, mttkrp_abs(dims, idx, val, exact, d), label=f"{name} mode {d}")
    t.free()


@pytest.mark.parametrize("lib", ["chosen"], indirect=True)
@pytest.mark.parametrize("shape", SHAPES + [("four_modes", synth.random_coo, 64, 3), ("kappa300", synth.random_coo, 16, 300)],
                         ids=lambda s: s[0])
@pytest.mark.parametrize("bf16", [False, True], ids=["f32", "bf16"])
def test_ordered_form_gives_the_bits_of_one_wave(lib, order_libs, shape, bf16):  # noqa: F811
    name, made, R, kappa = shape
    if callable(made):
        dims = (60, 50, 40, 7) if name == "four_modes" else (60, 50, 40)
        idx = made(dims, 6000, seed=3, dist="zipf", zipf_s=1.1)[0]
    else:
        dims, idx = made
    if R > 64:
        R = 64  # CP-ALS ranks
    val = synth.normal(3, 1, idx.shape[1]).astype(np.float32)
    Y = [bf16_bits(y) if bf16 else y for y in synth.random_factors(dims, R, seed=18)]
    outs = []
    for L in order_libs:
        t = T(L, dims, idx, val, kappa=kappa)
        outs.append([t.mttkrp(d, Y, R, bf16=bf16) for d in range(len(dims))])
        t.free()
    for one, ordered in zip(*outs):
        assert np.array_equal(one.view(np.uint32), ordered.view(np.uint32)), name
