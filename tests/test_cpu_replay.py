"""The gradient fit on the CPU build of the kernels (tests/cpuhip), no GPU needed.

Residuals: the forward kernel's value of every nonzero is held to its written
order of roundings, bit for bit.  A lane sums its four ranks as
fma(p0, y0, p1 y1) + fma(p2, y2, p3 y3), p the product of all modes but the
last; the lanes of a nonzero are added in a butterfly.  The residuals are read
from the gradient of mode 0: each of its rows has one nonzero and column 0 of
every other factor is 1, so column 0 of the gradient is the residual itself.
"""
import ctypes
import os
import subprocess

import numpy as np
import pytest

import test_cpu_kernels as K
from paper_2405_08470_amd import synth
from test_cpu_kernels import T, lib  # noqa: F401 (lib: the fixture that builds the objects)

WRAPPED = ["_ZN3spt9launch_ecEiiiiiiRKNS_6EcArgsEP13cpuhip_stream",
           "_ZN3spt12launch_fixupEiRKNS_9FixupArgsEP13cpuhip_stream",
           "_ZN3spt14launch_forwardEiiiiRKNS_11ForwardArgsEP13cpuhip_stream",
           "_ZN3spt19launch_remap_stagedEilPKjPjPKiPKtP13cpuhip_stream",
           "_ZN3spt22launch_reduce_partialsEPKdiiPdP13cpuhip_stream", "_Z9hipMallocPPvm"]


@pytest.fixture(scope="module")
def replay_lib(lib, tmp_path_factory):  # noqa: F811
    out = tmp_path_factory.mktemp("replay")
    o, so = str(out / "replay.o"), str(out / "lib.so")
    subprocess.run([K.CXX, "-std=c++17", "-O1", "-g", "-fPIC", "-I", K.HERE, "-I", os.path.join(K.ROOT, "include"),
                    "-I", K.CSRC, "-c", os.path.join(K.HERE, "replay.cpp"), "-o", o], check=True, capture_output=True)
    subprocess.run([K.CXX, "-shared", "-o", so, *K._OBJS.values(), o, "-pthread",
                    *[f"-Wl,--wrap={w}" for w in WRAPPED]], check=True, capture_output=True)
    L = ctypes.CDLL(so)
    for name in ("spt_tensor_load_coo", "spt_mttkrp", "spt_tensor_info", "spt_tensor_free"):
        getattr(L, name).argtypes = getattr(lib, name).argtypes
    vp, i32 = ctypes.c_void_p, ctypes.c_int32
    L.spt_cp_gradient.argtypes = [vp, vp, i32, i32, vp, vp, vp]
    L.spt_cp_loss.argtypes = [vp, vp, i32, i32, vp, vp]
    L.spt_cp_adjoint.argtypes = [vp, vp, i32, i32, vp, vp]
    L.spt_last_error.restype = ctypes.c_char_p
    return L


def ptrs(arrays):
    return (ctypes.c_void_p * len(arrays))(*[a.ctypes.data for a in arrays])


_fmaf = ctypes.CDLL("libm.so.6").fmaf
_fmaf.restype, _fmaf.argtypes = ctypes.c_float, [ctypes.c_float] * 3
fma = np.vectorize(lambda a, b, c: _fmaf(float(a), float(b), float(c)), otypes=[np.float32])


def readable_residuals(N, R, nnz):
    """A tensor and factors whose mode-0 gradient holds the residuals (column 0
    of row i: the one nonzero of row i)."""
    rng = np.random.default_rng(100 * N + R)
    dims = [nnz, 31, 17, 13, 11, 9, 7, 5][:N]
    idx = np.stack([rng.permutation(nnz)] + [rng.integers(0, d, nnz) for d in dims[1:]]).astype(np.int32)
    val = rng.standard_normal(nnz).astype(np.float32)
    Y = [rng.standard_normal((d, R)).astype(np.float32) for d in dims]
    for y in Y[1:]:
        y[:, 0] = 1.0
    return dims, idx, val, Y


def written_residuals(idx, val, Y):
    p = Y[0][idx[0]]
    for w in range(1, len(Y) - 1):
        p = p * Y[w][idx[w]]
    y = Y[-1][idx[-1]]
    m = fma(p[:, 0::4], y[:, 0::4], p[:, 1::4] * y[:, 1::4]) + fma(p[:, 2::4], y[:, 2::4], p[:, 3::4] * y[:, 3::4])
    off, L = 1, m.shape[1]
    while off < L:
        m = m + m[:, np.arange(L) ^ off]
        off *= 2
    return m[:, 0] - val


@pytest.mark.parametrize("lib", ["chosen"], indirect=True)  # (only its objects are used)
@pytest.mark.parametrize("copies", [0, 1])
@pytest.mark.parametrize("R", [8, 16, 32, 64])
@pytest.mark.parametrize("N", [2, 3, 4, 5, 8])
def test_residuals_have_the_written_roundings(lib, replay_lib, N, R, copies):  # noqa: F811
    # (whole turns of the block: the CPU build needs all lanes of a wave at a shuffle)
    dims, idx, val, Y = readable_residuals(N, R, 256)
    t = T(replay_lib, dims, idx, val, copies=copies)
    grads = [np.zeros_like(y) for y in Y]
    loss = np.zeros(1)
    assert replay_lib.spt_cp_gradient(t.h, ptrs(Y), 0, R, ptrs(grads), loss.ctypes.data, None) == 0
    want = written_residuals(idx, val, Y)
    assert np.array_equal(grads[0][idx[0], 0].view(np.uint32), want.view(np.uint32))
    r = want.astype(np.float64)
    assert abs(loss[0] - 0.5 * (r * r).sum()) <= 1e-14 * loss[0]
    t.free()


SHAPES = [(60, 50), (30, 20, 40), (20, 15, 12, 6), (12, 11, 10, 9, 8)]


def _adjoint_of(L, dims, **kw):
    idx, val = synth.random_coo(dims, 1024, seed=7, dist="zipf", zipf_s=1.1)
    Y = [0.5 * y for y in synth.random_factors(dims, 16, seed=18)]
    t = T(L, dims, idx, val, kappa=5, **kw)
    t.mttkrp(0, Y, 16, flags=0)  # the workspace of this rank
    grads = [np.zeros_like(y) for y in Y]

    def loss():
        assert L.spt_cp_loss(t.h, ptrs(Y), 0, 16, np.zeros(1).ctypes.data, None) == 0, L.spt_last_error()

    def adjoint():
        assert L.spt_cp_adjoint(t.h, ptrs(Y), 0, 16, ptrs(grads), None) == 0, L.spt_last_error()

    def taken():
        out = [g.view(np.uint32).copy() for g in grads]
        for g in grads:
            g.fill(np.nan)
        return out
    return t, loss, adjoint, taken


@pytest.mark.parametrize("lib", ["chosen"], indirect=True)
@pytest.mark.parametrize("kw", [{}, {"dr": 1}, {"copies": 1}], ids=["staged", "fused", "copies"])
@pytest.mark.parametrize("dims", SHAPES, ids=len)
def test_recorded_adjoint_runs_again(lib, replay_lib, dims, kw):  # noqa: F811
    L = replay_lib
    t, loss, adjoint, taken = _adjoint_of(L, dims, **kw)
    loss()
    L.cpuhip_record(1)
    adjoint()
    L.cpuhip_record(0)
    want = taken()
    for _ in range(3):
        assert L.cpuhip_replay() >= 2 * len(dims)
        assert all(np.array_equal(a, b) for a, b in zip(taken(), want))
    adjoint()
    assert all(np.array_equal(a, b) for a, b in zip(taken(), want))
    t.free()


@pytest.mark.parametrize("lib", ["chosen"], indirect=True)
@pytest.mark.parametrize("kw", [{}, {"dr": 1}, {"copies": 1}], ids=["staged", "fused", "copies"])
@pytest.mark.parametrize("dims", SHAPES[1:], ids=len)
def test_adjoint_without_the_spare_stream(lib, replay_lib, dims, kw):  # noqa: F811
    L = replay_lib
    t, loss, adjoint, taken = _adjoint_of(L, dims, **kw)
    loss()
    adjoint()
    want, whole = taken(), t.info().device_bytes
    t.free()
    t, loss, adjoint, taken = _adjoint_of(L, dims, **kw)
    L.cpuhip_fail_malloc(1 if kw.get("copies") else 2)
    loss()
    assert t.info().device_bytes == whole - t.nnz * t.info().record_bytes
    for _ in range(3):
        adjoint()
        assert all(np.array_equal(a, b) for a, b in zip(taken(), want))
    loss()
    adjoint()
    assert all(np.array_equal(a, b) for a, b in zip(taken(), want))
    t.free()


@pytest.mark.parametrize("lib", ["chosen"], indirect=True)
def test_loss_is_refused_without_its_streams(lib, replay_lib):  # noqa: F811
    """Every allocation that is needed, failed in turn: refused, and the next
    call finds what it needs."""
    L = replay_lib
    for k in (0, 1, 3):
        t, loss, adjoint, taken = _adjoint_of(L, SHAPES[1])
        Y = [0.5 * y for y in synth.random_factors(SHAPES[1], 16, seed=18)]
        L.cpuhip_fail_malloc(k)
        assert L.spt_cp_loss(t.h, ptrs(Y), 0, 16, np.zeros(1).ctypes.data, None) != 0
        loss()
        adjoint()
        t.free()
