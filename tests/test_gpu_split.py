"""The elementwise kernel at the edges of its launch choices, on the GPU:
partition counts on both sides of the lines between 8, 4 and 1 waves per
partition, one row over every lane group, fewer nonzeros than groups, split
rows, every rank, FP32 and BF16 factors, and 2- to 4-mode tensors (plain and
reuse form), against the oracle.  Tolerance: 1e-5 of M_abs per element.
"""
import numpy as np
import pytest

import oracle
from paper_2405_08470_amd import synth
from parity import check_elementwise, mttkrp_abs

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)
S = pytest.importorskip("paper_2405_08470_amd.spmttkrp")


def _one_row(nnz):
    e = np.arange(nnz)
    return (3, 70, 50), np.stack([0 * e, e % 70, e % 50]).astype(np.int32)


def _zipf(dims, nnz):
    return dims, synth.random_coo(dims, nnz, seed=5, dist="zipf", zipf_s=1.1)[0]


# name, (dims, indices), rank, kappa
SHAPES = [
    ("one_row_r8", _one_row(5001), 8, 1),
    ("one_row_r128", _one_row(1500), 128, 1),
    ("one_row_split", _one_row(5001), 16, 7),
    ("fewer_than_groups", _zipf((9, 8, 7), 40), 8, 1),
    ("kappa256", _zipf((300, 200, 4000), 60_000), 16, 256),
    ("kappa257", _zipf((300, 200, 4000), 60_000), 16, 257),
    ("kappa4096", _zipf((300, 200, 4000), 60_000), 32, 4096),
    ("kappa8191", _zipf((300, 200, 4000), 60_000), 32, 8191),
    ("kappa8192", _zipf((300, 200, 40_000), 100_000), 32, 8192),
    ("four_modes", _zipf((300, 200, 400, 30), 60_000), 64, 300),
    ("two_modes", _zipf((3000, 200), 60_000), 8, 300),
    ("eight_modes_r8", _zipf((9, 8, 7, 6, 5, 4, 3, 2), 6_000), 8, 3),
    # partitions of 4095 and 4096 nonzeros (longer steps at R 16, and at R 32 with BF16)
    ("steps_4095", _zipf((300, 200, 400, 30), 5 * 4095), 16, 5),
    ("steps_4096", _zipf((300, 200, 400, 30), 5 * 4096), 16, 5),
    ("steps_4096_r32", _zipf((300, 200, 400, 30), 300 * 4096), 32, 300),
    ("longer_eight_modes", _zipf((9, 8, 7, 6, 5, 4, 3, 2), 20_000), 16, 2),
]


@pytest.mark.parametrize("name,shape,R,kappa", SHAPES, ids=[s[0] for s in SHAPES])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_split_of_partitions(name, shape, R, kappa, dtype):
    print("case", name, dtype, flush=True)
    dims, idx = shape
    val = synth.normal(3, 1, idx.shape[1]).astype(np.float32)
    Y = synth.random_factors(dims, R, seed=18)
    exact = [oracle.bf16_round(y) for y in Y] if dtype == "bf16" else Y
    given = [torch.from_numpy(y).cuda().to(torch.bfloat16 if dtype == "bf16" else torch.float32) for y in Y]
    t = S.tensor_load_coo(dims, idx, val, kappa=kappa, prep="device")
    for d in range(len(dims)):
        out = torch.full((dims[d], R), float("nan"), device="cuda")
        S.mttkrp(t, d, given, out, flags=S.FUSE_REMAP_NEXT)
        ref = oracle.mttkrp(dims, idx, val, exact, d)
        check_elementwise(out.cpu().numpy(), ref, mttkrp_abs(dims, idx, val, exact, d), label=f"{name} mode {d}")
    t.free()


ALS = [
    # name, dims, nnz, rank, kappa (8 waves in turn up to 256, 2 up to 2047, then one), wide layout
    ("three_modes", (300, 200, 4000), 60_000, 16, 49, "word32"),
    ("kappa256", (300, 200, 4000), 60_000, 32, 256, "word32"),
    ("kappa257", (300, 200, 4000), 60_000, 32, 257, "word32"),
    ("kappa2047", (300, 200, 4000), 60_000, 8, 2047, "word32"),
    ("kappa2048", (300, 200, 4000), 60_000, 8, 2048, "word32"),
    ("four_modes", (300, 200, 400, 90), 60_000, 64, 300, "half16"),
    ("one_partition", (300, 200, 400, 90), 9_000, 64, 1, "half16"),
]


@pytest.mark.parametrize("name,dims,nnz,R,kappa,wide", ALS, ids=[c[0] for c in ALS])
@pytest.mark.parametrize("bf16", [False, True], ids=["f32", "bf16"])
def test_als_sums_keep_the_order_of_one_wave(name, dims, nnz, R, kappa, wide, bf16):
    """Wide records have no ordered form: one wave per partition computes them.
    The same sweep on 12-byte records must give the same bits."""
    print("case", name, bf16, flush=True)
    idx, val = synth.random_coo(dims, nnz, seed=5, dist="zipf", zipf_s=0.7)
    Y = synth.random_factors(dims, R, seed=18)
    res = []
    for layout in ("auto", wide):
        t = S.tensor_load_coo(dims, idx, val, kappa=kappa, prep="device", layout=layout)
        f = [torch.from_numpy(y).cuda() for y in Y]
        lam = torch.empty(R, dtype=torch.float64, device="cuda")
        fits = [S.cp_als_iter(t, f, lam, bf16_gather=bf16) for _ in range(2)]
        res.append((fits, lam.cpu().numpy(), [x.cpu().numpy() for x in f]))
        t.free()
    assert res[0][0] == res[1][0]
    assert np.array_equal(res[0][1], res[1][1])
    for a, b in zip(res[0][2], res[1][2]):
        assert np.array_equal(a.view(np.uint32), b.view(np.uint32))
