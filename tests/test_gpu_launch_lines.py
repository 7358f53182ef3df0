"""The elementwise kernel on both sides of the lines its launch draws by the number
of partitions and the nonzeros in them (1, 4 or 8 waves per partition; 1, 2 or 4
records per lane and step), by the share of nonzeros that repeat the row and last
index of the one before (the reuse form with 3 modes), by the bytes gathered and
by the number of modes (2 modes: never the reuse form), against the oracle.
Tolerance: 1e-5 of M_abs per element.
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

FEW, MANY = (0.0, 0.1), (0.4, 1.0)  # shares of repeats, every mode of the case

CASES = [
    # name, dims, nonzeros, dist, rank, kappa, shares
    # nonzeros per partition around the lines at up to 256, 512, 1024 and 2048 partitions
    ("w256_8", (300, 200, 4000), 256 * 512, "zipf", 16, 256, None),
    ("w256_4", (300, 200, 4000), 256 * 511, "zipf", 16, 256, None),
    ("w256_1", (300, 200, 4000), 256 * 127, "zipf", 16, 256, None),
    ("w512_4", (300, 200, 400, 30), 512 * 160, "zipf", 16, 512, None),
    ("w512_1", (300, 200, 400, 30), 512 * 159, "zipf", 16, 512, None),
    ("w1024_4", (300, 200, 400, 30), 1024 * 160, "zipf", 64, 1024, None),
    ("w1024_1", (300, 200, 400, 30), 1024 * 159, "zipf", 64, 1024, None),
    ("w2048_4", (90, 80, 70, 30, 9), 2048 * 252, "zipf", 64, 2048, None),
    ("w2048_1", (90, 80, 70, 30, 9), 2048 * 251, "zipf", 64, 2048, None),
    ("w4096_4", (9, 8, 7, 6, 5, 4, 3, 2), 4096 * 358, "zipf", 64, 4096, None),
    ("w4096_1", (9, 8, 7, 6, 5, 4, 3, 2), 4096 * 357, "zipf", 64, 4096, None),
    # steps of one record: fewer than 256 nonzeros per partition, or few shared rows
    # beyond 6 MB of gathered rows at 1025 to 2048 partitions
    ("steps_255", (300, 200, 4000), 300 * 255, "zipf", 16, 300, None),
    ("steps_256", (300, 200, 4000), 300 * 256, "zipf", 16, 300, None),
    ("crowded", (300_000, 200_000), 1025 * 300, "uniform", 16, 1025, FEW),
    ("not_crowded", (60_000, 50_000), 1025 * 300, "uniform", 16, 1025, FEW),
    # the reuse form with 3 modes: long rows above 256 partitions, any from 4096 on
    ("reuse3_256", (30, 20, 10), 256 * 300, "zipf", 64, 256, MANY),
    ("reuse3_257", (30, 20, 10), 257 * 300, "zipf", 64, 257, MANY),
    ("reuse3_r128", (30, 20, 10), 257 * 60, "zipf", 128, 257, MANY),
    ("reuse3_4095", (40, 30, 20), 4095 * 900, "zipf", 128, 4095, MANY),
    ("reuse3_4096", (40, 30, 20), 4096 * 900, "zipf", 128, 4096, MANY),
    ("reuse3_4096_r32", (40, 30, 20), 4096 * 1800, "zipf", 32, 4096, MANY),
    # two modes, of which nearly every nonzero repeats the row before it
    ("two_modes", (400, 6), 300 * 300, "zipf", 64, 300, MANY),
    ("two_modes_4096", (400, 6), 4096 * 60, "zipf", 16, 4096, MANY),
]


@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_both_sides_of_the_launch_lines(case, dtype):
    name, dims, nnz, dist, R, kappa, shares = case
    print("case", name, dtype, flush=True)
    idx, _ = synth.random_coo(dims, nnz, seed=5, dist=dist, zipf_s=1.1)
    val = synth.normal(3, 1, nnz).astype(np.float32)
    Y = synth.random_factors(dims, R, seed=18)
    exact = [oracle.bf16_round(y) for y in Y] if dtype == "bf16" else Y
    given = [torch.from_numpy(y).cuda().to(torch.bfloat16 if dtype == "bf16" else torch.float32) for y in Y]
    t = S.tensor_load_coo(dims, idx, val, kappa=kappa, prep="device")
    for d in range(len(dims)):
        if shares:
            i = S.tensor_get_records(t)[0]
            share = float(((i[d][1:] == i[d][:-1]) & (i[d - 1][1:] == i[d - 1][:-1])).mean())
            assert shares[0] <= share <= shares[1], (d, share)
        out = torch.full((dims[d], R), float("nan"), device="cuda")
        S.mttkrp(t, d, given, out, flags=S.FUSE_REMAP_NEXT)
        ref = oracle.mttkrp(dims, idx, val, exact, d)
        check_elementwise(out.cpu().numpy(), ref, mttkrp_abs(dims, idx, val, exact, d), label=f"{name} mode {d}")
    t.free()
