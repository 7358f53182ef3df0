"""The adjoint leaves the residual stream in the last mode's order and the next
adjoint starts from there: repeated adjoints of one loss give the same bits,
for both forms of the remap and one copy per mode, and a new loss starts over.
The loss kernel takes several nonzeros a turn: sizes around the turn of a
group, against the oracle.
"""
import numpy as np
import pytest

import oracle
from paper_2405_08470_amd import synth
from parity import check_grad_elements

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)
S = pytest.importorskip("paper_2405_08470_amd.spmttkrp")


@pytest.mark.parametrize("dims", [(60, 50), (300, 200, 400), (90, 80, 70, 6), (50, 40, 30, 20, 10)], ids=len)
@pytest.mark.parametrize("kw", [{}, {"remap": "fused"}, {"copies": 1}], ids=["staged", "fused", "copies"])
def test_repeated_adjoints(dims, kw):
    print("case", dims, kw, flush=True)
    idx, val = synth.random_coo(dims, 2000, seed=7, dist="zipf", zipf_s=1.1)
    Y = [0.5 * y for y in synth.random_factors(dims, 16, seed=18)]
    f = [torch.from_numpy(y).cuda() for y in Y]
    t = S.tensor_load_coo(dims, idx, val, **kw)
    want = [g.cpu().numpy().view(np.uint32) for g in S.cp_gradient(t, f)[1]]
    for _ in range(len(dims)):
        for a, b in zip(S.cp_adjoint(t, f), want):
            assert np.array_equal(a.cpu().numpy().view(np.uint32), b)
    S.cp_loss(t, f)
    for a, b in zip(S.cp_adjoint(t, f), want):
        assert np.array_equal(a.cpu().numpy().view(np.uint32), b)
    t.free()


@pytest.mark.parametrize("nnz", [1, 63, 64, 65, 257, 4097])
@pytest.mark.parametrize("N,R", [(2, 8), (4, 16), (5, 64)])
def test_loss_at_turn_edges(N, R, nnz):
    print("case", N, R, nnz, flush=True)
    dims = (40, 30, 20, 15, 10)[:N]
    idx, val = synth.random_coo(dims, nnz, seed=nnz, dist="zipf", zipf_s=1.1)
    Y = [0.5 * y for y in synth.random_factors(dims, R, seed=18)]
    f = [torch.from_numpy(y).cuda() for y in Y]
    t = S.tensor_load_coo(dims, idx, val)
    loss, grads = S.cp_gradient(t, f)
    r = oracle.model_at(idx, Y) - val.astype(np.float64)
    # the residuals' FP32 rounding, as in check_grad_elements
    m_abs = oracle.model_at(idx, [np.abs(y) for y in Y]) + np.abs(val)
    bound = float((np.abs(r) * (R + N + 2) * 2.0 ** -24 * m_abs).sum()) * 1.01
    assert abs(loss.item() - 0.5 * float((r * r).sum())) <= bound
    check_grad_elements(dims, idx, val, Y, [g.cpu().numpy() for g in grads])
    t.free()
