"""A captured adjoint gives the same gradients at every replay, with the program's
own work on the tensor between them: the residual stream is left in mode 0's
order.  2 to 5 modes, both forms of the remap and one copy per mode.
"""
import numpy as np
import pytest

from paper_2405_08470_amd import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)
S = pytest.importorskip("paper_2405_08470_amd.spmttkrp")


@pytest.mark.parametrize("dims", [(60, 50), (300, 200, 400), (90, 80, 70, 6), (50, 40, 30, 20, 10)], ids=len)
@pytest.mark.parametrize("kw", [{}, {"remap": "fused"}, {"copies": 1}], ids=["staged", "fused", "copies"])
def test_captured_adjoint_replays(dims, kw):
    print("case", dims, kw, flush=True)
    idx, val = synth.random_coo(dims, 5000, seed=7, dist="zipf", zipf_s=1.1)
    f = [torch.from_numpy(0.5 * y).cuda() for y in synth.random_factors(dims, 16, seed=18)]
    t = S.tensor_load_coo(dims, idx, val, **kw)
    S.cp_loss(t, f)
    want = [g.clone() for g in S.cp_adjoint(t, f)]
    grads = [torch.empty_like(x) for x in f]
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        S.cp_adjoint(t, f, grads)
    out = [torch.empty_like(x) for x in f]
    for k in range(4):
        for g in grads:
            g.fill_(float("nan"))
        graph.replay()
        for a, b in zip(grads, want):
            assert torch.equal(a, b), k
        if not kw.get("copies"):  # a pass of the tensor's own stream, back to mode 0's order
            for d in range(len(dims)):
                S.mttkrp(t, d, f, out[d], flags=S.FUSE_REMAP_NEXT)
        if k == 2:
            assert np.isfinite(S.cp_loss(t, f).item())
    for a, b in zip(S.cp_adjoint(t, f), want):
        assert torch.equal(a, b)
    torch.cuda.synchronize()
    del graph
    t.free()
