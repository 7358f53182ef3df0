"""A handle of the device planner holds the device memory of the host planner's
and gives the same remap ids: nothing of the load is left on the device for
spt_tensor_get_remap.  Sizes: none, one and many nonzeros, and both sides of the
line from which the remap ids are copied beside the rest of the load (2^21).
"""
import numpy as np
import pytest

from paper_2405_08470_amd import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)
S = pytest.importorskip("paper_2405_08470_amd.spmttkrp")


@pytest.mark.parametrize("nnz", [0, 1, 100_000, (1 << 21) - 1, 1 << 21])
@pytest.mark.parametrize("kw", [{}, {"remap": "fused"}, {"copies": 1}], ids=["staged", "fused", "copies"])
def test_device_planner_holds_no_more_than_the_host_planner(nnz, kw):
    print("case", nnz, kw, flush=True)
    dims = (700, 300, 500)
    idx, val = synth.random_coo(dims, max(nnz, 1), seed=9, dist="zipf", zipf_s=1.1)
    idx, val = idx[:, :nnz], val[:nnz]
    host, device = (S.tensor_load_coo(dims, idx, val, prep=p, **kw) for p in ("host", "device"))
    held = [S.tensor_info(t)["device_bytes"] for t in (host, device)]
    assert held[1] <= held[0] + 16 * len(dims)  # (an empty buffer may count 4 or 16 bytes)
    if not kw.get("copies"):
        for d in range(len(dims)):
            assert np.array_equal(S.tensor_get_remap(host, d), S.tensor_get_remap(device, d))
    host.free()
    device.free()
