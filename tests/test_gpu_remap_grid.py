"""The remap pass around the chunk count from which workgroups are dealt to the
XCDs by chunk (8 chunks of 131072 12-byte records), and the tables of chunks
with 1, 2, 3 and 32 sorted runs: every record where the remap ids put it, bit
for bit.
"""
import numpy as np
import pytest

from paper_2405_08470_amd import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)
S = pytest.importorskip("paper_2405_08470_amd.spmttkrp")

CHUNK = 131072


@pytest.mark.parametrize("nnz", [4095, 4097, 3 * 4096, CHUNK, 7 * CHUNK, 7 * CHUNK + 1, 8 * CHUNK, 8 * CHUNK + 1])
def test_remap_pass_at_chunk_counts(nnz):
    print("nnz", nnz, flush=True)
    dims = (700, 900, 1100)
    idx, val = synth.random_coo(dims, nnz, seed=nnz % 97, dist="zipf", zipf_s=1.1)
    t = S.tensor_load_coo(dims, idx, val, prep="device")
    assert S.tensor_info(t)["remap_chunk"] == CHUNK
    for mode in (1, 2, 0):
        S.remap_for_mode(t, mode)
        ridx, rval, cur = S.tensor_get_records(t)
        b = S.tensor_get_remap(t, mode)
        assert cur == mode
        assert np.array_equal(ridx[:, b], idx) and np.array_equal(rval[b].view(np.uint32), val.view(np.uint32))
    t.free()
