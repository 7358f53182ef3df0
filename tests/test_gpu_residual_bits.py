"""The forward kernel of the gradient fit holds its written order of roundings on
the GPU, bit for bit, for every mode count, rank and record layout (the
expression and the way the residuals are read: test_cpu_replay).
"""
import numpy as np
import pytest

from test_cpu_replay import readable_residuals, written_residuals

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)
S = pytest.importorskip("paper_2405_08470_amd.spmttkrp")

LAYOUTS = [(N, lay) for N, lays in {2: ("word32",), 3: ("word32",), 4: ("half16", "packed", "word32"),
                                    5: ("half16", "packed", "word32"), 6: ("half16", "packed", "word32"),
                                    7: ("word32",), 8: ("half16", "word32")}.items() for lay in ("auto",) + lays]


@pytest.mark.parametrize("R", [8, 16, 32, 64])
@pytest.mark.parametrize("N,layout", LAYOUTS)
def test_residuals_have_the_written_roundings(N, layout, R):
    print("case", N, layout, R, flush=True)
    dims, idx, val, Y = readable_residuals(N, R, 300)
    want = written_residuals(idx, val, Y)
    f = [torch.from_numpy(y).cuda() for y in Y]
    for copies in (0, 1):
        t = S.tensor_load_coo(dims, idx, val, layout=layout, copies=copies)
        loss, grads = S.cp_gradient(t, f)
        assert np.array_equal(grads[0].cpu().numpy()[idx[0], 0].view(np.uint32), want.view(np.uint32))
        r = want.astype(np.float64)
        assert abs(loss.item() - 0.5 * (r * r).sum()) <= 1e-13 * loss.item()
        t.free()
