"""The reverse sweep of phase 1 (precond_chain) in its two courses: a chunk whose sigma settles in two sweeps
goes on before its verdict is known, one that does not is fetched and done again (the last and the only chunk of a
launch among them), at every retention form, with clean and mixed masks in one workgroup, over segments."""
import numpy as np
import pytest

from paper_2605_13473_amd import binding as ob
from paper_2605_13473_amd.inputs import make_stress_inputs
from tests.gpu_util import compare_backward

pytestmark = pytest.mark.gpu


# eta = 1: one sweep moves sigma by more than a tenth of itself, no chunk settles in two (0.003: all do)
@pytest.mark.parametrize("eta", [0.003, 1.0])
@pytest.mark.parametrize("retention", ["none", "head", "channel"])
@pytest.mark.parametrize("K", [64, 128])
def test_chunks_that_settle_and_chunks_that_do_not(K, retention, eta):
    rng = np.random.Generator(np.random.Philox(7))
    for T, segments in ((64, 1), (128, 1), (128, 2), (200, 1), (449, 3)):
        x = make_stress_inputs(2, T, 2, K, 64, seed=171 + T, bf16=False, retention=0.97)
        if retention == "none":
            x["retention"] = None
        elif retention == "channel":
            x["retention"] = rng.uniform(0.9, 1.0, (2, T, 2, K)).astype(np.float32)
        x["k"][:, T // 2:] *= np.float32(1e-2) if T == 200 else np.float32(1.0)     # tiny sigma beside large
        dd = rng.standard_normal((2, 2, K)).astype(np.float32)
        compare_backward(x, ob.Hyper(eta=eta, p1_solved=-1, segments=segments), False, dd_out=dd)


def test_no_box_and_no_gradient():
    """No masks are written without a box; a zero adjoint (sigma = 0 throughout) settles at once."""
    x = make_stress_inputs(1, 192, 2, 128, 64, seed=181, bf16=True, retention=0.97)
    compare_backward(x, ob.Hyper(eta=0.3, d_min=1.0, d_max=0.0, p1_solved=-1, segments=1), True)
    x["dO"][:] = 0
    compare_backward(x, ob.Hyper(eta=0.3, p1_solved=-1, segments=1), True)
