"""Which course the library takes by itself where a rule on sizes decides, seen by the launches of each kernel."""
import pytest
import torch

from paper_2605_13473_amd import binding as ob
from paper_2605_13473_amd.inputs import make_stress_inputs
from tests.gpu_util import to_dev

pytestmark = pytest.mark.gpu

NAMES = ("q", "k", "v", "beta", "log_alpha", "retention", "d_in", "S_in")


def launches(chains, T, K, V, bf16, hp=ob.Hyper(), retention=None):
    """Launches per kernel of one forward and one backward call."""
    H = 8 if chains % 8 == 0 else 1
    x = make_stress_inputs(chains // H, T, H, K, V, seed=5, bf16=bf16, retention=0.97)
    if retention is None:
        x["retention"] = None
    t = to_dev(x, bf16)
    ob.osdn_profile_enable(True)
    try:
        *_, ctx = ob.forward(*[t[n] for n in NAMES], hp, for_backward=True)
        torch.cuda.synchronize()
        fwd = {n: c for n, (_, c) in ob.osdn_profile_read().items() if c}
        ob.backward(ctx, t["dO"])
        torch.cuda.synchronize()
        bwd = {n: c for n, (_, c) in ob.osdn_profile_read().items() if c}
    finally:
        ob.osdn_profile_enable(False)
    return fwd, bwd


@pytest.mark.parametrize("chains,K,V,bf16,solved", [
    (32, 128, 128, True, True), (33, 128, 128, True, True), (48, 128, 128, True, True), (56, 128, 128, True, False),
    (64, 128, 64, True, True), (33, 64, 64, True, True), (64, 64, 128, True, True), (65, 64, 64, True, False),
    (32, 64, 64, False, True), (33, 64, 64, False, False)])
def test_solved_form_without_retention(chains, K, V, bf16, solved):
    _, bwd = launches(chains, 1024, K, V, bf16)
    assert ("precond_lin" in bwd) == solved and ("precond_mask" in bwd) != solved
