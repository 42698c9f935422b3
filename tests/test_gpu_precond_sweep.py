"""Phase 1 where its sweeps change form: without retention a chunk that begins inside the box is swept
without it, and again with it if a coordinate met a face.  d starts inside, on a face and outside
the box, rises to the upper face in the middle of a run of tokens, is pushed down by tokens whose step is
negative, or has no box at all; lengths end inside a run, inside a chunk and on their edges."""
import numpy as np
import pytest
import torch

import oracle
from paper_2605_13473_amd import binding as ob
from paper_2605_13473_amd.inputs import make_stress_inputs
from tests.gpu_util import check, compare_forward, oracle_hp, to_dev

pytestmark = pytest.mark.gpu


def _case(case, T, K, bf16):
    x = make_stress_inputs(2, T, 2, K, 64, seed=161, bf16=bf16, retention=0.0)
    x["retention"] = None
    hp = ob.Hyper(eta=0.003)
    u = (x["d_in"] - x["d_in"].min()) / np.ptp(x["d_in"])
    x["d_in"] = (0.9 + 0.2 * u).astype(np.float32)          # well inside [0.5, 2]
    if case == "on_faces":
        x["d_in"][:, :, ::7] = 2.0
        x["d_in"][:, :, 3::11] = 0.5
    elif case == "outside":
        x["d_in"][:, :, 5] = 2.5
        x["d_in"][:, :, K - 1] = 0.25
    elif case == "meets_upper_face":
        x["d_in"][0, :, 1] = 1.999
        hp = ob.Hyper(eta=0.05)
    elif case == "negative_steps":                           # p = <d, k^2> well above 1 / beta
        x["d_in"] = (1.7 + 0.2 * u).astype(np.float32)
        hp = ob.Hyper(eta=0.5)
    elif case == "no_projection":
        hp = ob.Hyper(eta=0.05, d_min=1.0, d_max=0.0)
    return x, hp


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("K", [64, 128])
@pytest.mark.parametrize("case", ["inside", "on_faces", "outside", "meets_upper_face", "negative_steps", "no_projection"])
def test_sweeps_with_and_without_the_box(case, K, bf16):
    for T in (1, 8, 9, 63, 64, 65, 321):
        x, hp = _case(case, T, K, bf16)
        t = to_dev(x, bf16)
        kt, d_out, *ck = ob.precond_update(t["k"], t["beta"], None, t["d_in"], hp, want_ckpt=T % 64 == 0)
        torch.cuda.synchronize()
        okt, od, traj = oracle.precond(x["k"], x["beta"], None, x["d_in"], oracle_hp(hp), want_traj=True)
        check("k_tilde", kt, okt, bf16)
        check("d_out", d_out, od, False)
        if ck:
            check("d_ckpt", ck[0], traj[:, ::64].transpose(0, 2, 1, 3), False)
    compare_forward(x, hp, bf16)                             # the same sweeps inside a forward pass (padded tiles)


@pytest.mark.parametrize("case", ["inside", "meets_upper_face"])
def test_carried_d_is_bit_for_bit_across_calls(case):
    """With or without the box must follow from d alone, not from the chunks that the same call did before."""
    x, hp = _case(case, 256, 128, True)
    t = to_dev(x, True)
    kt, d_out = ob.precond_update(t["k"], t["beta"], None, t["d_in"], hp)
    d, parts = t["d_in"], []
    for cut in range(0, 256, 64):
        k1, d = ob.precond_update(t["k"][:, cut:cut + 64].contiguous(), t["beta"][:, cut:cut + 64].contiguous(), None, d, hp)
        parts.append(k1)
    assert torch.equal(torch.cat(parts, 1), kt) and torch.equal(d, d_out)


def _sweeps(x, hp):
    """Sweeps that each chunk of a forward pass took, [chains, chunks] (fourth scalar that is kept per token)."""
    t = to_dev(x, False)
    B, T, H, K = x["k"].shape
    p = ob.make_params(B, T, H, K, x["v"].shape[-1], False, hp)
    ws = torch.empty(ob.osdn_workspace_bytes(p, True), dtype=torch.uint8, device="cuda")
    ob.forward(*[t[n] for n in ("q", "k", "v", "beta", "log_alpha", "retention", "d_in", "S_in")], hp, workspace=ws, for_backward=True)
    torch.cuda.synchronize()
    at = B * T * H * K * 4 + B * H * T // 64 * K * 4         # behind k~ and the checkpoints of d
    sc = ws[at:at + B * T * H * 16].view(torch.float32).view(B, T // 64, 64, H, 4)[..., 3]
    assert torch.equal(sc, sc[:, :, :1].expand_as(sc)) and int(sc.min()) >= 1
    return sc[:, :, 0].permute(0, 2, 1).reshape(B * H, T // 64).cpu().numpy()


@pytest.mark.parametrize("K", [64, 128])
def test_first_guess_where_d_fades_and_where_the_face_holds_it(K):
    """d = 1 fades with gates of 0.999 (two sweeps: the guess knows the gates), reaches the lower face, and lies there (one)."""
    T = 64 * 16
    x = make_stress_inputs(1, T, 2, K, 64, seed=163, bf16=False, retention=0.97)
    x["retention"] = np.full((1, T, 2), 0.999, np.float32)
    x["d_in"] = np.ones((1, 2, K), np.float32)
    hp = ob.Hyper(eta=1e-4, p1_pieces=-1, segments=1)
    n = _sweeps(x, hp)
    assert (n[:, :10] <= 2).all() and (n[:, 12:] == 1).all(), n
    x["retention"][:] = 0.97                                 # on the face within a chunk
    n = _sweeps(x, hp)
    assert (n[:, 1:] == 1).all(), n
    compare_forward(x, hp, False)


def test_first_guess_with_a_large_eta():
    """The updates hold d up against gates of 0.999: no more sweeps than with gates of 1 (a chunk in twenty may differ)."""
    x = make_stress_inputs(2, 64 * 16, 4, 64, 64, seed=165, bf16=False, retention=0.97)
    total = {}
    for gate in (1.0, 0.999):
        x["retention"] = np.full((2, 64 * 16, 4), gate, np.float32)
        total[gate] = float(_sweeps(x, ob.Hyper(eta=1.0, p1_pieces=-1, segments=1)).sum())
    assert total[0.999] <= 1.05 * total[1.0], total


def test_carried_d_is_bit_for_bit_across_calls_with_retention():
    """Which first guess a chunk takes must follow from its own d and gates."""
    rng = np.random.Generator(np.random.Philox(13))
    x = make_stress_inputs(1, 64 * 18, 2, 128, 64, seed=167, bf16=True, retention=0.97)
    x["retention"] = (1 - 0.003 * rng.random((1, 64 * 18, 2))).astype(np.float32)
    x["retention"][:, 64 * 14:] = 1.0
    t = to_dev(x, True)
    hp = ob.Hyper(eta=0.003)
    kt, d = ob.precond_update(t["k"], t["beta"], t["retention"], t["d_in"], hp)[:2]
    parts, dd = [], t["d_in"]
    for a, b in ((0, 1), (1, 2), (2, 9), (9, 15), (15, 18)):
        sl = slice(64 * a, 64 * b)
        k2, dd = ob.precond_update(t["k"][:, sl].contiguous(), t["beta"][:, sl].contiguous(), t["retention"][:, sl].contiguous(), dd, hp)[:2]
        parts.append(k2)
    torch.cuda.synchronize()
    assert torch.equal(kt, torch.cat(parts, dim=1)) and torch.equal(d, dd)
