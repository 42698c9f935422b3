"""Without retention the forward sweep marks the chunks whose coordinates stay well off the box, and the backward pass takes
every decision of such a chunk as "inside" without a replay: that it does so, that a replay would find the same, and that a chunk which
stands close to a face is not swept more often for it."""
import numpy as np
import pytest
import torch

from paper_2605_13473_amd import binding as ob
from paper_2605_13473_amd.inputs import make_stress_inputs
from tests.gpu_util import gpu_box_decisions, to_dev

pytestmark = pytest.mark.gpu


def _forward(x, hp, d_in=None):
    t = to_dev(x, False)
    d = t["d_in"] if d_in is None else torch.from_numpy(d_in).cuda()
    _, _, d_out, ctx = ob.forward(t["q"], t["k"], t["v"], t["beta"], t["log_alpha"], None, d, t["S_in"], hp, for_backward=True)
    return t, ctx, d_out


def _decisions(t, ctx, T):
    ob.backward(ctx, t["dO"])
    torch.cuda.synchronize()
    return gpu_box_decisions(ctx, T)


@pytest.mark.parametrize("K", [64, 128])
def test_a_marked_chunk_is_not_replayed(K):
    """The backward pass is handed keys a thousand times as long: a replay of them leaves the box."""
    T = 64 * 4
    x = make_stress_inputs(1, T, 3, K, 64, seed=181, bf16=False, retention=0.97)
    x["k"] /= np.linalg.norm(x["k"], axis=-1, keepdims=True)
    d = np.ones((1, 3, K), np.float32)
    d[0, 1, 3] = 2.0                                                  # on a face: swept with the box, not marked
    d[0, 2, 5] = np.float32(2.0) * np.float32(1 - 1e-5)               # within the margin: swept without it, not marked
    t, ctx, _ = _forward(x, ob.Hyper(eta=1e-6, p1_solved=-1, segments=1), d)
    q, k, *rest = ctx["inputs"]
    ctx["inputs"] = (q, 1000.0 * k, *rest)
    inside = _decisions(t, ctx, T).reshape(1, 4, 64, 3, K)
    assert inside[..., 0, :].all()
    for h in (1, 2):
        assert not inside[:, :, :, h].all(axis=(2, 3)).any(), "a chunk that has to be replayed was not"


@pytest.mark.parametrize("lo", [-4.0, -float("inf")])
@pytest.mark.parametrize("K", [64, 128])
def test_a_replay_decides_the_same_next_to_a_small_upper_face(K, lo):
    """Every chain has one coordinate that ends at zero, the face, to within rounding: that of the sums, not that of the face.  (So small
    an eta that the first sweep is as good as the last: one that goes past the face is done again with the box.)  The solved form's
    first kernel replays every chunk."""
    B, T, H = 8, 64, 8
    x = make_stress_inputs(B, T, H, K, 64, seed=185, bf16=False, retention=0.97)
    x["k"] /= np.linalg.norm(x["k"], axis=-1, keepdims=True)
    rise = _forward(x, ob.Hyper(eta=1e-7, d_min=lo, d_max=1.0), np.zeros((B, H, K), np.float32))[2].cpu().numpy()
    near = np.arange(K) == np.random.default_rng(186).integers(0, K, (B, H, 1))
    d = np.where(near, -rise, -2 * rise)
    got = []
    for solved in (1, -1):
        t, ctx, _ = _forward(x, ob.Hyper(eta=1e-7, d_min=lo, d_max=0.0, p1_solved=solved, segments=1), d)
        got.append(_decisions(t, ctx, T))
    assert np.array_equal(*got), f"{int((got[0] != got[1]).sum())} decisions differ"


def _sweeps(ctx, x):
    """How many sweeps every chunk took [B,N,H]: the fourth of a token's scalars, next to its sum k^2."""
    n = torch.from_numpy((x["k"].astype(np.float64) ** 2).sum(-1).astype(np.float32)).cuda().flatten()
    w = ctx["workspace"][:ctx["workspace"].numel() // 16 * 16].view(torch.float32).view(-1, 4)
    first = torch.nonzero((w[:, 2].abs() - n[0]).abs() <= 1e-5 * n[0]).flatten().tolist()
    at = [i for i in first if i + n.numel() <= len(w) and bool(((w[i:i + n.numel(), 2].abs() - n).abs() <= 1e-5 * n).all())]
    assert len(at) == 1
    B, T, H = x["k"].shape[:3]
    return w[at[0]:at[0] + n.numel(), 3].reshape(B, T // 64, 64, H)[:, :, 0].cpu().numpy()


@pytest.mark.parametrize("K", [64, 128])
def test_a_chain_that_stands_close_to_a_face_is_not_swept_in_vain(K):
    x = make_stress_inputs(1, 256, 3, K, 64, seed=183, bf16=False, retention=0.97)
    x["k"] /= np.linalg.norm(x["k"], axis=-1, keepdims=True)
    x["beta"] *= np.float32(0.4)                                      # (beta |k|^2 d below 1: no step down)
    d = np.ones((1, 3, K), np.float32)
    d[0, 1] = np.float32(2.0) * np.float32(1 - 1.5e-5)
    d[0, 2] = np.float32(0.5) * np.float32(1 + 1.5e-5)
    _, ctx, _ = _forward(x, ob.Hyper(eta=1e-8, segments=1), d)
    torch.cuda.synchronize()
    sweeps = _sweeps(ctx, x)
    assert (sweeps == sweeps[..., :1]).all(), sweeps
