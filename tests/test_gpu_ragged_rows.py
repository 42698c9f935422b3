"""Results of ragged sequences go straight to the caller's rows: they are what the same call on inputs
padded to whole chunks by the caller gives, bit for bit, and nothing is written around them."""
import pytest
import torch

from paper_2605_13473_amd import binding as ob
from paper_2605_13473_amd.inputs import make_stress_inputs
from tests.gpu_util import to_dev

pytestmark = pytest.mark.gpu
NAMES = ("q", "k", "v", "dO", "beta", "log_alpha", "retention")


def _call(t, hp, cu, B, T, H, K, V, bf16, vec):
    """Forward and backward into buffers with 64 guard rows at both ends; the results, guards checked."""
    guards = []

    def out(like):
        n, row = like.shape[0] * like.shape[1], like[0, 0].numel()
        buf = torch.full(((n + 128) * row,), 7.0, dtype=like.dtype, device=like.device)
        guards.append((buf, 64 * row))
        return buf[64 * row:(n + 64) * row].view(like.shape)

    p = ob.make_params(B, T, H, K, V, bf16, hp, retention_per_channel=vec, gate_per_channel=vec)
    nb = B if cu is None else len(cu) - 1
    f32 = dict(dtype=torch.float32, device="cuda")
    n = ob.osdn_workspace_bytes(p, True) if cu is None else ob.osdn_workspace_bytes_packed(p, cu, True)
    ws = torch.empty(n, dtype=torch.uint8, device="cuda")
    inputs = tuple(t[x] for x in ("q", "k", "v", "beta", "log_alpha", "retention")) + (None, None)
    fwd = (out(t["v"]), torch.empty(nb, H, V, K, **f32), torch.empty(nb, H, K, **f32))
    grads = tuple(out(t[x]) for x in ("q", "k", "v", "beta", "log_alpha", "retention")) + (
        torch.empty(nb, H, K, **f32), torch.empty(nb, H, V, K, **f32))
    if cu is None:
        ob.osdn_fwd(p, *inputs, *fwd, ws)
        ob.osdn_bwd(p, *inputs, t["dO"], None, None, *grads, ws)
    else:
        ob.osdn_fwd_packed(p, *inputs, *fwd, cu, ws)
        ob.osdn_bwd_packed(p, *inputs, t["dO"], None, None, *grads, cu, ws)
    for buf, g in guards:
        assert (buf[:g] == 7).all() and (buf[-g:] == 7).all()
    return fwd + grads


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("vec", [False, True])
@pytest.mark.parametrize("K,V", [(64, 64), (128, 192)])
@pytest.mark.parametrize("lens,packed", [([1, 1], False), ([65, 65], False), ([127, 127], False),
                                         ([63, 64, 1, 130, 65], True)])
def test_ragged_equals_padded_by_the_caller(lens, packed, K, V, vec, bf16):
    H = 2
    B, T = (1, sum(lens)) if packed else (len(lens), lens[0])
    x = make_stress_inputs(B, T, H, K, V, seed=T + K, bf16=bf16, retention=0.97)
    t = to_dev({n: x[n] for n in NAMES}, bf16)
    if vec:                                     # one gate per key channel, one retention per coordinate
        for n in ("log_alpha", "retention"):
            t[n] = t[n].unsqueeze(-1).expand(B, T, H, K).contiguous()
        t["log_alpha"] = t["log_alpha"].clamp(min=-0.5)
    # rows of the padded axis, whole chunks per sequence
    start, rows, at, cu, cup = 0, [], 0, [0], [0]
    for n in lens:
        rows.append(torch.arange(at, at + n))
        start += n
        at += -(-n // 64) * 64
        cu.append(start)
        cup.append(at)
    if packed:
        idx, Tp = torch.cat(rows).cuda(), at
    else:
        idx, Tp = torch.arange(T).cuda(), -(-T // 64) * 64
        cu = cup = None

    def pad(a, fill):
        o = torch.full((B, Tp, *a.shape[2:]), fill, dtype=a.dtype, device=a.device)
        o[:, idx] = a
        return o
    tp = {n: pad(a, 1.0 if n == "retention" else 0.0) for n, a in t.items()}
    hp = ob.Hyper(eta=0.5, segments=1)
    got = _call(t, hp, cu, B, T, H, K, V, bf16, vec)
    want = _call(tp, hp, cup, B, Tp, H, K, V, bf16, vec)
    token_wise = (0, 3, 4, 5, 6, 7, 8)          # o and the gradients of the token inputs
    for i, (g, w) in enumerate(zip(got, want)):
        assert torch.equal(g, w[:, idx] if i in token_wise else w), i


@pytest.mark.parametrize("bf16,offset", [(False, 4), (True, 2), (True, 8)])
@pytest.mark.parametrize("vec", [False, True])
@pytest.mark.parametrize("lens,packed,H,K,V", [([65, 65], False, 2, 128, 64), ([321], False, 2, 64, 128), ([127, 1, 64, 200], True, 2, 128, 128),
                                               ([77] * 70, True, 4, 64, 64)])
def test_ragged_tensors_off_a_16_byte_boundary(lens, packed, H, K, V, vec, bf16, offset):
    """q, k, v and dO of ragged calls are read where they are: off a 16-byte boundary, with rows that are not numbers on both
    sides of them, they give what aligned tensors give (few chains and many, slices of 16 and of 32 values)."""
    B, T = (1, sum(lens)) if packed else (len(lens), lens[0])
    x = make_stress_inputs(B, T, H, K, V, seed=T + V, bf16=bf16, retention=0.97)
    t = to_dev({n: x[n] for n in NAMES}, bf16)
    if vec:
        for n in ("log_alpha", "retention"):
            t[n] = t[n].unsqueeze(-1).expand(B, T, H, K).contiguous()
        t["log_alpha"] = t["log_alpha"].clamp(min=-0.5)
    cu = None
    if packed:
        cu = [0]
        for n in lens:
            cu.append(cu[-1] + n)

    def shifted(a):
        row = a[0, 0].numel()
        at = 64 * row + offset // a.element_size()
        buf = torch.full((a.numel() + 129 * row,), float("nan"), dtype=a.dtype, device=a.device)
        out = buf[at:at + a.numel()].view(a.shape)
        out.copy_(a)
        assert out.data_ptr() % 16 == offset
        return out

    hp = ob.Hyper(eta=0.3)
    moved = {n: shifted(a) if n in ("q", "k", "v", "dO") else a for n, a in t.items()}
    for a, b in zip(_call(t, hp, cu, B, T, H, K, V, bf16, vec), _call(moved, hp, cu, B, T, H, K, V, bf16, vec)):
        assert torch.isfinite(a).all() and torch.equal(a, b)
