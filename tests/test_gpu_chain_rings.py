"""GPU parity of the chain kernels where their operand rings can go wrong: sequences shorter than,
as long as and just longer than the rings are deep, in one launch and cut into segments, with wide and
narrow slices of the state, and token tensors that do not start on a 16-byte boundary (their tiles
then take the way through registers)."""
import numpy as np
import pytest
import torch

from paper_2605_13473_amd import binding as ob
from paper_2605_13473_amd.inputs import make_stress_inputs
from tests.gpu_util import compare_backward, compare_forward, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("chunks,segments", [(1, 1), (2, 1), (3, 1), (4, 1), (5, 2), (9, 4)])
@pytest.mark.parametrize("shape", [(1, 2, 128, 192), (2, 2, 64, 64)])
def test_short_sequences(shape, chunks, segments, bf16):
    """Few chains: slices of 16 values (the backward pass in bf16: in one piece; cut into segments, slices of 32)."""
    B, H, K, V = shape
    x = make_stress_inputs(B, 64 * chunks, H, K, V, seed=131 + chunks, bf16=bf16, retention=0.97)
    hp = ob.Hyper(eta=0.5, segments=segments)
    compare_forward(x, hp, bf16)
    compare_backward(x, hp, bf16)


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("chunks,segments", [(1, 1), (2, 1), (3, 1), (5, 1), (6, 2)])
@pytest.mark.parametrize("K", [64, 128])
def test_many_chains_wide_slices(K, chunks, segments, bf16):
    """Enough chains for slices of 32 values, forward and backward (but for fp32 at K = 128, whose backward
    pass always takes slices of 16)."""
    x = make_stress_inputs(8, 64 * chunks, 16, K, 64, seed=141 + chunks, bf16=bf16, retention=0.0)
    hp = ob.Hyper(eta=0.5, segments=segments)
    compare_forward(x, hp, bf16)
    compare_backward(x, hp, bf16)


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("K", [64, 128])
def test_many_chains_wide_slices_channel_gate(K, bf16):
    """The same with one state gate per key channel, whose decays travel with K~."""
    x = make_stress_inputs(8, 64 * 4, 16, K, 64, seed=148, bf16=bf16, retention=0.0)
    rng = np.random.default_rng(149)
    x["log_alpha"] = (-0.1 * rng.random((8, 64 * 4, 16, K))).astype(np.float32)
    compare_forward(x, ob.Hyper(eta=0.5, segments=1), bf16)
    compare_backward(x, ob.Hyper(eta=0.5, segments=1), bf16)


@pytest.mark.parametrize("bf16,offset", [(False, 4), (True, 2), (True, 4)])
@pytest.mark.parametrize("B,H,K,V,segments", [(1, 2, 128, 128, 0), (8, 16, 128, 64, 1), (8, 16, 64, 64, 2), (2, 2, 64, 128, 2)])
def test_token_tensors_off_a_16_byte_boundary(B, H, K, V, segments, bf16, offset):
    """q, k, v and dO two or four bytes past a 16-byte boundary give exactly what aligned tensors give:
    few chains and many (slices of 16 and of 32 values), both widths of K, slots refilled within one launch
    and by a second one."""
    x = make_stress_inputs(B, 64 * 5, H, K, V, seed=151, bf16=bf16, retention=0.97)
    t = to_dev({n: x[n] for n in ("q", "k", "v", "dO", "beta", "log_alpha", "retention", "d_in", "S_in")}, bf16)

    def shifted(a):
        skip = offset // a.element_size()
        buf = torch.empty(a.numel() + skip, dtype=a.dtype, device=a.device)
        out = buf[skip:].view(a.shape)
        out.copy_(a)
        assert out.data_ptr() % 16 == offset
        return out

    def run(f):
        o, S, d, ctx = ob.forward(f(t["q"]), f(t["k"]), f(t["v"]), t["beta"], t["log_alpha"], t["retention"], t["d_in"],
                                  t["S_in"], ob.Hyper(eta=0.5, segments=segments), for_backward=True)
        g = ob.backward(ctx, f(t["dO"]))
        torch.cuda.synchronize()
        return [o, S, d] + [g[n] for n in sorted(g)]

    for a, b in zip(run(lambda a: a), run(shifted)):
        assert torch.equal(a, b)


@pytest.mark.parametrize("B,T,H,K,V", [
    (1, 64 * 8, 1, 128, 128),        # as long as the lines are asked for ahead, one and four chunks longer
    (1, 64 * 9, 1, 64, 192),
    (2, 64 * 12, 1, 128, 512),
    (1, 64 * 10 + 5, 2, 128, 64),    # a ragged last chunk; more than 64 lines a slice
    (1, 64 * 8 + 63, 1, 64, 64),
])
@pytest.mark.parametrize("channel_gate", [False, True])
def test_lines_asked_for_ahead(B, T, H, K, V, channel_gate):
    """bf16, few chains: the forward chain kernel with slices of 16, in lengths about the eight chunks by which it asks for lines ahead
    (which it does for longer calls: below)."""
    x = make_stress_inputs(B, T, H, K, V, seed=161, bf16=True, retention=0.97)
    if channel_gate:
        x["log_alpha"] = (-0.1 * np.random.default_rng(162).random((B, T, H, K))).astype(np.float32)
    compare_forward(x, ob.Hyper(eta=0.5, segments=1), True)


@pytest.mark.parametrize("B,T,H,K,V", [
    (4, 64 * 9 + 5, 8, 128, 64),     # 128 workgroups, more than two lines a lane; a ragged last chunk
    (2, 64 * 10, 4, 64, 256),
])
@pytest.mark.parametrize("channel_gate", [False, True])
def test_lines_asked_for_ahead_in_the_backward_pass(B, T, H, K, V, channel_gate):
    """bf16, slices of 16 values, enough workgroups: the backward chain kernel asks ahead too, right to left."""
    x = make_stress_inputs(B, T, H, K, V, seed=163, bf16=True, retention=0.97)
    if channel_gate:
        x["log_alpha"] = (-0.1 * np.random.default_rng(164).random((B, T, H, K))).astype(np.float32)
    compare_backward(x, ob.Hyper(eta=0.5, segments=1), True)


@pytest.mark.parametrize("bf16", [True, False])
@pytest.mark.parametrize("B,T,H,K,V", [
    (1, 64 * 3, 9, 128, 64),         # filled up to 16 chains
    (3, 64 * 2 + 9, 10, 64, 128),    # 32
    (3, 64 * 2, 7, 128, 192),        # not filled up: 24 chains of 12 slices find no CU each
    (2, 64, 5, 64, 256),             # 16 chains of 16 slices: the whole chip
])
def test_chains_that_are_not_a_multiple_of_the_xcds(B, T, H, K, V, bf16):
    x = make_stress_inputs(B, T, H, K, V, seed=165, bf16=bf16, retention=0.97)
    hp = ob.Hyper(eta=0.5, segments=1)
    compare_forward(x, hp, bf16)
    compare_backward(x, hp, bf16)


@pytest.mark.parametrize("B,T,H,K,V,channel_gate", [
    (2, 64 * 160, 8, 128, 128, False),
    (2, 64 * 160 + 5, 8, 128, 128, False),       # a ragged last chunk
    (1, 64 * 400 + 63, 8, 128, 64, False),       # more than 64 lines a slice
    (1, 64 * 600, 8, 64, 64, False),
    (1, 64 * 100, 8, 128, 512, False),           # 32 slices
    (3, 64 * 120, 4, 128, 256, False),           # filled up to 16 chains
    (2, 64 * 100 + 1, 8, 128, 128, True),
])
def test_a_long_call_that_asks_for_lines_ahead(B, T, H, K, V, channel_gate):
    """bf16, slices that share an XCD and more than the last level cache holds: the same bits as two calls of half the length, which do
    not ask for lines ahead."""
    g = torch.Generator(device="cuda").manual_seed(167)
    rnd = lambda *s: torch.randn(*s, device="cuda", generator=g)
    unit = lambda a: (a / a.norm(dim=-1, keepdim=True)).bfloat16()
    q, k, v, beta = unit(rnd(B, T, H, K)), unit(rnd(B, T, H, K)), rnd(B, T, H, V).bfloat16(), torch.sigmoid(rnd(B, T, H))
    la = -0.1 * torch.rand(B, T, H, K, device="cuda", generator=g) if channel_gate else -torch.nn.functional.softplus(rnd(B, T, H))
    hp = ob.Hyper(eta=0.05, segments=1, p1_pieces=-1)         # (pieces go by the length of the call)
    o, S, d, _ = ob.forward(q, k, v, beta, la, hp=hp)
    m = T // 128 * 64
    part = lambda a, b: [x[:, a:b].contiguous() for x in (q, k, v, beta, la)]
    o1, S1, d1, _ = ob.forward(*part(0, m), hp=hp)
    o2, S2, d2, _ = ob.forward(*part(m, T), None, d1, S1, hp=hp)
    same = [torch.equal(a, b) for a, b in ((d, d2), (S, S2), (o[:, :m], o1), (o[:, m:], o2))]
    assert all(same), same


def test_packed_sequences_with_channel_gates_that_ask_for_lines_ahead():
    """bf16, enough chains and tiles for both chain kernels to ask ahead, ragged documents longer than the eight chunks: the same bits as
    one call per document, which has too few of either."""
    lens, H, K, V = [64 * 180, 64 * 90 + 5, 64 * 100, 64 * 40 + 63], 8, 128, 64
    cu = [0, *np.cumsum(lens).tolist()]
    T = cu[-1]
    g = torch.Generator(device="cuda").manual_seed(169)
    rnd = lambda *s: torch.randn(*s, device="cuda", generator=g)
    unit = lambda a: (a / a.norm(dim=-1, keepdim=True)).bfloat16()
    x = [unit(rnd(1, T, H, K)), unit(rnd(1, T, H, K)), rnd(1, T, H, V).bfloat16(), torch.sigmoid(rnd(1, T, H)),
         -0.1 * torch.rand(1, T, H, K, device="cuda", generator=g)]
    dO = rnd(1, T, H, V).bfloat16()
    hp = ob.Hyper(eta=0.05, segments=1, p1_pieces=-1, p1_solved=-1)

    def run(lo, hi, cu_seqlens):
        part = [a[:, lo:hi].contiguous() for a in x]
        o, S, d, ctx = ob.forward(*part, hp=hp, for_backward=True, cu_seqlens=cu_seqlens)
        return dict(ob.backward(ctx, dO[:, lo:hi].contiguous()), o=o, S_out=S, d_out=d)

    whole = run(0, T, cu)
    for s, (lo, hi) in enumerate(zip(cu, cu[1:])):
        for name, a in run(lo, hi, None).items():
            if a is not None:
                ref = whole[name][s:s + 1] if name in ("S_out", "d_out", "dd_in", "dS_in") else whole[name][:, lo:hi]
                assert torch.equal(a, ref), (name, s)
