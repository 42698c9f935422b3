"""GPU parity of the recurrent step (decode) entry point against the CPU oracle, and its
agreement with the chunkwise path (Appendix K: chunk vs. single-token kernel, prefill + one
decode token vs. one chunkwise call on the concatenation)."""
import numpy as np
import pytest
import torch

import oracle
from paper_2605_13473_amd import binding as ob
from paper_2605_13473_amd.inputs import make_stress_inputs
from tests.gpu_util import check, f64, oracle_hp, to_dev

pytestmark = pytest.mark.gpu


def _oracle_fwd(x, hp):
    y = f64(x)
    return oracle.fwd(y["q"], y["k"], y["v"], y["beta"], y.get("log_alpha"), y.get("retention"),
                      y.get("d_in"), y.get("S_in"), oracle_hp(hp))


def _slice_t(x, t0, t1):
    return {n: (a[:, t0:t1] if (a is not None and n in ("q", "k", "v", "dO", "beta", "log_alpha", "retention"))
                else a) for n, a in x.items()}


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("shape", [(1, 1, 1, 64, 64), (2, 5, 3, 64, 128), (1, 64, 2, 128, 192), (3, 17, 1, 128, 64)])
def test_step_against_oracle(shape, bf16):
    """1..64 tokens in one launch, stress inputs (large eta, both faces of the box, carried state)."""
    B, T, H, K, V = shape
    x = make_stress_inputs(B, T, H, K, V, seed=31, bf16=bf16, retention=0.97)
    hp = ob.Hyper(eta=0.5)
    t = to_dev(x, bf16)
    o, S, d = ob.step(t["q"], t["k"], t["v"], t["beta"], t["log_alpha"], t["retention"], t["d_in"], t["S_in"], hp)
    torch.cuda.synchronize()
    oo, oS, od = _oracle_fwd(x, hp)
    check("o", o, oo, bf16)
    check("S_out", S, oS, bf16)
    check("d_out", d, od, False)


def test_token_by_token_equals_one_call_and_updates_in_place():
    """Sixteen launches of one token each, state carried in place, against one launch of 16."""
    B, T, H, K, V = 2, 16, 2, 128, 64
    x = make_stress_inputs(B, T, H, K, V, seed=32, bf16=False, retention=0.95)
    hp = ob.Hyper(eta=0.3)
    t = to_dev(x, False)
    o_all, S_all, d_all = ob.step(t["q"], t["k"], t["v"], t["beta"], t["log_alpha"], t["retention"],
                                  t["d_in"], t["S_in"], hp)
    S = t["S_in"].clone()
    d = t["d_in"].clone()
    outs = []
    for i in range(T):
        sl = slice(i, i + 1)
        o, S2, d = ob.step(t["q"][:, sl].contiguous(), t["k"][:, sl].contiguous(), t["v"][:, sl].contiguous(),
                           t["beta"][:, sl].contiguous(), t["log_alpha"][:, sl].contiguous(),
                           t["retention"][:, sl].contiguous(), d, S, hp, in_place=True)
        assert S2.data_ptr() == S.data_ptr()
        outs.append(o)
    torch.cuda.synchronize()
    assert torch.equal(torch.cat(outs, 1), o_all)            # the same arithmetic in the same order
    assert torch.equal(S, S_all) and torch.equal(d, d_all)


@pytest.mark.parametrize("bf16", [False, True])
def test_prefill_then_one_decode_token(bf16):
    """Chunkwise prefill of 128 tokens + one recurrent step against the oracle on 129 tokens."""
    B, T, H, K, V = 2, 129, 2, 128, 128
    x = make_stress_inputs(B, T, H, K, V, seed=33, bf16=bf16, retention=0.98)
    hp = ob.Hyper(eta=0.2)
    t = to_dev(x, bf16)
    pre = {n: (a[:, :128].contiguous() if (a is not None and a.dim() >= 3 and a.shape[1] == T) else a) for n, a in t.items()}
    last = {n: (a[:, 128:].contiguous() if (a is not None and a.dim() >= 3 and a.shape[1] == T) else a) for n, a in t.items()}
    o1, S1, d1, _ = ob.forward(pre["q"], pre["k"], pre["v"], pre["beta"], pre["log_alpha"], pre["retention"],
                               pre["d_in"], pre["S_in"], hp)
    o2, S2, d2 = ob.step(last["q"], last["k"], last["v"], last["beta"], last["log_alpha"], last["retention"],
                         d1, S1, hp)
    torch.cuda.synchronize()
    oo, oS, od = _oracle_fwd(x, hp)
    check("o[:128]", o1, oo[:, :128], bf16)
    check("o[128]", o2, oo[:, 128:], bf16)
    check("S_out", S2, oS, bf16)
    check("d_out", d2, od, False)


def test_chunk_equals_step_on_one_chunk():
    """One chunk through the chunkwise kernels and through the recurrent kernel: fp32, so the two
    evaluation orders agree to fp32 reassociation."""
    B, T, H, K, V = 1, 64, 2, 64, 64
    x = make_stress_inputs(B, T, H, K, V, seed=34, bf16=False, retention=0.97)
    hp = ob.Hyper(eta=0.5)
    t = to_dev(x, False)
    args = (t["q"], t["k"], t["v"], t["beta"], t["log_alpha"], t["retention"], t["d_in"], t["S_in"], hp)
    o1, S1, d1, _ = ob.forward(*args)
    o2, S2, d2 = ob.step(*args)
    torch.cuda.synchronize()
    for name, a, b in (("o", o1, o2), ("S", S1, S2), ("d", d1, d2)):
        err = (a - b).abs().max().item()
        assert err <= 1e-4 * max(b.abs().max().item(), 1e-30), (name, err)


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("shape", [(2, 1, 2, 64, 64), (1, 33, 3, 128, 128), (2, 64, 1, 128, 64)])
def test_step_with_a_gate_per_key_channel(shape, bf16):
    """The online-scaled KDA recurrence: S <- S Diag(alpha_t) with one gate per key channel (and,
    on the last shape, one retention per coordinate as well), against the oracle; launches of
    one token each, state carried in place, agree with one launch bit for bit."""
    B, T, H, K, V = shape
    x = make_stress_inputs(B, T, H, K, V, seed=35, bf16=bf16, retention=0.97)
    rng = np.random.default_rng(36)
    x["log_alpha"] = (-np.logaddexp(0.0, rng.standard_normal((B, T, H, K)) - 1.0)).astype(np.float32)
    if V == 64:
        x["retention"] = np.clip(x["retention"][..., None] + 0.03 * rng.standard_normal((B, T, H, K)), 0, 1).astype(np.float32)
    hp = ob.Hyper(eta=0.5)
    t = to_dev(x, bf16)
    o, S, d = ob.step(t["q"], t["k"], t["v"], t["beta"], t["log_alpha"], t["retention"], t["d_in"], t["S_in"], hp)
    torch.cuda.synchronize()
    oo, oS, od = _oracle_fwd(x, hp)
    check("o", o, oo, bf16)
    check("S_out", S, oS, bf16)
    check("d_out", d, od, False)
    S2, d2, outs = t["S_in"].clone(), t["d_in"], []
    for i in range(T):
        c = lambda a: a[:, i:i + 1].contiguous()
        oi, S2, d2 = ob.step(c(t["q"]), c(t["k"]), c(t["v"]), c(t["beta"]), c(t["log_alpha"]), c(t["retention"]),
                             d2, S2, hp, in_place=True)
        outs.append(oi)
    torch.cuda.synchronize()
    assert torch.equal(torch.cat(outs, 1), o) and torch.equal(S2, S) and torch.equal(d2, d)


def test_step_argument_errors():
    p = ob.make_params(1, 65, 1, 64, 64, False)
    z = torch.zeros(1, 65, 1, 64, device="cuda")
    with pytest.raises(ob.OsdnError):        # more than 64 tokens: chunkwise path
        ob.osdn_step(p, z, z, z, z[..., 0].contiguous(), None, None, None, None, z.clone(),
                     torch.zeros(1, 1, 64, 64, device="cuda"), torch.zeros(1, 1, 64, device="cuda"))
    p = ob.make_params(1, 1, 1, 64, 64, False)
    z = torch.zeros(1, 1, 1, 64, device="cuda")
    d = torch.ones(1, 1, 64, device="cuda")
    with pytest.raises(ob.OsdnError):        # d_out must not be d_in
        ob.osdn_step(p, z, z, z, z[..., 0].contiguous(), None, None, d, None, z.clone(),
                     torch.zeros(1, 1, 64, 64, device="cuda"), d)


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("retention,gate", [("head", "head"), ("channel", "channel"), (None, None)])
@pytest.mark.parametrize("B,T,H,K,V", [
    (1, 4, 1, 128, 64),      # 16 rows per workgroup, one block of tokens
    (1, 5, 3, 64, 128),      # ... one token left over
    (2, 63, 1, 128, 64),
    (1, 2, 17, 64, 512),     # 32 rows per workgroup (more than 512 slices of 16 rows), less than a block
    (1, 7, 17, 128, 512),
])
def test_tokens_of_one_call_equal_single_calls(B, T, H, K, V, retention, gate, bf16):
    """A call of several tokens gives, bit for bit, what that many calls of one token give: every sum
    of the several-token kernel is formed in the order of the one-token kernel, which the oracle pins."""
    g = torch.Generator(device="cuda").manual_seed(B * 1000 + T)
    rnd = lambda *s: torch.randn(*s, device="cuda", generator=g)
    dt = torch.bfloat16 if bf16 else torch.float32
    shape = {None: None, "head": (B, T, H), "channel": (B, T, H, K)}
    sh, sr = shape[gate], shape[retention]
    x = dict(q=rnd(B, T, H, K).to(dt), k=(rnd(B, T, H, K) / K ** 0.5).to(dt), v=rnd(B, T, H, V).to(dt),
             beta=torch.sigmoid(rnd(B, T, H)),
             log_alpha=None if sh is None else -torch.nn.functional.softplus(rnd(*sh)),
             retention=None if sr is None else torch.sigmoid(4.0 + rnd(*sr)))
    d0, S0 = (1.0 + 0.1 * rnd(B, H, K)).clamp(0.5, 2.0), 0.1 * rnd(B, H, V, K)
    hp = ob.Hyper(eta=0.5)
    o_all, S_all, d_all = ob.step(*x.values(), d0, S0, hp)
    S, d, outs = S0, d0, []
    for i in range(T):
        o, S, d = ob.step(*(None if a is None else a[:, i:i + 1].contiguous() for a in x.values()), d, S, hp)
        outs.append(o)
    assert torch.equal(torch.cat(outs, 1), o_all)
    assert torch.equal(S, S_all) and torch.equal(d, d_all)
