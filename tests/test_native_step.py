"""binding.step's way through the extension module against its way through Python: the same bits for what the
module takes, and everything else left to the Python code with the errors it gives."""
import dataclasses

import pytest
import torch

from paper_2605_13473_amd import binding as ob


def _inputs(dev, bf16=True, B=2, T=1, H=3, K=64, V=128, gate="head", retention="head", carried=True):
    g = torch.Generator(device=dev).manual_seed(5)
    rnd = lambda *s: torch.randn(*s, device=dev, generator=g)
    dt = torch.bfloat16 if bf16 else torch.float32
    shape = {None: None, "head": (B, T, H), "channel": (B, T, H, K)}
    sg, sr = shape[gate], shape[retention]
    return dict(q=rnd(B, T, H, K).to(dt), k=(rnd(B, T, H, K) / 8).to(dt), v=rnd(B, T, H, V).to(dt), beta=torch.sigmoid(rnd(B, T, H)),
                log_alpha=None if sg is None else -torch.nn.functional.softplus(rnd(*sg)),
                retention=None if sr is None else torch.sigmoid(4.0 + rnd(*sr)),
                d_in=(1.0 + 0.1 * rnd(B, H, K)).clamp(0.5, 2.0) if carried else None, S_in=rnd(B, H, V, K) if carried else None)


def test_the_module_is_built_and_leaves_tensors_of_the_host_alone():
    ob.lib()
    assert ob._step_native is not None
    x = _inputs("cpu")
    assert ob._step_native(*x.values(), ob.Hyper(), False, 0, 0) is None
    with pytest.raises(TypeError):
        ob.step(*x.values())


@pytest.mark.gpu
@pytest.mark.parametrize("hp", [ob.Hyper(), ob.Hyper(scale=0.3, eta=0.5, d_min=0.9, beta_aware=False)])
@pytest.mark.parametrize("case", [dict(), dict(bf16=False, K=128), dict(T=5, gate="channel", retention="channel"),
                                  dict(gate=None, retention=None, carried=False)])
def test_same_bits_as_the_python_way(case, hp, monkeypatch):
    x = _inputs("cuda", **case)
    clone = lambda: {n: None if a is None else a.clone() for n, a in x.items()}
    for in_place in (False, True):
        a, b = clone(), clone()
        dev = torch.cuda.current_device()
        native = ob._step_native if ob._lib is not None else (ob.lib(), ob._step_native)[1]
        r = native(*a.values(), hp, in_place, dev, torch.cuda.current_stream().cuda_stream)
        assert type(r) is tuple and (not in_place or a["S_in"] is None or r[1] is a["S_in"])
        with monkeypatch.context() as m:
            m.setattr(ob, "_step_native", None)
            w = ob.step(*b.values(), hp, in_place)
        for y, z in zip(r, w):
            assert y.dtype == z.dtype and y.device == z.device and y.stride() == z.stride() and torch.equal(y, z)


@pytest.mark.gpu
def test_what_is_out_of_the_ordinary_goes_through_python():
    x = _inputs("cuda")
    ob.lib()
    dev, st = torch.cuda.current_device(), torch.cuda.current_stream().cuda_stream
    call = lambda hp=ob.Hyper(), in_place=False, **kw: ob._step_native(*dict(x, **kw).values(), hp, in_place, dev, st)
    step = lambda hp=ob.Hyper(), **kw: ob.step(*dict(x, **kw).values(), hp)

    call_outside = call()[0]

    class Sub(torch.Tensor):
        pass

    bad = [(dict(v=x["v"].float()), TypeError), (dict(beta=x["beta"][:, :, :2]), ValueError), (dict(q=x["q"].transpose(2, 3)), ValueError),
           (dict(d_in=x["d_in"].double()), TypeError), (dict(S_in=x["S_in"].cpu()), TypeError), (dict(log_alpha=x["log_alpha"][0]), ValueError)]
    for kw, error in bad:
        assert call(**kw) is None
        with pytest.raises(error):
            step(**kw)
    assert call(q=x["q"].as_subclass(Sub)) is None
    with torch.device("cuda"):                                                      # (a torch function mode)
        assert call() is None and torch.equal(step()[0], call_outside)
    assert call(dataclasses.replace(ob.Hyper(), eta=1)) is None                     # (an int: taken as Python takes it)
    assert torch.equal(step(dataclasses.replace(ob.Hyper(), eta=1))[0], step(dataclasses.replace(ob.Hyper(), eta=1.0))[0])
    assert type(call(ob.Hyper(eps=-1.0))) is int                                    # (a status: nothing was launched)
    with pytest.raises(ob.OsdnError):
        step(ob.Hyper(eps=-1.0))
