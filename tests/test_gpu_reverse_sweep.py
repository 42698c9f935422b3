"""The reverse sweep of phase 1 (precond_chain) in its two courses: a chunk whose sigma settles in two sweeps
goes on before its verdict is known, one that does not is fetched and done again (the last and the only chunk of a
launch among them), at every retention form, with clean and mixed masks in one workgroup, over segments; and
its sweeps over pieces of the sequence."""
import numpy as np
import pytest
import torch

from paper_2605_13473_amd import binding as ob
from paper_2605_13473_amd.inputs import make_stress_inputs
from tests.gpu_util import compare_backward, to_dev

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


# chunk by chunk (0: nothing couples, one sweep; 1: two; 2: three; 3: more): runs of either kind, single ones among others
COURSES = {"three_and_back": [1] * 3 + [2] + [1] * 10 + [2] * 3 + [1] * 2, "waited_for_and_back": [2, 3] + [1] * 19 + [3] + [2] * 9,
           "alternating": [1, 2, 0, 3] * 4}


@pytest.mark.parametrize("retention", ["none", "head", "channel"])
@pytest.mark.parametrize("course", COURSES)
def test_chunks_of_every_course_in_turn(course, retention):
    rng = np.random.Generator(np.random.Philox(11))
    kinds = COURSES[course]
    T = 64 * len(kinds)
    x = make_stress_inputs(1, T, 2, 64, 64, seed=173, bf16=False, retention=0.97)
    x["retention"] = {"none": None, "head": np.ones((1, T, 2), np.float32) * np.float32(0.9999),
                      "channel": rng.uniform(0.9998, 1.0, (1, T, 2, 64)).astype(np.float32)}[retention]
    # (the coupling goes with beta^2: eta = 1 alone would need more than three sweeps)
    x["beta"] = np.repeat(np.array([0.0, 0.01, 0.05, 0.9], np.float32)[kinds], 64)[None, :, None].repeat(2, axis=2)
    compare_backward(x, ob.Hyper(eta=1.0, p1_solved=-1, segments=1), False)


@pytest.mark.parametrize("K", [64, 128])
@pytest.mark.parametrize("retention", ["head", "channel"])
def test_chunks_that_the_box_holds_throughout(retention, K):
    """Retention 0.5: every coordinate lies on the lower face at every token, but in chunks whose gates are 1."""
    T = 64 * 9
    x = make_stress_inputs(1, T, 2, K, 64, seed=175, bf16=False, retention=0.97)
    r = np.full((1, T, 2) + ((K,) if retention == "channel" else ()), 0.5, np.float32)
    r[:, 128:192] = 1.0
    r[:, 384:448] = 1.0
    if retention == "channel":
        r[:, 256:320, :, K - 1] = 1.0            # (one coordinate is let go)
    x["retention"] = r
    x["d_in"] = np.full((1, 2, K), 0.5, np.float32)
    dd = np.random.Generator(np.random.Philox(12)).standard_normal((1, 2, K)).astype(np.float32)
    for segments in (1, 2):
        compare_backward(x, ob.Hyper(eta=0.3, p1_solved=-1, segments=segments), False, dd_out=dd)


def test_no_box_and_no_gradient():
    """No masks are written without a box; a zero adjoint (sigma = 0 throughout) settles at once."""
    x = make_stress_inputs(1, 192, 2, 128, 64, seed=181, bf16=True, retention=0.97)
    compare_backward(x, ob.Hyper(eta=0.3, d_min=1.0, d_max=0.0, p1_solved=-1, segments=1), True)
    x["dO"][:] = 0
    compare_backward(x, ob.Hyper(eta=0.3, p1_solved=-1, segments=1), True)


@pytest.mark.parametrize("retention", ["none", "head", "channel"])
@pytest.mark.parametrize("pieces", [2, 7, 24])
def test_pieces_of_uneven_length(pieces, retention):
    """The last piece shorter than the others, pieces of one chunk, a ragged end, an adjoint from outside."""
    rng = np.random.Generator(np.random.Philox(9))
    T = 64 * 23 + 5
    x = make_stress_inputs(1, T, 2, 64, 64, seed=191, bf16=False, retention=0.97)
    if retention == "none":
        x["retention"] = None
    elif retention == "channel":
        x["retention"] = rng.uniform(0.9, 1.0, (1, T, 2, 64)).astype(np.float32)
    dd = rng.standard_normal((1, 2, 64)).astype(np.float32)
    compare_backward(x, ob.Hyper(eta=0.3, p1_pieces=pieces, p1_solved=-1), False, dd_out=dd)


@pytest.mark.parametrize("retention", ["head", "channel"])
def test_pieces_settle_where_the_gates_hardly_fade(retention):
    """Gates of 1, large beta, K = 64: the coupling of the coordinates is what moves from piece to piece.  Chains that settle within six
    sweeps have the same bits with any higher limit (those that do not are done by the sequential sweep, with others)."""
    T = 64 * 64
    x = make_stress_inputs(1, T, 4, 64, 64, seed=195, bf16=True, retention=0.97)
    x["retention"] = np.ones((1, T, 4) + ((64,) if retention == "channel" else ()), np.float32)
    x["beta"] = (0.9 + 0.1 * np.random.Generator(np.random.Philox(14)).random((1, T, 4))).astype(np.float32)
    t, got = to_dev(x, True), []
    for pieces, limit in ((-1, 0), (16, 6), (16, 13)):
        *_, ctx = ob.forward(*[t[n] for n in ("q", "k", "v", "beta", "log_alpha", "retention", "d_in", "S_in")],
                             ob.Hyper(p1_pieces=-1), for_backward=True)
        ctx["params"].p1_pieces, ctx["params"].p1_piece_sweeps = pieces, limit
        got.append(ob.backward(ctx, t["dO"]))
    torch.cuda.synchronize()
    seq, six, many = got
    assert all(torch.equal(six[n], many[n]) for n in six)
    assert not torch.equal(six["dd_in"], seq["dd_in"])
    for n in ("dretention", "dd_in", "dbeta"):
        assert (six[n] - seq[n]).abs().max() <= 1e-5 * seq[n].abs().max(), n


def test_values_that_are_not_finite_reach_what_they_reached_without_pieces():
    """A gradient that is not finite never settles: the sequential sweep has the last word."""
    x = to_dev(make_stress_inputs(1, 64 * 12, 2, 64, 64, seed=193, bf16=False, retention=0.97), False)
    x["dO"][0, 500, 1, 3] = float("inf")
    got = []
    for pieces in (-1, 4):
        o, S, d, ctx = ob.forward(*[x[n] for n in ("q", "k", "v", "beta", "log_alpha", "retention", "d_in", "S_in")],
                                  ob.Hyper(eta=0.3, p1_pieces=pieces), for_backward=True)
        got.append(ob.backward(ctx, x["dO"]))
    torch.cuda.synchronize()
    assert not torch.isfinite(got[0]["dd_in"][0, 1]).all() and torch.isfinite(got[0]["dd_in"][0, 0]).all()
    for n, a in got[0].items():
        assert torch.equal(torch.isfinite(a), torch.isfinite(got[1][n])), n


def test_a_sigma_that_is_not_a_number_has_no_say_in_the_verdict():
    """Retention inf at one token: the box takes d to its upper face there, as any large retention would, and what lies left of it
    gets gradients that are not numbers.  The seven tokens right of it have the ones they have with 1e6, to ten times the sweeps'
    tolerance (the large eta makes two sweeps far too few for them: 1e-4 off; the chunk behind settles in two)."""
    x = to_dev(make_stress_inputs(1, 128, 1, 64, 64, seed=199, bf16=False, retention=0.97), False)
    x["beta"][0, 64:] = 1e-4
    got = []
    for big in (1e6, float("inf")):
        x["retention"][0, 56, 0] = big
        o, S, d, ctx = ob.forward(*[x[n] for n in ("q", "k", "v", "beta", "log_alpha", "retention", "d_in", "S_in")],
                                  ob.Hyper(eta=64.0, p1_solved=-1, segments=1), for_backward=True)
        got.append((o, ob.backward(ctx, x["dO"])))
    torch.cuda.synchronize()
    assert torch.equal(got[0][0], got[1][0])
    assert not torch.isfinite(got[1][1]["dbeta"][0, :56]).all()
    for n in ("dk", "dbeta"):
        a, b = (g[n][0, 57:64] for _, g in got)
        assert (a - b).abs().max() <= 1e-6 * a.abs().max(), n


def test_segments_in_a_captured_graph():
    """Short sequences take one stream by themselves; the side stream's part of a capture, forced here, and
    replays between eager calls."""
    t = to_dev(make_stress_inputs(2, 64 * 6, 2, 64, 64, seed=197, bf16=True, retention=0.97), True)
    p = ob.make_params(2, 384, 2, 64, 64, True, ob.Hyper(eta=0.3, segments=3))
    ws = ob.alloc_workspace(p, True)
    names = ("q", "k", "v", "beta", "log_alpha", "retention", "d_in", "S_in")
    fwd = [torch.empty_like(t["v"]), torch.empty_like(t["S_in"]), torch.empty_like(t["d_in"])]
    grads = [torch.empty_like(t[n]) for n in names]

    def step():
        ob.osdn_fwd(p, *[t[n] for n in names], *fwd, ws)
        ob.osdn_bwd(p, *[t[n] for n in names], t["dO"], None, None, *grads, ws)

    step()
    torch.cuda.synchronize()
    ref = [a.clone() for a in fwd + grads]
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        step()
    for _ in range(3):
        for a in fwd + grads:
            a.fill_(float("nan"))
        g.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(a, r) for a, r in zip(fwd + grads, ref))
        step()
        torch.cuda.synchronize()
        assert all(torch.equal(a, r) for a, r in zip(fwd + grads, ref))


@pytest.mark.parametrize("eta", [0.003, 0.05])
@pytest.mark.parametrize("T", [64 * 6, 64 * 4 + 7])
@pytest.mark.parametrize("K", [64, 128])
def test_masks_of_chunks_off_the_box_and_close_to_it(K, T, eta):
    """Without retention the forward sweep marks the chunks that stay off the box and the backward pass does not replay them: heads
    whose coordinates are far from the faces, start on one, within the margin of the mark and just outside it, or come to
    one along the sequence; every decision is checked one by one.  A second backward pass on the same context gives the same."""
    H = 6
    x = make_stress_inputs(1, T, H, K, 64, seed=177, bf16=False)
    x["retention"] = None
    d = np.full((1, H, K), 1.0, np.float32)
    d[0, 1, 3] = 2.0
    d[0, 2, 5] = np.float32(2.0) * np.float32(1 - 1e-5)
    d[0, 3, 7] = np.float32(2.0) * np.float32(1 - 4e-5)
    d[0, 4, 0], d[0, 4, 1] = 0.5, np.float32(0.5) * np.float32(1 + 1e-5)
    d[0, 5, ::2] = 1.98
    x["d_in"] = d
    hp = ob.Hyper(eta=eta, p1_solved=-1, segments=1)
    compare_backward(x, hp, False)
    t = to_dev(x, False)
    _, _, _, ctx = ob.forward(t["q"], t["k"], t["v"], t["beta"], t["log_alpha"], None, t["d_in"], t["S_in"], hp, for_backward=True)
    a, b = ob.backward(ctx, t["dO"]), ob.backward(ctx, t["dO"])
    torch.cuda.synchronize()
    assert all(torch.equal(a[n], b[n]) for n in a if a[n] is not None)
