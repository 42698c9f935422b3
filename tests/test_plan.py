"""The rules that cut the work (csrc/osdn_plan.h), compiled for the CPU and asked over sizes: every plan covers the sequence and stays
inside the buffers that are laid out for it, and the calls that measurements put on one course take it."""
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2605_13473_amd", "csrc")
MAIN = r"""
#include "osdn_plan.h"
#include <cstdio>
#include <vector>
using namespace osdn;
// in: chains chunks K V bf16 retention(0, 1, 2) eta forced_pieces backward; out: pieces, chunks of one, sweeps, solved, segments, begins
// or, with an argument, in: slices chains narrow V bf16 K; out: workgroups, 1 if every slice of every chain is one of them once, 1 if the slices of
// a chain share an XCD, slices of 16 in the backward pass beside a phase-1 chain and without one, lines asked
// for ahead in a long call
int slices() {
    int ns, narrow, V, bf, K; long long ch;
    while (std::scanf("%d %lld %d %d %d %d", &ns, &ch, &narrow, &V, &bf, &K) == 6) {
        osdn_params p{};
        p.K = K; p.V = V; p.io_dtype = bf ? OSDN_BF16 : OSDN_F32;
        const SliceMap m = slice_map(ns, ch, narrow);
        const int wgs = chain_workgroups(m);
        std::vector<int> seen(ch * ns, 0), xcd(ch, -1);
        bool share = true;
        for (int w = 0; w < wgs; ++w) {
            int c = -1, s = -1;
            chain_slice_of(w, m, c, s);
            if (c >= ch) continue;
            ++seen.at(c * ns + s);
            if (xcd[c] >= 0 && xcd[c] != w % NUM_XCD) share = false;
            xcd[c] = w % NUM_XCD;
        }
        bool once = true;
        for (int x : seen) once = once && x == 1;
        std::printf("%d %d %d %d %d %d\n", wgs, once, share, narrow_backward(&p, ch, true), narrow_backward(&p, ch, false), asks_ahead(&p, 1 << 20, ch));
    }
    return 0;
}
int main(int argc, char **) {
    if (argc > 1) return slices();
    long long ch; int N, K, V, bf, ret, forced, back; float eta;
    while (std::scanf("%lld %d %d %d %d %d %f %d %d", &ch, &N, &K, &V, &bf, &ret, &eta, &forced, &back) == 9) {
        osdn_params p{};
        p.K = K; p.V = V; p.io_dtype = bf ? OSDN_BF16 : OSDN_F32; p.eta = eta; p.retention_per_channel = ret == 2; p.p1_pieces = forced;
        int pieces, len, sweeps;
        const bool solved = back && solved_plan(&p, ch, N, ret != 0);
        pieces_plan(&p, N, ch, false, ret != 0, back != 0, pieces, len, sweeps);
        if (solved) pieces = 0;
        const int S = pieces ? 1 : segment_count(0, N, N, ch, ch * (V / 32) + ch, back != 0, 512);
        std::printf("%d %d %d %d %d", pieces, len, sweeps, (int)solved, S);
        for (int s = 0; s <= S; ++s) std::printf(" %d", back || ch * (V / 32) + ch <= NUM_CU ? seg_begin(N, S, s) : seg_begin_grow(N, S, s, 1.7));
        std::printf("\n");
    }
}
"""


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    d = tmp_path_factory.mktemp("plan")
    (d / "main.cpp").write_text(MAIN)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-I", CSRC, "-o", str(d / "plan"), str(d / "main.cpp")])

    def ask(calls, *which):
        """calls: (chains, chunks, K, V, bf16, retention, eta, forced, backward) each."""
        text = "\n".join(" ".join(str(x) for x in c) for c in calls) + "\n"
        r = subprocess.run([str(d / "plan"), *which], input=text, capture_output=True, text=True, check=True)
        return [[int(x) for x in line.split()] for line in r.stdout.splitlines()]
    return ask


def test_every_plan_covers_the_sequence(plan):
    calls = [(ch, N, K, V, bf, ret, eta, forced, back)
             for ch in (1, 2, 3, 5, 8, 16, 17, 32, 33, 64, 100, 255, 256, 300, 1000)
             for N in (1, 2, 23, 24, 25, 31, 47, 63, 64, 65, 127, 200, 448, 513, 1024, 4001)
             for K, V in ((64, 64), (128, 512)) for bf in (0, 1) for ret in (0, 1, 2) for eta in (0.003, 1.0)
             for forced in (-1, 0, 1, 7, 600) for back in (0, 1)]
    for c, (P, length, sweeps, solved, S, *cuts) in zip(calls, plan(calls)):
        ch, N = c[:2]
        assert 1 <= sweeps <= 13
        if P:
            assert P >= 2 and (P - 1) * length < N <= P * length and P * ch <= 512 and ch <= 256, c
        assert 1 <= S <= min(N, 16) and cuts[0] == 0 and cuts[-1] == N and all(a < b for a, b in zip(cuts, cuts[1:])), c
        if c[7] == -1:
            assert not P, c


@pytest.mark.parametrize("ret", [0, 1])
@pytest.mark.parametrize("chains,chunks,pieces", [(1, 1024, 128), (2, 1024, 128), (4, 512, 64), (2, 296, 37), (4, 300, 38), (4, 64, 16),
                                                  (8, 128, 32), (4, 256, 32)])
def test_long_sequences_of_few_chains_are_cut_into_pieces_of_eight(plan, chains, chunks, pieces, ret):
    assert plan([(chains, chunks, 128, 128, 1, ret, 0.003, 0, 0)])[0][0] == pieces


@pytest.mark.parametrize("back", [0, 1])
def test_no_pieces_beyond_an_eighth_of_the_cus(plan, back):
    """With a retention gate pieces win there only if it fades much, which the rule does not know."""
    calls = [(ch, N, K, 128, bf, ret, 0.003, 0, back) for ch in (33, 48, 64) for N in (24, 32, 64, 128, 256) for K in (64, 128)
             for bf in (0, 1) for ret in (0, 1, 2)]
    assert not any(r[0] for r in plan(calls))
    assert all(r[0] for r in plan([(32, N, 128, 128, 1, 1, 0.003, 0, back) for N in (24, 32, 64)]))


@pytest.mark.parametrize("K,bf16,ret,back,pieces", [(128, 1, 0, 0, 32), (128, 0, 0, 0, 32), (128, 1, 1, 0, 32), (128, 0, 1, 0, 16), (128, 1, 2, 0, 16),
                                                    (128, 0, 2, 0, 16), (128, 1, 1, 1, 16), (128, 1, 2, 1, 16), (64, 1, 1, 1, 32), (64, 0, 2, 0, 32)])
def test_two_workgroups_a_cu_only_where_the_kernel_fits_twice(plan, K, bf16, ret, back, pieces):
    assert plan([(16, 256, K, 128, bf16, ret, 0.003, 0, back)])[0][0] == pieces


def test_pieces_by_eta(plan):
    """A large eta, where the sweeps over pieces need many rounds or never settle: backward none, forward pieces of eight chunks."""
    for K, fwd_most, bwd_most in ((64, 0.0032, 0.016), (128, 0.0064, 0.032)):
        ask = lambda N, eta, back: plan([(16, N, K, 128, 1, 1, eta, 0, back)])[0][:2]
        for eta in (1e-4, 0.003, 0.99 * fwd_most):
            assert ask(24, eta, 0)[0] and ask(128, eta, 0)[0] == 16 and ask(64, eta, 0) == [16, 4]
        for eta in (1.01 * fwd_most, 0.1, 1.0):
            assert not ask(24, eta, 0)[0] and not ask(63, eta, 0)[0] and ask(64, eta, 0) == [8, 8] and ask(256, eta, 0) == [16, 16]
        assert ask(24, 0.99 * bwd_most, 1)[0] and ask(128, 0.99 * bwd_most, 1)[0]
        assert not any(ask(N, 1.01 * bwd_most, 1)[0] for N in (24, 64, 256))


@pytest.mark.parametrize("chains,K,bf16,most", [(16, 128, 1, 4096), (17, 128, 1, 64), (32, 64, 1, 64), (32, 128, 0, 64), (16, 128, 0, 96), (9, 128, 0, 96),
                                                (8, 128, 0, 4096), (16, 64, 0, 4096)])
def test_no_pieces_in_reverse_for_long_sequences_of_many_chains(plan, chains, K, bf16, most):
    got = {N: plan([(chains, N, K, 128, bf16, 1, 0.003, 0, 1)])[0][0] for N in (24, 64, 65, 96, 97, 256, 4096)}
    assert all((P > 0) == (N <= most) for N, P in got.items()), got


@pytest.mark.parametrize("chains,K,V,bf16,ret", [(33, 128, 128, 1, 1), (48, 128, 128, 1, 2), (16, 128, 128, 1, 0), (9, 128, 128, 0, 1)])
def test_segments_of_long_sequences_in_reverse(plan, chains, K, V, bf16, ret):
    """Seven from 448 chunks on, in the solved form and with sweeps."""
    for N in (448, 512, 2000):
        assert plan([(chains, N, K, V, bf16, ret, 0.003, 0, 1)])[0][4] == 7


@pytest.mark.parametrize("chains,K,V,bf16,least", [(32, 128, 128, 1, 1), (33, 128, 128, 1, 16), (48, 128, 128, 1, 16), (49, 128, 128, 1, None),
                                                   (64, 128, 64, 1, 16), (64, 64, 128, 1, 16), (65, 64, 64, 1, None), (32, 64, 64, 0, 1), (33, 64, 64, 0, None)])
def test_solved_form_without_retention(plan, chains, K, V, bf16, least):
    for N in (1, 8, 15, 16, 64, 1000):
        assert plan([(chains, N, K, V, bf16, 0, 0.003, 0, 1)])[0][3] == (least is not None and N >= least), N
    assert not any(r[3] for r in plan([(chains, 64, K, V, bf16, ret, 0.003, 0, 1) for ret in (1, 2)]))


def test_slices_of_the_chain_kernels(plan):
    calls = [(V // (16 if narrow else 32), ch, narrow, V, bf, K)
             for V in range(64, 513, 64) for ch in (*range(1, 70), 127, 128, 256, 1000, 65537) for narrow in (0, 1) for bf in (0, 1) for K in (64, 128)]
    for (ns, ch, narrow, V, bf, K), (wgs, once, share, beside, alone, ahead) in zip(calls, plan(calls, "slices")):
        assert once, (ns, ch)
        filled = narrow and ch > 8 and -(-ch // 8) * 8 * ns <= 256
        assert wgs == (-(-ch // 8) * 8 if filled else ch) * ns
        assert share or not (filled or ch % 8 == 0)
        assert not narrow or ahead == (share and (filled or ch % 8 == 0))
        if bf:
            # never on more XCDs than slices of 32, but with up to eight chains
            assert not beside and alone == (ch * (V // 16) <= 256 and (ch <= 8 or ch % 8 == 0 or V >= 256 or -(-ch // 8) * (V // 16) <= 32))
        else:
            assert beside == alone == (K == 128 or ch * (V // 16) <= 256)
