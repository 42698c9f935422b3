// The rules by which osdn_fwd and osdn_bwd cut the work: segments of the sequence, pieces of a chain, the solved form of the
// reverse sweep, and the slices of the chain kernels.  Plain code without a device in it, so that the rules can be tested by themselves.
#pragma once
#include "../../include/osdn.h"

#include <cmath>

namespace osdn {

constexpr int NUM_CU = 256, NUM_XCD = 8;         // (workgroups are dealt to the XCDs in turn; each has its own L2)
constexpr int MAX_SEGMENTS = 16, MAX_PIECES = 512, MAX_PIECE_SWEEPS = 13;

// The chain kernels run V/VS workgroups (slices) per chain that all read the same tiles (-W, K~, P, ...): they are to share an XCD.
// Where the chains are not a multiple of the XCDs, narrow slices (VS = 16) are filled up to one with workgroups that end at once, if all still
// find a CU each; else the slices of a chain stand side by side on as many XCDs.  20 chains of 40 chunks, V = 128, us, side by
// side and filled up: forward 161 and 136, backward 222 and 189 (with slices of 32 203); of 128 chunks, forward 446 and 399; 28 chains of
// 128 chunks, forward 605 and 491; 12 of 64, V = 256, 181 and 163; fp32, 10 of 32, backward 336 and 328.  Not up to eight chains, which leave the L2s
// time (2 chains of 512 chunks, V = 256, forward 598 and 608, 6 of 64 with K = 64 118 and 122, 4 of 512 599 and 555), nor for slices of 32
// (50 chains of 64 chunks, forward 360 and 366, backward 521 and 527).
inline bool chains_filled_up(int nslices, long long chains, bool narrow) {
    return narrow && chains > NUM_XCD && (chains + NUM_XCD - 1) / NUM_XCD * nslices * NUM_XCD <= NUM_CU;
}
// How the workgroups of such a launch are laid out, with what a workgroup needs to find its slice: a multiplication in place of a division
// (reciprocal: the next above 2^32 / slices, exact below 2^27 workgroups), and nothing that it would have to wait for twice.
struct SliceMap { int slices, chains, share; unsigned reciprocal; };
inline SliceMap slice_map(int nslices, long long chains, bool narrow) {
    return {nslices, (int)chains, chains % NUM_XCD == 0 || chains_filled_up(nslices, chains, narrow), (unsigned)(((1ull << 32) + nslices - 1) / nslices)};
}
inline int chain_workgroups(const SliceMap &m) { return (m.share ? (m.chains + NUM_XCD - 1) / NUM_XCD * NUM_XCD : m.chains) * m.slices; }
// (constexpr: for the device too; a chain that there is not: nothing to do)
constexpr void chain_slice_of(int wg, const SliceMap &m, int &chain, int &slice) {
    const unsigned j = m.share ? (unsigned)wg / NUM_XCD : (unsigned)wg, c = (unsigned)(((unsigned long long)j * m.reciprocal) >> 32);
    slice = (int)(j - c * m.slices);
    chain = m.share ? (int)(wg % NUM_XCD + NUM_XCD * c) : (int)c;
}

// state_fwd_run_kernel with slices of 16: whether it asks for the lines of its operands ahead of its tiles (tiles: chunks of all chains).
// That pays where they come from HBM and the slices that share them share an L2: what the forward pass reads and writes around the chain
// kernel (-W, K~, T diag(beta), V, the checkpoint of S, E; three more with a gate per channel) is then more than the 256 MB
// of the last level cache hold beside the inputs.  Forward pass, us, without and with, K = V = 128 unless said, calls repeated: 16 chains of 64
// chunks (106 MB) 172.9 and 174.5, of 96 (160) 244.4 and 247.8, of 128 (213) 343 and 338, of 256 with retention 542 and 509; 24 of 48 (120)
// 178.7 and 180.6, of 128 (319) 456 and 451; V = 256: 16 of 64 (172) 180.8 and 182.7, of 128 (344) 331 and 324, 8 of 128 (172) 219.8 and 231.3, of
// 256 430 and 415; V = 64: 32 of 64 (147) 264.5 and 265.8, of 128 (295) 478 and 456, 8 of 512 (295) 945 and 890; K = V = 64: 8 of 512 (197)
// 707 and 729; V = 128: 16 of 512 (590) 747 and 738; a gate per channel: 16 of 64 (156) 207.9 and 209.9, 24 of 64 (233) 284 and 278, 16 of 128 (311)
// 413 and 393.  With the caches cleared between calls the line is the same (16 of 96 277 and 280, of 128 357 and 357; 8 of 512 773 and 722).  Slices
// on eight XCDs: 4 chains of 512 585 and 598, 2 of 512 431 and 463.
inline bool asks_ahead(const osdn_params *p, long long tiles, long long chains) {
    const long long K = p->K, V = p->V, kept = 2 * (64 * 64 + (p->gate_per_channel ? 5 : 2) * 64 * K + 2 * 64 * V + V * K);
    return slice_map(p->V / 16, chains, true).share && tiles * kept > 200ll << 20;
}

// Number of segments for a sequence of N chunks (params->segments > 0 overrides it; 1 = no
// pipelining).  A segment more shortens the stretch of phase 1 that runs with nothing beside it (the
// first segment of the forward pass, the last of the backward pass) and costs launches, cross-stream
// waits (25 us a call for the first) and partly filled rounds of workgroups.  Times below: one stream against the best
// of two to six segments, us, K = V = 128 in bf16.
//  - short sequences take one stream: forward up to 32 chunks (2 chains of 4 chunks 34 and 79, 64 of 16 106 and
//    127, 64 of 32 215 and 220; 64 of 48 319 and 304), backward up to 48 (2 of 4 53 and 117, 64 of 16
//    149 and 179, 8 of 32 116 and 159, 64 of 48 449 and 443, 128 of 48 773 and 755; 32 of 64 368 and 370).
//  - so do many chains, which fill the chip by themselves: 256 of 64 forward 1122 and 1182, backward 1779 and 1944;
//    from 128 chains on the forward pass takes two at most (128 of 128 1253, with four 1238, with six 1291).
//  - forward otherwise: about 16 chunks per segment, at most six segments (measured flat beyond).
//  - backward otherwise: a segment more costs more there, because every launch of the phase-2 chain kernel
//    meets a phase-1 chain kernel on the other stream and the two do not fit on one CU together:
//    when the workgroups of both (chain_wgs) outnumber the CUs, the count that balances the
//    exposed tail against that cost is about sqrt(N / 15) (2 at 64 chunks, 4 at 256); when they
//    all fit side by side, about 32 chunks per segment, at most four: of that count and the two
//    above it, the one whose segments fill whole rounds of bwd_post workgroups (one per chunk and
//    chain, post_round at a time) best; from 448 chunks on, where a segment is many rounds, seven.
//    16 chains, bf16, backward pass alone: 128 chunks 483, 503, 493, 517, 546, 575 us with 3 to 8 segments
//    (5 taken); 256 chunks, V = 256 989, 989, 1045, 1056, 1094, 1020 with 4 to 9 (5); 512 chunks 1603, 1593, 1604,
//    1599, 1623, 1769 with 4 to 8 and 12; chains that are swept, gates of 0.999, 512 chunks with 4 to 8, 10 and 12: 33 chains 2381,
//    2436, 2342, 2426, 2369, 2472, 2463; 48 2939, 2970, 2936, 2984, 2954, 3055, 3050; fp32, 8 chains 3653, 3647, 3616, 3704, 3810, 3675, 3867.
// Segments cut the chunk axis as a whole.  With packed sequences the sequential kernels of a
// segment only have the sequences that cross it to work on, one after the other segment by
// segment, so cutting pays only while one sequence makes up most of the axis; otherwise the
// many independent chains fill the chip by themselves and everything runs in one piece.
inline int segment_count(int forced, int N, int longest, long long chains, long long chain_wgs, bool backward, int post_round = 0) {
    if (forced <= 0 && (long long)longest * 4 < (long long)N * 3) return 1;
    int S = forced;
    if (forced <= 0) {
        if (N <= (backward ? 48 : 32) || chains >= NUM_CU) return 1;
        if (!backward) S = N / 16 > 6 ? 6 : N / 16;
        else if (chain_wgs > NUM_CU) S = (int)std::lround(std::sqrt(N / 15.0)) > 6 ? 6 : (int)std::lround(std::sqrt(N / 15.0));
        else {
            S = N >= 448 ? 7 : N / 32 > 4 ? 4 : N / 32;
            if (S < 2) S = 2;
            double best = 0.0;
            int pick = S;
            for (int c = S; N < 448 && c <= S + 2 && c <= N; ++c) {
                const int first = N / (2 * c) > 0 ? N / (2 * c) : 1;
                const double wgs = (double)(N - first) / (c - 1) * (double)chains;   // bwd_post workgroups of a segment
                const double fill = wgs / (std::ceil(wgs / post_round) * post_round);
                if (fill > best + 1e-9) { best = fill; pick = c; }
            }
            S = pick;
        }
        if (S < 2 || (!backward && chains * 2 >= NUM_CU)) S = 2;
    }
    if (S > MAX_SEGMENTS) S = MAX_SEGMENTS;
    if (S > N) S = N;
    return S < 1 ? 1 : S;
}
// first chunk of segment s.  Segment 0 is half as long as the others: it is the one that runs
// without a partner (phase 1 of it before anything of phase 2 can start in the forward pass,
// and after everything else in the backward pass).
// First chunk of segment s when every segment is r times as long as the one before.  Used by
// the forward pass when phase 2 is the slower of the two phases (many chains): phase 2 then
// starts early on a short segment and is never left waiting for phase 1, and the long last
// segment runs when phase 1 is already out of the way.
inline int seg_begin_grow(int N, int S, int s, double r) {
    if (s <= 0) return 0;
    if (s >= S) return N;
    const double f = (std::pow(r, s) - 1.0) / (std::pow(r, S) - 1.0);
    int b = (int)std::lround(N * f);
    if (b < s) b = s;                       // at least one chunk per segment
    if (b > N - (S - s)) b = N - (S - s);
    return b;
}
inline int seg_begin(int N, int S, int s) {
    if (s <= 0) return 0;
    if (s >= S) return N;
    const int first = N / (2 * S) > 0 ? N / (2 * S) : 1;
    return first + (int)((long long)(N - first) * (s - 1) / (S - 1));
}

// Phase 1 as sweeps over the whole sequence, for few long chains: one workgroup per chain leaves most
// of the chip idle and its walk over the chunks is most of the pass.  Every chain is cut into pieces
// (a workgroup per CU over all chains; two where a piece still has eight chunks and the kernel's registers let two onto a CU, at
// most 128: that shortens the walk more than two workgroups on a CU slow each other); a sweep runs all pieces side by
// side, each from its current start value, and leaves every piece as a composed map per
// coordinate; the next sweep walks those maps for its start values; a chain is settled when none
// of its start values moves any more.  Plain batches only.  params->p1_pieces forces a number of
// pieces per chain (-1: never), params->p1_piece_sweeps the sweep limit.
//
// Where the line lies (us per pass, sequential or in segments against pieces; K = V = 128 in bf16):
//  - forward, chains on an eighth of the CUs or fewer, from 24 chunks on: 16 chains of 24 108 and 90, with a retention
//    gate 121 and 109, of 32 136 and 97, 149 and 116, of 64 260 and 174 (pieces of 4 chunks; of 8: 221), 32 of
//    32 162 and 134; 16 chains of 16, with a gate, 90 and 94.
//  - not for more chains: how many sweeps the pieces need with a retention gate goes by how much it fades, two with gates of 0.999,
//    three to five with 0.9999 or 1, and with 33 to 64 chains only two pay (64 chains, segments and pieces, gates of 0.999, then of
//    1: forward of 32 chunks 226 and 214, 246 and 250, of 64 420 and 395, 426 and 468, of 128 761 and 697, 792 and 917, of 256 1336 and
//    1261, 1468 and 1947; backward of 64 572 and 564, 593 and 620, of 128 1025 and 1057, 1070 and 1170).
//  - how many pieces, forward without retention: 4 chains of 64 chunks 193 with 8 pieces, 144 with 16, 126 with 32; of 256 380 with
//    32, 337 with 64, 367 with 128; of 512 848, 721, 741; 2 of 1024 1600, 1270, 1152 and with 256 1238; 1 of 1024 1082 with 64, 959
//    with 128, 986 with 256.
//  - two workgroups a CU where they fit (us, one and two): forward, K = 128, one gate in bf16 (127 registers) 16 chains of 256 chunks
//    525 and 514, with gates of 1 739 and 686; where they do not, the pieces run in two rounds: one gate in fp32 (136) 1285 and 1311,
//    1526 and 1573; a gate per coordinate (159) 557 and 606, 774 and 825; backward (153 and more) 698 and 733, 807 and 844.
//  - backward, only with a retention gate (without, the solved form has the shorter chain), gates of 0.999, then of 1: 16 chains of
//    24 chunks 121 and 131, 133 and 131, of 32 144 and 141, 161 and 141, of 128 500 and 378, 569 and 408, of 512 1677 and 1341, 1897
//    and 1569; pieces of four chunks at least (16 chains of 32 chunks, gates of 0.999: pieces of two 131).
//    Not for long sequences of many chains, where segments keep phase 1 beside phase 2 (gates of 0.999, then of 1): 32 chains of 64
//    chunks 391 and 317, 431 and 347, of 128 710 and 577, 694 and 679, of 256 1216 and 1133, 1277 and 1352; with fp32 I/O and K = 128
//    16 chains of 96 959 and 910, 966 and 965, of 128 1232 and 1200, 1240 and 1268, of 256 2331 and 2344, 2336 and 2487.
//  - all this for eta up to what K allows (the sweeps over the pieces need the more the larger eta / K is, and beyond a limit do not
//    settle: 0.003 is within it by a factor of 2.1 and 1.07 for the forward pass, K = 128 and 64, of 11 and 5 for the
//    backward pass).  16 chains of 48 chunks, gates of 1, segments and pieces: forward, K = 128, eta 0.01 257 and 151, 0.03 312 and 206,
//    0.1 311 and 459; K = 64, 0.003 198 and 118, 0.01 235 and 143, 0.03 235 and 340; backward, K = 128, 0.03 266 and 222, 1 416 and
//    728, K = 64, 16 chains of 128 chunks 0.01 495 and 323, 0.1 672 and 976.  Beyond it only the forward pass of 64 chunks and more is
//    cut, into pieces of eight chunks.
inline void pieces_plan(const osdn_params *p, int N, long long chains, bool packed, bool retention, bool backward, int &pieces,
                        int &piece_chunks, int &sweeps) {
    pieces = 0; piece_chunks = 0;
    // sweeps needed without retention, measured: 4 at 64 and 128 chunks, then one more per
    // doubling (7 at 1024); the limit leaves two in hand
    sweeps = 7;                                  // (the last one only finds that nothing moved)
    for (int n = 128; n < N && sweeps < MAX_PIECE_SWEEPS; n *= 2) ++sweeps;
    if (packed || chains > MAX_PIECES / 2 || (backward && !retention)) return;
    const int forced = p->p1_pieces;              // 0: decide here; -1: never; n > 0: n pieces per chain
    int target, min_chunks;
    if (forced != 0) { target = forced > 0 ? forced : 0; min_chunks = 1; }
    else {
        if (chains * 8 > NUM_CU || N < 24) return;
        target = (int)(NUM_CU / chains);
        const bool gentle = p->eta <= (backward ? 2.5e-4f : 5e-5f) * p->K;
        if (backward && N > (chains > 16 ? 64 : p->io_dtype == OSDN_F32 && p->K == 128 && chains > 8 ? 96 : N)) return;
        if (!gentle) {
            if (backward || N < 64) return;
            min_chunks = 8;
        } else {
            const bool two = p->K == 64 || (!backward && (!retention || (p->io_dtype == OSDN_BF16 && !p->retention_per_channel)));
            if (two && N >= 16 * target) target *= 2;
            // (every workgroup walks the maps of all pieces of its chain, eight at a time; but pieces of more than eight chunks cost more than that walk)
            const int most = N <= 64 ? 16 : N <= 256 ? 32 : (N + 7) / 8;
            if (target > most) target = most;
            min_chunks = backward ? 4 : 2;
        }
    }
    if ((long long)target * chains > MAX_PIECES) target = (int)(MAX_PIECES / chains);
    if (target < 2) return;
    int len = (N + target - 1) / target;
    if (len < min_chunks) len = min_chunks;
    const int P = (N + len - 1) / len;
    if (P < 2) return;
    pieces = P; piece_chunks = len;
    if (p->p1_piece_sweeps >= 1) sweeps = p->p1_piece_sweeps;
}

// Slices of bwd_chain, 16 values or 32 (beside: a phase-1 chain runs on another stream; fp32 I/O at K = 128 always takes 16).
//  - bf16 takes 32 values beside a phase-1 chain: with 16 its workgroups hold twice the CUs, and what they
//    take from that chain, which bounds the pass there, costs more than the kernel gains.  With everything on one stream it takes 16 while the
//    workgroups find a CU each (training step, us, 32 and 16: 16 chains of 128 chunks, V = 256 848 and 836, of 24, V = 128 224 and
//    214, without retention of 32 245 and 234; 8 of 16 163 and 158; 2 of 300 799 and 697; 32 of 40 416 and 410), unless that puts the
//    slices of a chain on more XCDs than slices of 32 (backward pass: 21 chains of 32 chunks, V = 192 167 and 182).
//  - fp32 I/O at K = 64: 16 values while the
//    workgroups find a CU each (64 chains of 32 chunks, V = 64: training step 705 against 721 us; 16 chains of
//    128 chunks, V = 128: 1240 against 1400), above that 32, which read the shared tiles half as often
//    (256 chains of 16 chunks, V = 64: 1109 against 1155; 128 chains, V = 256: 1330 against 1404).
inline bool narrow_backward(const osdn_params *p, long long chains, bool beside) {
    const int slices = p->V / 16;
    if (p->io_dtype == OSDN_F32) return p->K == 128 || chains * slices <= NUM_CU;
    return !beside && chains * slices <= NUM_CU &&
           (chains <= NUM_XCD || chains % NUM_XCD == 0 || slices >= 2 * NUM_XCD || chains_filled_up(slices, chains, true));
}

// Without retention, chunks that never met the box can take the solved form of the reverse
// sweep: a dependent chain shorter than the sweeps' for 0.6 KB more memory traffic per
// token-head.  It pays while the phase-1 chain is what the pass waits for (us of the backward pass, sweeps and solved, V = K
// unless said; beta = sigmoid(N(0, 1)), then about 0.95, where a chunk takes three sweeps; the solved form knows neither):
//  - chains on at most an eighth of the CUs (K = 128, bf16: 32 of 64 chunks 430 and 380, 485 and 380; K = 64: 302 and 250);
//  - with bf16 I/O on a quarter, from 16 chunks on (48 chains, K = 128: 8 chunks 84 and 88, 16 129 and 134, with V = 64 121 and 119; 33 of 8
//    83 and 87, of 16 126 and 123; K = 64, 48 of 8 66 and 65, of 16 99 and 92; K = 64: 40 of 64 339 and 288, 64 of 32 201 and 191, of 64 395 and 352, of 128 639 and 701; K = 128:
//    40 of 64 476 and 443, 527 and 443; V = 64: 64 of 64 514 and 510, 569 and 508, of 128 916 and 1014), but for K = 128 with
//    V >= 128 beyond 48 chains, where the traffic of phase 2 fills the chip (48 of 64 507 and 500, 559 and 501; 64 of 32 319 and
//    328, 350 and 327; 64 of 64 611 and 636, 668 and 637; 64 of 128 1102 and 1200, 1163 and 1200).
// longest: chunks of the longest sequence
inline bool solved_plan(const osdn_params *p, long long chains, int longest, bool retention) {
    const bool bf = p->io_dtype == OSDN_BF16, quarter = bf && longest >= 16 && !(p->K == 128 && p->V >= 128 && chains > 48);
    if (retention) return !p->retention_per_channel && p->p1_solved > 0;       // (the form with a retention gate and any masks)
    return p->p1_solved > 0 || (p->p1_solved == 0 && chains * (quarter ? 4 : 8) <= NUM_CU);
}

}  // namespace osdn
