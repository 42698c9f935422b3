// Phase 2 backward of OSDN in chunkwise form.  The paper prints only the chain rule through
// k~ = d . k (Section 4.5); the chunk-level adjoints below are plain matrix calculus on the
// forward formulas (Appendix A.2 / B.1), per chunk, with S the state at the start of the
// chunk, dS' the adjoint of the state at its end, G the in-chunk cumulative log-decay,
// gamma = e^G, rho = e^{G_C - G}, Gamma_ij = e^{G_i - G_j}:
//
//   forward:  A = tril(beta_i Gamma_ij <k_i,k~_j>, -1), T = (I+A)^-1, R0 = V - gamma.(K S^T),
//             E = T (beta . R0), P = tril(Gamma . Q K~^T), O = scale[gamma.(Q S^T) + P E],
//             S' = gamma_C S + E^T (rho . K~)
//   bwd_chain (sequential, right to left, per (b, h, slice of V)):
//             dE = scale P^T dO + (rho . K~) dS'^T ;  dS = gamma_C dS' + scale dO^T (gamma . Q) - dE^T W
//             (P is the tile output_fwd left; q and dO are read where the caller put them)
//   bwd_post  (parallel):  dR = T^T dE ; dV = beta . dR ; dA = -tril(dR E^T, -1) ;
//             dP = scale tril(dO E^T) ; cA = dA . beta_i Gamma ; cP = dP . Gamma ;
//             dQ = cP K~ + scale gamma . (dO S) ; dK = cA K~ - gamma beta . (dR S) ;
//             dK~ = cA^T K + cP^T Q + rho . (E dS') ;
//             dbeta_i = <dR_i, R0_i> + sum_j dA_ij Gamma_ij <k_i,k~_j> ;
//             dG from every place G enters; dlog_alpha = suffix sums of dG inside the chunk.
//
// With one state gate per key channel (GV) the same kernels run, ungated, on the operands in
// which the forward pass folded the channel decays (Gamma . Q, Gamma . K, K~ / Gamma); S' =
// S Diag(gamma_C) + E^T (gamma_C . K~ / Gamma) with the chunk's decay per channel gamma_C, whose last
// operand takes the place of rho . K~, and the unfold kernel at the end of this file maps the
// gradients back to q, k, k~ and log alpha.
#include "osdn_kernels.h"
#include "osdn_tile.h"

namespace osdn {


// sum over the 16 lanes of a DPP row (lanes sharing lane>>4), returned to all of them
__device__ __forceinline__ float row16_sum(float x) {
    x += dpp_f32<0xB1>(x);
    x += dpp_f32<0x4E>(x);
    x += dpp_f32<0x141>(x);
    x += dpp_f32<0x140>(x);
    return x;
}

// a fragment times one factor per value of the contraction index (rounded once more to the I/O type)
__device__ __forceinline__ bf16x8 scale_frag(bf16x8 f, const float *g) {      // g: 8 factors, 32-byte aligned, in LDS
    const f32x4 g0 = *reinterpret_cast<const f32x4 *>(g), g1 = *reinterpret_cast<const f32x4 *>(g + 4);
    const u32x4 w = __builtin_bit_cast(u32x4, f);
    bf16x8 o;
#pragma unroll
    for (int e = 0; e < 8; ++e) o[e] = (bf16)(vec_get<bf16>(w, e) * (e < 4 ? g0[e & 3] : g1[e & 3]));
    return o;
}
__device__ __forceinline__ float scale_frag(float f, const float *g) { return f * *g; }

// ------------------------------------------------------------- bwd_chain ----
// Right to left over the chunks of one chain, one workgroup per slice of VS rows of dS: eight wavefronts on the chain (two barriers per
// chunk), four that move the operands in and the dS' checkpoint and dE^T out (as in state_fwd_kernel):
//   A  dS', rounded to the I/O type, into LDS                                        | barrier 1
//   B  dE = scale P^T dO + rho . (K~ dS'^T), one 16x16 tile per wavefront, into LDS  | barrier 2
//   C  dS <- gamma_C dS' + scale (gamma . dO)^T Q - dE^T W in the MFMA accumulators (the part
//      without dE already in phase B)
// The operands come as the forward pass and the caller left them (K~, -W, P, q, the slice of dO, all
// in their natural [token][feature] layout; those whose contraction index runs down the rows are
// fetched with the LDS transpose read), by direct global -> LDS loads into two rings, and with bf16 I/O are in
// registers when the phase that multiplies them begins (PRE; fp32 fragments would not fit): what phase B needs (K~; P
// and dO, whose product and whose scaled fragments are formed at once; the gates) is prepared in
// phase C of the chunk before, what phase C needs (-W, q) in phase B.  64 chains of 64 chunks, K = V =
// 128 in bf16: 134 us; with the tiles staged through registers by loader wavefronts, 157 us (16 chains of
// 128 chunks, V = 256: 206 against 282 us; with slices of 16 whose lines are asked for ahead 161).
constexpr int CW_ = 8, CM_ = 2, CS_ = 2, CT_ = (CW_ + CM_ + CS_) * 64;     // wavefronts that compute, load, store; threads
// ring depths (chunks of operands in LDS) of what phase B takes and of what phase C takes, from what fits the LDS
template <typename T, int K> constexpr int BC_NSB = sizeof(T) == 2 ? 2 : (K == 64 ? 2 : 1);
template <typename T, int K> constexpr int BC_NSC = sizeof(T) == 2 ? 2 : 1;

// GV: one state gate per key channel: every coordinate of dS has its own gamma_C, and K~ is
// gamma_C . K~ / Gamma.  dS' itself is rounded and kept: gamma_C . dS' would lose bits, and then
// itself, below the smallest normal number (at a decay of e^-79 from |dS'| = 2.4e-4 on), which K~ /
// Gamma would bring back to the size of dS'.
// VS: rows of S (values) owned by one workgroup, 32 or 16 (launch_chain_v says which).
template <typename T, int K, bool GV, int VS, bool RAG>
__global__ __launch_bounds__(CT_) void bwd_chain_kernel(ChunkArgs a) {
    constexpr int ES = sizeof(T), RK = K * ES, RC = C * ES, RV = VS * ES;      // bytes per row of a tile
    constexpr int NVT = VS / 16, NFB = K / 16;
    constexpr int NTC = NFB * NVT, TPW = NTC > CW_ ? NTC / CW_ : 1;            // state tiles, ... per wavefront
    constexpr int KS = Mfma<T>::KSTEP, NKK = K / KS, NKC = C / KS;
    typedef typename Mfma<T>::Frag Frag;
    constexpr bool PRE = sizeof(T) == 2;        // operands in registers ahead of their phase (fp32: they would not fit)
    constexpr int NSB = BC_NSB<T, K>, NSC = BC_NSC<T, K>;
    constexpr int B_K = 0, B_P = B_K + C * RK, B_O = B_P + C * RC, B_G = B_O + C * RV, B_BYTES = B_G + 2 * C * 4;
    constexpr int C_W = 0, C_Q = C_W + C * RK, C_D = C_Q + C * RK, C_BYTES = C_D + (GV ? K * 4 : 0);
    __shared__ __attribute__((aligned(1024))) char ringB[NSB * B_BYTES];
    __shared__ __attribute__((aligned(1024))) char ringC[NSC * C_BYTES];
    __shared__ __attribute__((aligned(1024))) char dSb[VS * RK];        // dS' in the I/O type [v][kf]
    __shared__ __attribute__((aligned(1024))) char dEs[VS * RC];        // dE^T [v][i]
    constexpr bool TOUCH = PRE && VS == 16;
    constexpr int PF = 8;
    __shared__ __attribute__((aligned(1024))) char dump[TOUCH ? 256 : 16];

    int chain = 0, slice = 0;
    chain_slice_of(blockIdx.x, a.map, chain, slice);
    if (chain >= a.map.chains) return;
    const int vs = slice * VS, h = chain % a.H;
    int b = chain / a.H;                        // batch entry, or packed sequence
    int bt = b;                                 // batch entry of the token tensors
    if (a.seq_chunks) {
        b = sequence_of(a.seq_chunks, a.n_seqs, b);
        bool begins, ends;
        if (!clip_to_sequence(a.seq_chunks, b, a.n0, a.n1, begins, ends)) return;
        a.dS_out = ends ? a.dS_last : a.dS_in;
        bt = 0;
    }
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const bool loader = wave >= CW_ && wave < CW_ + CM_, storer = wave >= CW_ + CM_;
    const int mw = wave - CW_, mt = tid - (CW_ + CM_) * 64;     // loader wavefront, storer thread
    const size_t bh = (size_t)b * a.H + h;      // the chain: indexes dS_out / dS_in
    const uint32_t gK = (uint32_t)a.H * RK, gV = (uint32_t)a.H * (uint32_t)a.V * ES;   // bytes between tokens
    const bool wideO = (reinterpret_cast<uintptr_t>(a.dO) & 15) == 0, wideQ = (reinterpret_cast<uintptr_t>(a.q) & 15) == 0;

    LdsLoad<RK, C, CM_> lK, lQ;                 // (tiles of the workspace; q where the caller put it)
    LdsLoad<RC, C, CM_> lP;
    LdsLoad<RV, C, CM_> lO;
    lK.init(RK, mw, lane); lQ.init(gK, mw, lane); lP.init(RC, mw, lane); lO.init(gV, mw, lane);
    const ChainRows<RAG> rows(a.rows, a.seq_chunks, b, a.n0);
    auto loadB = [&](int n, int slot) {
        const size_t bhn = ((size_t)bt * a.N + n) * a.H + h, tok = rows.first(n) * a.H + h;
        char *s = ringB + slot * B_BYTES;
        lK.issue(s + B_K, static_cast<const char *>(a.kt) + bhn * C * RK, RK, mw, lane, slice);
        lP.issue(s + B_P, static_cast<const char *>(a.Pm) + bhn * C * RC, RC, mw, lane, slice);
        lO.issue(s + B_O, static_cast<const char *>(a.dO) + tok * a.V * ES + (size_t)vs * ES, gV, mw, lane, 0, wideO, rows.count(n) - 1);
        if (!GV && mw < 2) {                    // gamma (loader 0) and rho (1)
            const int w = mw;
            load_lds4(a.gates + (bhn * 3 + 1 + w) * C, lane * 4, lds_offset(s + B_G + w * C * 4));
        }
    };
    auto loadC = [&](int n, int slot) {
        const size_t bhn = ((size_t)bt * a.N + n) * a.H + h, tok = rows.first(n) * a.H + h;
        char *s = ringC + slot * C_BYTES;
        lK.issue(s + C_W, static_cast<const char *>(a.Wn) + bhn * C * RK, RK, mw, lane, slice);
        if (GV) lK.issue(s + C_Q, static_cast<const char *>(a.q) + bhn * C * RK, RK, mw, lane, slice);
        else lQ.issue(s + C_Q, static_cast<const char *>(a.q) + tok * RK, gK, mw, lane, slice, wideQ, rows.count(n) - 1);
        if (GV && mw < K / 64)
            load_lds4(a.gamC + bhn * K, mw * 256 + lane * 4, lds_offset(s + C_D + mw * 256));
    };
    // loads of a loader that are newer than the tiles it waits for (at least)
    constexpr int LB = LdsLoad<RK, C, CM_>::MIN + LdsLoad<RC, C, CM_>::MIN + LdsLoad<RV, C, CM_>::MIN, LC = 2 * LdsLoad<RK, C, CM_>::MIN;
    constexpr int NMAX = NSB > NSC ? NSB : NSC;
    constexpr int NEWER_B = (NSB - 1) * (LB + LC), NEWER_C = (NSC - 1) * (LB + LC);
    static_assert(NEWER_B < 64 && NEWER_C < 64, "the counter has six bits");
#pragma unroll
    for (int j = 0; j < NMAX; ++j) {
        if (loader && j < NSB && a.n1 - 1 - j >= a.n0) loadB(a.n1 - 1 - j, j);
        if (loader && j < (PRE ? NSC : NSC - 1) && a.n1 - 1 - j >= a.n0) loadC(a.n1 - 1 - j, j);
    }

    // this wavefront's tiles of dS (feature block fb, value blocks vtC ..) and of dE (row block rb, value block vtB)
    const bool inC = wave * TPW < NTC, inB = wave < 4 * NVT;
    const int fb = wave % NFB, vtC = wave / NFB;
    const int rb = wave & 3, vtB = wave >> 2;
    f32x4 dSt[TPW] = {};                        // rows = features, cols = values
    if (inC) {
#pragma unroll
        for (int q = 0; q < TPW; ++q) {
            const int v = vs + (vtC + q) * 16 + acc_col(lane), c0 = fb * 16 + acc_row(lane, 0);
            if (a.dS_out) dSt[q] = *reinterpret_cast<const f32x4 *>(a.dS_out + (bh * a.V + v) * K + c0);
        }
    }
    if (loader) wait_vm<0>();
    __syncthreads();
    if (const int cnt = rows.count(a.n1 - 1); cnt < C) {        // (only the first chunk here can have missing tokens) their dO is zero
        for (int i = tid; i < (C - cnt) * (RV / 16); i += CT_)
            *reinterpret_cast<u32x4 *>(ringB + B_O + cnt * RV + i * 16) = u32x4{0u, 0u, 0u, 0u};
        __syncthreads();
    }
    int sb = 0, sc = 0;                         // ring slots of chunk n
    if (loader) {
        // (all is there; said to the compiler too, which does not count wait_vm: it would wait for the state's loads where
        // their registers are used again in the loop, and with them for every tile on its way: 122 -> 142 us)
        __builtin_amdgcn_s_waitcnt(0x0f70);     // vmcnt(0)
        // A slot is refilled once its operands have been read.  PRE: those of phase B are read in phase C of the chunk before, those of phase
        // C in phase B, so that B's slot is free behind barrier 1 and C's behind barrier 2.  Barrier 1 then opens on C of this chunk, behind which B and
        // C of the next NSC - 1 have been asked for (NEWER_C), barrier 2 on B of the next, behind which C of it and B of the one after have
        // (NSB = 2: NEWER_B).  Not PRE: either is read in its own phase; barrier 1 opens on B of this chunk, behind which C of the chunk before and
        // B of the next have been asked for (NSB = 2; NSB = 1: nothing), barrier 2 on C, asked for behind barrier 1.
        for (int n = a.n1 - 1; n >= a.n0; --n) {
            const bool full = n - NMAX >= a.n0; // everything counted as newer has been asked for
            if (full) wait_vm<PRE ? NEWER_C : NEWER_B>(); else wait_vm<0>();
            __syncthreads();                                        // barrier 1
            if (PRE && n - NSB >= a.n0) loadB(n - NSB, sb);
            if (!PRE && n + 1 - NSC >= a.n0) loadC(n + 1 - NSC, sc == 0 ? NSC - 1 : sc - 1);
            if (full) wait_vm<PRE ? NEWER_B : NEWER_C>(); else wait_vm<0>();
            __syncthreads();                                        // barrier 2
            if (PRE && n - NSC >= a.n0) loadC(n - NSC, sc);
            if (!PRE && n - NSB >= a.n0) loadB(n - NSB, sb);
            sb = sb + 1 == NSB ? 0 : sb + 1;
            sc = sc + 1 == NSC ? 0 : sc + 1;
        }
        return;
    }
    if (storer) {
        // TOUCH: this slice's share of the lines of a chunk's operands, in the order K~, -W, P, gates, q, dO, asked for PF chunks ahead
        // (whole chunks all, as only a sequence's last may be ragged): lane l asks for the l-th, the (64 + l)-th and the
        // (128 + l)-th, whose addresses step from chunk to chunk
        constexpr int GS = (GV ? K : 3 * C) * 4, LK = C * RK / LINE, LP = C * RC / LINE, LG = (GV ? K : 2 * C) * 4 / LINE, L0 = 2 * LK + LP + LG;
        constexpr int QR = RK / LINE;           // lines of a row of q
        const int lpr = a.V * ES / LINE, all = L0 + C * QR + C * lpr, share = (all + a.V / VS - 1) / (a.V / VS);
        // From 128 workgroups on, whose loads make lines from HBM late (backward pass, us, without and with, calls repeated, then with the caches
        // cleared between them: 128 workgroups, 16 chains of 32 chunks 134.0 and 134.8, 169.6 and 160.0, of 128 chunks 415 and 382, 465 and 418, a
        // gate per channel, 32 chunks 149.2 and 149.7, 194.2 and 185.2, 4 chains of 128, V = 512, on eight XCDs each 288 and 276, 357 and 315;
        // 256, 16 chains of 32, V = 256, a gate per channel 188 and 179, 216 and 204; 160, 10 of 32, V = 384 152.7 and 156.0, 198 and 187;
        // training step, calls repeated: 16, 300 chunks 698 and 698; 64 with K = 64, 16 chunks 131.7 and 132.2; 32 with channel gates, 40 chunks 243
        // and 247).
        const bool touches = TOUCH && gridDim.x >= 128 && wave == CW_ + CM_ + 1;
        const char *lp[TOUCH ? 3 : 1] = {};
        uint32_t ls[TOUCH ? 3 : 1] = {};
        bool own[TOUCH ? 3 : 1] = {};
        if (touches) {
            const size_t t1 = ((size_t)bt * a.N + a.n1 - 1) * a.H + h;
#pragma unroll
            for (int j = 0; j < (TOUCH ? 3 : 1); ++j) {
                const int i = lane + 64 * j, l = slice * share + i;
                own[j] = i < share && l < all;
                if (l < LK) { lp[j] = static_cast<const char *>(a.kt) + t1 * C * RK + l * LINE; ls[j] = C * RK; }
                else if (l < 2 * LK) { lp[j] = static_cast<const char *>(a.Wn) + t1 * C * RK + (l - LK) * LINE; ls[j] = C * RK; }
                else if (l < 2 * LK + LP) { lp[j] = static_cast<const char *>(a.Pm) + t1 * C * RC + (l - 2 * LK) * LINE; ls[j] = C * RC; }
                else if (l < L0) { lp[j] = reinterpret_cast<const char *>(GV ? a.gamC : a.gates + C) + t1 * GS + (l - 2 * LK - LP) * LINE; ls[j] = GS; }
                else if (l < L0 + C * QR) {
                    const int r = (l - L0) / QR, c = (l - L0) % QR;
                    lp[j] = static_cast<const char *>(a.q) + (GV ? t1 * C + r : (rows.first(a.n1 - 1) + r) * a.H + h) * RK + c * LINE;
                    ls[j] = C * RK;
                } else {
                    const int r = (l - L0 - C * QR) / lpr;
                    lp[j] = static_cast<const char *>(a.dO) + ((rows.first(a.n1 - 1) + r) * a.H + h) * a.V * ES + (l - L0 - C * QR) % lpr * LINE;
                    ls[j] = C * a.V * ES;
                }
            }
        }
        int stand = a.n1 - 1;                   // the chunk that lp stands at
        for (int n = a.n1 - 1; n >= a.n0; --n) {
            const size_t bhn = ((size_t)bt * a.N + n) * a.H + h;
            __syncthreads();                                        // barrier 1
            tile_to_global<RK, VS>(static_cast<char *>(a.dS_ckpt) + (bhn * a.V + vs) * RK, RK, dSb, mt, CS_ * 64);
            __syncthreads();                                        // barrier 2
            tile_to_global<RC, VS>(static_cast<char *>(a.dEt) + (bhn * a.V + vs) * RC, RC, dEs, mt, CS_ * 64);
            if (touches && n - PF >= a.n0) {
                const size_t step = (size_t)(stand - (n - PF)) * a.H;
                stand = n - PF;
#pragma unroll
                for (int j = 0; j < (TOUCH ? 3 : 1); ++j) {
                    if (64 * j >= share) break;
                    lp[j] -= step * ls[j];
                    if (own[j]) touch(lp[j], lds_offset(dump));
                }
            }
        }
        if (touches) wait_vm<0>();
        return;
    }
    TileFrag<T, RK> fK;
    TileFrag<T, RC> fC;
    TileFrag<T, RV> fV;
    fK.init(lane); fC.init(lane); fV.init(lane);
    // operands of phase B of one chunk: fragments of K~, P^T dO, rho of this lane's rows; gamma_C and
    // the scaled fragments of dO, which phase C multiplies
    Frag kf[NKK], of[TPW][NKC];
    f32x4 loc = {}, rho = {1.f, 1.f, 1.f, 1.f};
    float gC = 1.f;
    auto fetchB = [&](const char *tB) {
        if (inB) {
            if (PRE) {
#pragma unroll
                for (int kk = 0; kk < NKK; ++kk) kf[kk] = fK.kc(tB + B_K, rb * 16, kk * KS);
            }
            loc = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int kk = 0; kk < NKC; ++kk)
                if (kk * KS + KS > rb * 16)                     // P[i'][i] = 0 for i' < i
                    loc = Mfma<T>::mma(fC.tr(tB + B_P, kk * KS, rb * 16), fV.tr(tB + B_O, kk * KS, vtB * 16), loc);
            if (!GV) rho = *reinterpret_cast<const f32x4 *>(tB + B_G + (rb * 16 + acc_row(lane, 0)) * 4 + C * 4);
        }
        if (inC) {
#pragma unroll
            for (int q = 0; q < TPW; ++q)
#pragma unroll
                for (int kk = 0; kk < NKC; ++kk) {
                    of[q][kk] = fV.tr(tB + B_O, kk * KS, (vtC + q) * 16);
                    if (!GV) of[q][kk] = scale_frag(of[q][kk], reinterpret_cast<const float *>(tB + B_G) + kk * KS + (lane >> 4) * (KS / 4));
                }
        }
        if (!GV) gC = *reinterpret_cast<const float *>(tB + B_G + (C - 1) * 4);
    };
    if (PRE) fetchB(ringB);
    for (int n = a.n1 - 1; n >= a.n0; --n) {
        const char *tB = ringB + sb * B_BYTES, *tC = ringC + sc * C_BYTES;
        // ---- phase A ----
        if (inC) {
#pragma unroll
            for (int q = 0; q < TPW; ++q) fK.put(dSb, (vtC + q) * 16, fb * 16, dSt[q]);
        }
        __syncthreads();                                            // barrier 1
        // ---- phase B ----
        Frag sf[NKK], qf[NKC], wf[NKC];
        f32x4 dc = {};
        if (!PRE) fetchB(tB);
        if (inB) {
#pragma unroll
            for (int kk = 0; kk < NKK; ++kk) sf[kk] = fK.kc(dSb, vtB * 16, kk * KS);
        }
        if (PRE && inC) {
#pragma unroll
            for (int kk = 0; kk < NKC; ++kk) qf[kk] = fK.tr(tC + C_Q, kk * KS, fb * 16);
#pragma unroll
            for (int kk = 0; kk < NKC; ++kk) wf[kk] = fK.tr(tC + C_W, kk * KS, fb * 16);
            if (GV) dc = *reinterpret_cast<const f32x4 *>(tC + C_D + (fb * 16 + acc_row(lane, 0)) * 4);
        }
        if (inB) {
            f32x4 acc = {0.f, 0.f, 0.f, 0.f}, acc2 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int kk = 0; kk < NKK; kk += 2) {
                acc = Mfma<T>::mma(PRE ? kf[kk] : fK.kc(tB + B_K, rb * 16, kk * KS), sf[kk], acc);
                acc2 = Mfma<T>::mma(PRE ? kf[kk + 1] : fK.kc(tB + B_K, rb * 16, (kk + 1) * KS), sf[kk + 1], acc2);
            }
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[r] = __builtin_fmaf(rho[r], acc[r] + acc2[r], a.scale * loc[r]);
            fC.put(dEs, vtB * 16, rb * 16, acc);
        }
        auto withoutE = [&] {                   // what does not need dE
#pragma unroll
            for (int q = 0; q < TPW; ++q) {
                f32x4 part = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int kk = 0; kk < NKC; ++kk) part = Mfma<T>::mma(PRE ? qf[kk] : fK.tr(tC + C_Q, kk * KS, fb * 16), of[q][kk], part);
#pragma unroll
                for (int r = 0; r < 4; ++r) dSt[q][r] = __builtin_fmaf(GV ? dc[r] : gC, dSt[q][r], a.scale * part[r]);
            }
        };
        if (PRE && inC) withoutE();
        __syncthreads();                                            // barrier 2
        // ---- phase C ----
        if (inC) {
            Frag fe[TPW][NKC];
            if (!PRE) {
                if (GV) dc = *reinterpret_cast<const f32x4 *>(tC + C_D + (fb * 16 + acc_row(lane, 0)) * 4);
                withoutE();
            }
#pragma unroll
            for (int q = 0; q < TPW; ++q)
#pragma unroll
                for (int kk = 0; kk < NKC; ++kk) fe[q][kk] = fC.kc(dEs, (vtC + q) * 16, kk * KS);
#pragma unroll
            for (int q = 0; q < TPW; ++q)
#pragma unroll
                for (int kk = 0; kk < NKC; ++kk) dSt[q] = Mfma<T>::mma(PRE ? wf[kk] : fK.tr(tC + C_W, kk * KS, fb * 16), fe[q][kk], dSt[q]);
        }
        sb = sb + 1 == NSB ? 0 : sb + 1;
        sc = sc + 1 == NSC ? 0 : sc + 1;
        if (PRE && n > a.n0) fetchB(ringB + sb * B_BYTES);
    }
    if (inC) {
#pragma unroll
        for (int q = 0; q < TPW; ++q) {
            const int v = vs + (vtC + q) * 16 + acc_col(lane), c0 = fb * 16 + acc_row(lane, 0);
            *reinterpret_cast<f32x4 *>(a.dS_in + (bh * a.V + v) * K + c0) = dSt[q];
        }
    }
}

// -------------------------------------------------------------- bwd_post ----
// One workgroup of 8 wavefronts per chunk and head.  V is walked in slabs of VB columns; the slab
// buffers are reused for Q and K~ once the walk is over, and so are the registers that carry the next
// slab while the workgroup computes on this one.
//
// Two workgroups share a CU with bf16 I/O (slabs of 32 columns: 80 KB of LDS; at most 128 registers, which
// is why the scheduler is fenced in below), so that one computes while the other waits for its tiles or at
// one of its barriers.  Every product is formed with the features (values, or j of a 64 x 64 matrix)
// down the rows of the accumulator and the tokens across: a lane then holds four adjacent features of one
// token, so that results leave as 8-byte stores (dv from the accumulators), operands come as
// 8-byte reads, gates are one number per lane and sums over features need two lane swaps.
// 16816 chunk-heads, K = V = 128 in bf16: 900 us (4.1 GB needed); with tokens down the rows, 1019; one workgroup
// per CU on slabs of 64, two chunks in turn, 1072.
template <typename T> constexpr int BP_WGS = sizeof(T) == 2 ? 2 : 1;      // workgroups that share a CU

// GV: one state gate per key channel.  The kernel then runs on the folded operands with no
// scalar gate (log_alpha null) and takes gamma_C, per channel, in place of rho (see the top of this
// file); the gradient of the chunk's decays, times the decays, is collected per channel.
template <typename T, int K, bool GV, int PW_, bool RAG>
__global__ __launch_bounds__(PW_ * 64, (BP_WGS<T>) * PW_ / 4) void bwd_post_kernel(ChunkArgs a) {
    constexpr int PT_ = PW_ * 64;
    constexpr int PAD = sizeof(T) == 2 ? 16 : Pad<T>::v, LDK = K + PAD, LDE = C + PAD;   // bf16: rows 32 bytes apart modulo 128
    constexpr int LDC = C + Pad<T>::v;                  // (T, cA, cP)
    constexpr int VB = 32;                              // slab width
    constexpr int LDV = VB + PAD;
    constexpr int NVT = VB / 16;                         // column tiles of a slab
    constexpr int WPR = PW_ / 4;                         // wavefronts that share a row block in steps (1), (2)
    constexpr int NVW = NVT / WPR;                       // column tiles of a slab per wavefront there
    static_assert(NVT % WPR == 0 && NVW >= 1, "slab too narrow for this many wavefronts");
    constexpr int NCT = K / 16;                          // column tiles of the [64 x K] results
    constexpr int WPC = PW_ / NCT > 0 ? PW_ / NCT : 1;   // wavefronts per column tile ...
    constexpr int IBN = 4 / WPC;                         // ... and row blocks per wavefront
    static_assert(WPC <= 4 && 4 % WPC == 0, "column tiles / wavefronts");
    constexpr int NLT = (10 + PW_ - 1) / PW_;            // lower 16x16 tiles per wavefront
    constexpr int KS = Mfma<T>::KSTEP;
    // persistent
    __shared__ __attribute__((aligned(16))) T Ks[C * LDK];
    __shared__ __attribute__((aligned(16))) T Tt[C * LDC];       // T; after the walk: cA
    __shared__ __attribute__((aligned(16))) float Gs[C];
    __shared__ float Bs[C];
    __shared__ float Egs[C], Ers[C];                     // gamma_i = e^{G_i} and rho_i = e^{G_C - G_i}, once per row
    __shared__ float red[4 * C];                         // [4][64] partial sums across tiles
    __shared__ float red2[GV ? 1 : 4 * C];               // (with per-channel gates dG is not collected here)
    __shared__ __attribute__((aligned(16))) float red3[GV ? 1 : 4 * C];
    __shared__ float dbeta_s[WPR * C];
    __shared__ float sdot[PW_], trsum_s[PW_];
    __shared__ float colss[GV ? PT_ : 1];                // <dS', S> column by column (partials)
    __shared__ __attribute__((aligned(16))) float dgam_s[GV ? (PW_ / (K / 16) > 0 ? PW_ / (K / 16) : 1) * K : 1];   // gamma_C sum_i (K~/Gamma)_ic (E dS')_ic, per row-block group
    // slab buffers, later Q / K~ / cP and the row-dot partials
    constexpr int SLAB_ELEMS = 3 * C * LDV + 2 * VB * LDE + 2 * VB * LDK;
    constexpr int POST_ELEMS = 2 * C * LDK + C * LDC + (GV ? 0 : (PW_ * C * 4) / (int)sizeof(T));
    constexpr int POOL = SLAB_ELEMS > POST_ELEMS ? SLAB_ELEMS : POST_ELEMS;
    __shared__ __attribute__((aligned(16))) T pool[POOL];
    T *dOs = pool;                      // [64][LDV]  dO slab (natural), later dV staging
    T *Vs = dOs + C * LDV;              // [64][LDV]  V slab
    T *dRs = Vs + C * LDV;              // [64][LDV]  dR slab (natural)
    T *Ets = dRs + C * LDV;             // [VB][LDE]  E^T slab
    T *dEts = Ets + VB * LDE;           // [VB][LDE]  dE^T slab
    T *Ss = dEts + VB * LDE;            // [VB][LDK]  S slab
    T *dSs = Ss + VB * LDK;             // [VB][LDK]  dS' slab
    T *Qs = pool;                       // after the walk
    T *Kts = Qs + C * LDK;
    T *cPs = Kts + C * LDK;             // [64][LDC]
    float *pq = reinterpret_cast<float *>(cPs + C * LDC);        // [PW_][64]
    T *cAs = Tt;                        // [64][LDC]

    const int n = a.n0 + (int)(blockIdx.x / a.H), h = blockIdx.x % a.H, b = blockIdx.y;
    int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const size_t bhn = ((size_t)b * a.N + n) * a.H + h;
    const size_t tok0 = a.rows.first<RAG>(b, n) * a.H + h;
    const int rows = a.rows.count<RAG>(n);           // tokens that exist; the others: dO and v zero, beta zero, the rest repeats the last one
    const size_t tstride = a.H;
    // the slab tiles travel through registers: the next slab (after the last one: Q and K~) is
    // fetched while the workgroup computes on the current one
    PairRegs<T, C, VB, PT_> r_dOV;
    PairRegs<T, VB, C, PT_> r_EdE;
    TileRegs<T, VB, K, PT_> r_S, r_dS;                  // after the last slab: the two halves of Q (and K~ in r_dOV, r_EdE)
    static_assert(2 * VB == C, "halves of Q");
    constexpr int NVP = PairRegs<T, C, VB, PT_>::NVP;
    TileRegs<T, C, K, PT_> r_Kn;
    static_assert(TileRegs<T, C, K, PT_>::NV <= 2 * NVP, "K~ fits the registers of the slab");
    TileRegs<T, C, C, PT_> r_Tn;
    float r_g = 0.f, r_b = 0.f;
    auto fetch_slab = [&](int v0) {
        r_EdE.fetch(static_cast<const T *>(a.Et) + (bhn * a.V + v0) * C, static_cast<const T *>(a.dEt) + (bhn * a.V + v0) * C, (size_t)C, tid, wave);
        r_S.fetch(static_cast<const T *>(a.S_ckpt) + (bhn * a.V + v0) * K, (size_t)K, tid);
        r_dS.fetch(static_cast<const T *>(a.dS_ckpt) + (bhn * a.V + v0) * K, (size_t)K, tid);
        r_dOV.fetch(static_cast<const T *>(a.dO) + tok0 * a.V + v0, static_cast<const T *>(a.v) + tok0 * a.V + v0, tstride * a.V, tid, wave, rows - 1);
    };
    if (wave == 0) {
        r_g = a.log_alpha ? a.gates[bhn * 3 * C + lane] : 0.f;
        r_b = lane < rows ? a.beta[tok0 + (size_t)lane * tstride] : 0.f;
    }
    r_Kn.fetch(static_cast<const T *>(a.k) + (GV ? bhn * C : tok0) * K, GV ? (size_t)K : tstride * K, tid, GV ? C - 1 : rows - 1);
    r_Tn.fetch(static_cast<const T *>(a.Tm) + bhn * C * C, (size_t)C, tid);
    fetch_slab(0);
    const int ct = (wave % NCT) * 16;   // this wave's column tile of the [64 x K] results ...
    const int ib0 = (wave / NCT) * IBN; // ... and its first row block
    const bool has_ct = wave < NCT * WPC;

    if (wave == 0) {
        const float G = r_g;
        Gs[lane] = G;
        Egs[lane] = __expf(G);
        Ers[lane] = __expf(lane_bcast63(G) - G);
        Bs[lane] = r_b;
    }
    r_Kn.put(Ks, LDK, tid);
    r_Tn.put(Tt, LDC, tid);

    // accumulators over the walk
    f32x4 dP[NLT], dA[NLT];             // the lower tiles idx = wave, wave + PW_ (< 10)
    f32x4 dQg[IBN], dKg[IBN], dKr[IBN]; // [row block ib0 + .], column tile ct
    float dbeta_part = 0.f;             // token 16*rb + acc_col(lane), this lane's values
    float ss_part = 0.f;                // <dS', S>
#pragma unroll
    for (int t = 0; t < NLT; ++t) { dP[t] = f32x4{0.f, 0.f, 0.f, 0.f}; dA[t] = f32x4{0.f, 0.f, 0.f, 0.f}; }
#pragma unroll
    for (int ib = 0; ib < IBN; ++ib) {
        dQg[ib] = f32x4{0.f, 0.f, 0.f, 0.f};
        dKg[ib] = f32x4{0.f, 0.f, 0.f, 0.f};
        dKr[ib] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    const int rb = wave / WPR;          // row block of steps (1), (2)

    // (the thread index is made opaque here and there, so that the lane addresses of what follows are not
    // all computed far ahead and kept in registers; and the scheduler is kept from mixing the row blocks)
#define OSDN_BP_FRESH() asm volatile("" : "+v"(tid), "+v"(lane))
    for (int v0 = 0; v0 < a.V; v0 += VB) {
        OSDN_BP_FRESH();
        __syncthreads();
        if (rows < C) r_dOV.cut(tid, rows - 1);
        r_dOV.put(dOs, Vs, LDV, tid, wave);
        r_EdE.put(Ets, dEts, LDE, tid, wave);
        r_S.put(Ss, LDK, tid); r_dS.put(dSs, LDK, tid);
        if (!GV) ss_part = TileRegs<T, VB, K, PT_>::dot(r_S, r_dS, ss_part, tid);      // <dS', S> over this slab
        if (v0 + VB < a.V) {
            fetch_slab(v0 + VB);
        } else {
            const size_t ldq = GV ? (size_t)K : tstride * K;
            const T *qp = static_cast<const T *>(a.q) + (GV ? bhn * C : tok0) * K;
            const int lastq = GV ? C - 1 : rows - 1;
            r_S.fetch(qp, ldq, tid, lastq);
            if (lastq >= VB) r_dS.fetch(qp + VB * ldq, ldq, tid, lastq - VB);
            else r_dS.fetch(qp, ldq, tid, 0);            // (of no consequence: cP and dq have no such rows)
            TileRegs<T, C, K, PT_> r_Kt;
            r_Kt.fetch(static_cast<const T *>(a.kt) + bhn * C * K, (size_t)K, tid);
#pragma unroll
            for (int m = 0; m < r_Kt.NV; ++m) (m < NVP ? r_dOV.vec(m) : r_EdE.vec(m - NVP)) = r_Kt.v[m];
        }
        __syncthreads();
        // <dS', S> over this slab with per-channel gates: column by column, thread tid keeps column tid % K
        if (GV) {
            for (int idx = tid; idx < VB * K; idx += PT_) {
                const int r = idx / K, c = idx % K;
                ss_part += to_f32(Ss[r * LDK + c]) * to_f32(dSs[r * LDK + c]);
            }
        }
        // (1) dR = T^T dE, rows j = 16*rb.. ; (2) R0 = V - gamma . (K S^T), same rows
        {
            const int k0 = (rb * 16) / KS * KS;         // T[i][j] = 0 for i < j
            f32x4 dr[NVW], ks[NVW];             // the first product of each takes 0 as its addend
            {
                typename Mfma<T>::Frag ft = Mfma<T>::template load<false>(Tt + k0 * LDC + rb * 16, LDC, lane);
#pragma unroll
                for (int q = 0; q < NVW; ++q) {
                    const int vt = (wave % WPR) * NVW + q;
                    typename Mfma<T>::Frag fe = Mfma<T>::template load<true>(dEts + vt * 16 * LDE + k0, LDE, lane);
                    dr[q] = Mfma<T>::mma(fe, ft, f32x4{0.f, 0.f, 0.f, 0.f});
                }
            }
            for (int kk = k0 + KS; kk < C; kk += KS) {
                typename Mfma<T>::Frag ft = Mfma<T>::template load<false>(Tt + kk * LDC + rb * 16, LDC, lane);
#pragma unroll
                for (int q = 0; q < NVW; ++q) {
                    const int vt = (wave % WPR) * NVW + q;
                    typename Mfma<T>::Frag fe = Mfma<T>::template load<true>(dEts + vt * 16 * LDE + kk, LDE, lane);
                    dr[q] = Mfma<T>::mma(fe, ft, dr[q]);
                }
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int kk = 0; kk < K; kk += KS) {
                typename Mfma<T>::Frag fk = Mfma<T>::template load<true>(Ks + rb * 16 * LDK + kk, LDK, lane);
#pragma unroll
                for (int q = 0; q < NVW; ++q) {
                    const int vt = (wave % WPR) * NVW + q;
                    typename Mfma<T>::Frag fs = Mfma<T>::template load<true>(Ss + vt * 16 * LDK + kk, LDK, lane);
                    ks[q] = Mfma<T>::mma(fs, fk, kk == 0 ? f32x4{0.f, 0.f, 0.f, 0.f} : ks[q]);
                }
            }
#pragma unroll
            for (int q = 0; q < NVW; ++q) {
                const int vt = (wave % WPR) * NVW + q;
                const int i = rb * 16 + acc_col(lane), c = vt * 16 + acc_row(lane, 0);
                const f32x4 vv = load4(Vs + i * LDV + c);
                const float gam = Egs[i], bet = Bs[i];
                f32x4 dv;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    dbeta_part = __builtin_fmaf(dr[q][r], vv[r] - gam * ks[q][r], dbeta_part);
                    dv[r] = bet * dr[q][r];
                }
                store4(dRs + i * LDV + c, dr[q]);
                const uint32_t go = ((uint32_t)i * (uint32_t)(tstride * a.V) + (uint32_t)(v0 + c)) * (uint32_t)sizeof(T);
                if (i < rows) store4(reinterpret_cast<T *>(reinterpret_cast<char *>(static_cast<T *>(a.dv) + tok0 * a.V) + go), dv);
            }
        }
        __syncthreads();
        OSDN_BP_FRESH();
        // (3,4) dP += dO E^T, dA -= dR E^T on the lower tiles
#pragma unroll
        for (int t = 0; t < NLT; ++t) {
            const int idx = wave + PW_ * t;
            if (idx < 10) {
                const int ib = idx < 1 ? 0 : idx < 3 ? 1 : idx < 6 ? 2 : 3;
                const int jb = idx - (ib * (ib + 1)) / 2;
                for (int kk = 0; kk < VB; kk += KS) {
                    typename Mfma<T>::Frag fb = Mfma<T>::template load<false>(Ets + kk * LDE + jb * 16, LDE, lane);
                    typename Mfma<T>::Frag fo = Mfma<T>::template load<true>(dOs + ib * 16 * LDV + kk, LDV, lane);
                    typename Mfma<T>::Frag fr = Mfma<T>::template load<true>(dRs + ib * 16 * LDV + kk, LDV, lane);
                    dP[t] = Mfma<T>::mma(fb, fo, dP[t]);
                    dA[t] = Mfma<T>::mma(fb, fr, dA[t]);
                }
            }
        }
        // (5,6,7) dQg += dO S ; dKg += dR S ; dKr += E dS'   (column tile ct)
        if (has_ct) {
            for (int kk = 0; kk < VB; kk += KS) {
                typename Mfma<T>::Frag fs = Mfma<T>::template load<false>(Ss + kk * LDK + ct, LDK, lane);
                typename Mfma<T>::Frag fd = Mfma<T>::template load<false>(dSs + kk * LDK + ct, LDK, lane);
#pragma unroll
                for (int iq = 0; iq < IBN; ++iq) {
                    const int ib = ib0 + iq;
                    typename Mfma<T>::Frag fo = Mfma<T>::template load<true>(dOs + ib * 16 * LDV + kk, LDV, lane);
                    typename Mfma<T>::Frag fr = Mfma<T>::template load<true>(dRs + ib * 16 * LDV + kk, LDV, lane);
                    typename Mfma<T>::Frag fe = Mfma<T>::template load<false>(Ets + kk * LDE + ib * 16, LDE, lane);
                    dQg[iq] = Mfma<T>::mma(fs, fo, dQg[iq]);
                    dKg[iq] = Mfma<T>::mma(fs, fr, dKg[iq]);
                    dKr[iq] = Mfma<T>::mma(fd, fe, dKr[iq]);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
        }
    }
    __syncthreads();
    // ---- after the walk: Q, K~ into the pool ----
    r_S.put(Qs, LDK, tid);
    r_dS.put(Qs + VB * LDK, LDK, tid);
    {
        TileRegs<T, C, K, PT_> r_Kt;
#pragma unroll
        for (int m = 0; m < r_Kt.NV; ++m) r_Kt.v[m] = m < NVP ? r_dOV.vec(m) : r_EdE.vec(m - NVP);
        r_Kt.put(Kts, LDK, tid);
    }
    {                                                   // upper triangle of cA, cP is zero
        constexpr int VN = 16 / sizeof(T);
        for (int v = tid; v < C * C / VN; v += PT_) {
            const int i = v / (C / VN), j = (v % (C / VN)) * VN;
            *reinterpret_cast<u32x4 *>(cAs + i * LDC + j) = u32x4{0u, 0u, 0u, 0u};
            *reinterpret_cast<u32x4 *>(cPs + i * LDC + j) = u32x4{0u, 0u, 0u, 0u};
        }
    }
    if (GV) colss[GV ? tid : 0] = ss_part;               // thread tid summed rows of column tid % K
    ss_part = wave_sum(ss_part);
    if (lane == 0) sdot[wave] = ss_part;
    for (int idx = tid; idx < 4 * C; idx += PT_) {
        red[idx] = 0.f;
        if (!GV) { red2[idx] = 0.f; red3[idx] = 0.f; }
    }
    if (!GV)
        for (int idx = tid; idx < PW_ * C; idx += PT_) pq[idx] = 0.f;          // row-dot partials: a wavefront fills its own row blocks
    // dbeta: the walk's part, summed over the four lanes of a token; WPR wavefronts share a row block
    dbeta_part = add_xor32(add_xor16(dbeta_part));
    if (lane < 16) dbeta_s[(wave % WPR) * C + rb * 16 + lane] = dbeta_part;
    __syncthreads();
    OSDN_BP_FRESH();
    // ---- lower tiles: A0, P, X, cA, cP ----
#pragma unroll
    for (int t = 0; t < NLT; ++t) {
        const int idx = wave + PW_ * t;
        if (idx < 10) {
            const int ib = idx < 1 ? 0 : idx < 3 ? 1 : idx < 6 ? 2 : 3;
            const int jb = idx - (ib * (ib + 1)) / 2;
            const f32x4 kk = mma_tile0<T, true, true>(Kts + jb * 16 * LDK, LDK, Ks + ib * 16 * LDK, LDK, K, lane);
            __builtin_amdgcn_sched_barrier(0);
            const f32x4 qk = mma_tile0<T, true, true>(Kts + jb * 16 * LDK, LDK, Qs + ib * 16 * LDK, LDK, K, lane);
            f32x4 ca, cp, colx;
            const int i = ib * 16 + acc_col(lane), j0 = jb * 16 + acc_row(lane, 0);
            const float Gi = Gs[i], bi = Bs[i];
            const f32x4 Gj = *reinterpret_cast<const f32x4 *>(Gs + j0);
            float rs_a = 0.f, rs_x = 0.f;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int j = j0 + r;
                const float gam = (j <= i) ? __expf(Gi - Gj[r]) : 0.f;
                const float da = (j < i) ? -dA[t][r] : 0.f;             // dA_ij
                const float dp = (j <= i) ? a.scale * dP[t][r] : 0.f;   // dP_ij
                const float a0 = gam * kk[r];                            // A_ij / beta_i
                colx[r] = da * bi * a0 + dp * gam * qk[r];              // dA.A + dP.P
                ca[r] = da * bi * gam;
                cp[r] = dp * gam;
                rs_a = __builtin_fmaf(da, a0, rs_a);
                rs_x += colx[r];
            }
            rs_a = add_xor32(add_xor16(rs_a));
            if (lane < 16) red[jb * C + i] = rs_a;              // each (jb, i) is written by exactly one lane
            if (!GV) {
                rs_x = add_xor32(add_xor16(rs_x));
                if (lane < 16) red2[jb * C + i] = rs_x;
#pragma unroll
                for (int r = 0; r < 4; ++r) colx[r] = row16_sum(colx[r]);
                if (acc_col(lane) == 0) *reinterpret_cast<f32x4 *>(red3 + ib * C + j0) = colx;    // each (ib, j) written once
            }
            store_tile_t(cAs + ib * 16 * LDC + jb * 16, LDC, ca, lane);
            store_tile_t(cPs + ib * 16 * LDC + jb * 16, LDC, cp, lane);
        }
    }
    __syncthreads();
    OSDN_BP_FRESH();
    // ---- dQ, dK (read side), dK~ and the inner products that enter dG (column tile ct) ----
    // dG_i takes <d(gamma Q)_i, gamma_i Q_i> + <d(gamma K)_i, gamma_i K_i> - <d(rho K~)_i, rho_i K~_i>
    // as one number per row; the last term, summed over all rows, goes to the chunk's last token
    float trs = 0.f;                              // the last term over this lane's elements
    T *dq_g = static_cast<T *>(a.dq) + tok0 * K;
    T *dk_g = static_cast<T *>(a.dk_read) + bhn * C * K;
    T *dkt_g = static_cast<T *>(a.dkt) + bhn * C * K;
    f32x4 dgc = {0.f, 0.f, 0.f, 0.f}, gcv = {1.f, 1.f, 1.f, 1.f};
    if (GV && has_ct) gcv = *reinterpret_cast<const f32x4 *>(a.gamC + bhn * K + ct + acc_row(lane, 0));     // this lane's channels
    if (has_ct) {
#pragma unroll
        for (int iq = 0; iq < IBN; ++iq) {
            OSDN_BP_FRESH();
            __builtin_amdgcn_sched_barrier(0);
            const int ib = ib0 + iq;
            f32x4 aq, ak, at;                   // the first product of each takes 0 as its addend
            const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
            // cP K~ and cA K~: contraction over j <= i
            const int kd = min(C, ((ib + 1) * 16 + KS - 1) / KS * KS);
            for (int kk = 0; kk < kd; kk += KS) {
                typename Mfma<T>::Frag fk = Mfma<T>::template load<false>(Kts + kk * LDK + ct, LDK, lane);
                typename Mfma<T>::Frag fp = Mfma<T>::template load<true>(cPs + ib * 16 * LDC + kk, LDC, lane);
                typename Mfma<T>::Frag fa = Mfma<T>::template load<true>(cAs + ib * 16 * LDC + kk, LDC, lane);
                if (kk == 0) { aq = Mfma<T>::mma(fk, fp, zero); ak = Mfma<T>::mma(fk, fa, zero); }
                else { aq = Mfma<T>::mma(fk, fp, aq); ak = Mfma<T>::mma(fk, fa, ak); }
            }
            // cA^T K + cP^T Q: rows j = 16*ib.., contraction over i >= j
            const int k0 = (ib * 16) / KS * KS;
            {
                typename Mfma<T>::Frag fat = Mfma<T>::template load<false>(cAs + k0 * LDC + ib * 16, LDC, lane);
                typename Mfma<T>::Frag fpt = Mfma<T>::template load<false>(cPs + k0 * LDC + ib * 16, LDC, lane);
                typename Mfma<T>::Frag fkk = Mfma<T>::template load<false>(Ks + k0 * LDK + ct, LDK, lane);
                typename Mfma<T>::Frag fqq = Mfma<T>::template load<false>(Qs + k0 * LDK + ct, LDK, lane);
                at = Mfma<T>::mma(fkk, fat, zero);
                at = Mfma<T>::mma(fqq, fpt, at);
            }
            for (int kk = k0 + KS; kk < C; kk += KS) {
                typename Mfma<T>::Frag fat = Mfma<T>::template load<false>(cAs + kk * LDC + ib * 16, LDC, lane);
                typename Mfma<T>::Frag fpt = Mfma<T>::template load<false>(cPs + kk * LDC + ib * 16, LDC, lane);
                typename Mfma<T>::Frag fkk = Mfma<T>::template load<false>(Ks + kk * LDK + ct, LDK, lane);
                typename Mfma<T>::Frag fqq = Mfma<T>::template load<false>(Qs + kk * LDK + ct, LDK, lane);
                at = Mfma<T>::mma(fkk, fat, at);
                at = Mfma<T>::mma(fqq, fpt, at);
            }
            const int i = ib * 16 + acc_col(lane), c = ct + acc_row(lane, 0);
            const float gam = a.scale * Egs[i], bgam = -Bs[i] * Egs[i], rho = Ers[i];
            const f32x4 qv = load4(Qs + i * LDK + c), kv = load4(Ks + i * LDK + c), ktv = load4(Kts + i * LDK + c);
            float sc = 0.f;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const float gq = gam * dQg[iq][r];            // gamma . d(gamma Q)
                const float gk = bgam * dKg[iq][r];           // gamma . d(gamma K)
                const float gr = (GV ? gcv[r] : rho) * dKr[iq][r];      // rho . d(rho K~)
                if (GV) {
                    dgc[r] = __builtin_fmaf(ktv[r], gr, dgc[r]);
                } else {
                    sc += __builtin_fmaf(gq, qv[r], __builtin_fmaf(gk, kv[r], -(gr * ktv[r])));
                    trs = __builtin_fmaf(gr, ktv[r], trs);
                }
                aq[r] = __builtin_fmaf(gam, dQg[iq][r], aq[r]);
                ak[r] = __builtin_fmaf(bgam, dKg[iq][r], ak[r]);
                at[r] = __builtin_fmaf(GV ? gcv[r] : rho, dKr[iq][r], at[r]);
            }
            if (!GV) {              // over the four lanes of a token here, over the column tiles through LDS
                sc = add_xor32(add_xor16(sc));
                if (lane < 16) pq[wave * C + i] = sc;
            }
            const uint32_t go = ((uint32_t)i * (uint32_t)(tstride * K) + (uint32_t)c) * (uint32_t)sizeof(T);
            if (i < rows) store4(reinterpret_cast<T *>(reinterpret_cast<char *>(dq_g) + go), aq);
            const uint32_t gt = ((uint32_t)i * K + (uint32_t)c) * (uint32_t)sizeof(T);
            store4(reinterpret_cast<T *>(reinterpret_cast<char *>(dk_g) + gt), ak);
            store4(reinterpret_cast<T *>(reinterpret_cast<char *>(dkt_g) + gt), at);
        }
    }
    if (GV && has_ct) {                 // channel sums over the rows: the 16 lanes of a channel group
#pragma unroll
        for (int r = 0; r < 4; ++r) dgc[r] = row16_sum(dgc[r]);
        if (acc_col(lane) == 0) *reinterpret_cast<f32x4 *>(dgam_s + (GV ? (wave / NCT) * K + ct + acc_row(lane, 0) : 0)) = dgc;
    }
    trs = wave_sum(trs);
    if (lane == 0) trsum_s[wave] = trs;
    __syncthreads();
    if (GV && tid < K) {                // gamma_C . dL/d(decay of channel tid over the chunk)
        float sd = 0.f, ss = 0.f;
#pragma unroll
        for (int j = 0; j < WPC; ++j) sd += dgam_s[GV ? j * K + tid : 0];
#pragma unroll
        for (int j = 0; j < PT_ / K; ++j) ss += colss[GV ? tid + j * K : 0];
        a.dgamC[bhn * K + tid] = __builtin_fmaf(a.gamC[bhn * K + tid], ss, sd);
    }
    if (wave == 0) {
        const int i = lane;
        const float rowa = red[i] + red[C + i] + red[2 * C + i] + red[3 * C + i];
        const size_t th = tok0 + (size_t)i * tstride;
        float dbw = rowa;
#pragma unroll
        for (int w = 0; w < WPR; ++w) dbw += dbeta_s[w * C + i];
        if (i < rows) a.dbeta[th] = dbw;
        if (!GV && a.dlog_alpha) {
            float t_c = 0.f;
#pragma unroll
            for (int w = 0; w < PW_; ++w) t_c += pq[w * C + i];
            const float rowx = red2[i] + red2[C + i] + red2[2 * C + i] + red2[3 * C + i];
            const float colx = red3[i] + red3[C + i] + red3[2 * C + i] + red3[3 * C + i];
            float dG = rowx - colx + t_c;
            float ssum = 0.f, tr_sum = 0.f;
#pragma unroll
            for (int w = 0; w < PW_; ++w) { ssum += sdot[w]; tr_sum += trsum_s[w]; }
            if (i == C - 1) dG += tr_sum + __expf(Gs[C - 1]) * ssum;
            const float dg = wave_suffix_sum(dG, lane);
            if (i < rows) a.dlog_alpha[th] = dg;
        }
    }
}

// -------------------------------------------------------------- launchers ----
template <typename T, int K, bool GV, int VS>
static void launch_chain_t(const ChunkArgs &a, hipStream_t st) {
    ChunkArgs b = a;
    b.map = slice_map(a.V / VS, a.H * (long long)(a.seq_chunks ? a.n_seqs : a.B), VS == 16);
    dim3 grid(chain_workgroups(b.map)), block(CT_);
    with_rows(a.rows, [&](auto rag) { hipLaunchKernelGGL((bwd_chain_kernel<T, K, GV, VS, decltype(rag)::value>), grid, block, 0, st, b); });
}
// Slices of 16 values with fp32 I/O at K = 128 (beside slices of 32 one chunk's operands would fill the LDS, with nothing in
// flight for the next), else of 16 or 32 (narrow_backward in osdn_plan.h says which).
template <typename T, bool GV>
static int launch_chain_v(const ChunkArgs &a, hipStream_t st) {
    if ((GV && !a.gamC) || !a.Pm || !a.q || !a.dO) return -1;
    if (a.K != 64 && a.K != 128) return -1;
    if constexpr (sizeof(T) == 2) {
        if (a.narrow_slices) {
            if (a.K == 64) launch_chain_t<T, 64, GV, 16>(a, st);
            else launch_chain_t<T, 128, GV, 16>(a, st);
        } else {
            if (a.K == 64) launch_chain_t<T, 64, GV, 32>(a, st);
            else launch_chain_t<T, 128, GV, 32>(a, st);
        }
    } else {
        if (a.K == 128) launch_chain_t<T, 128, GV, 16>(a, st);
        else if (a.narrow_slices) launch_chain_t<T, 64, GV, 16>(a, st);
        else launch_chain_t<T, 64, GV, 32>(a, st);
    }
    return 0;
}
int launch_bwd_chain(const ChunkArgs &a, bool bf16_io, hipStream_t st) {
    if (a.gate_vec) return bf16_io ? launch_chain_v<bf16, true>(a, st) : launch_chain_v<float, true>(a, st);
    return bf16_io ? launch_chain_v<bf16, false>(a, st) : launch_chain_v<float, false>(a, st);
}
template <typename T, bool GV>
static int launch_post_t(const ChunkArgs &a, hipStream_t st) {
    constexpr int PW = 8;           // wavefronts per workgroup
    dim3 grid((a.n1 - a.n0) * a.H, a.B), block(PW * 64);
    if (GV && (!a.gamC || !a.dgamC || a.log_alpha || a.dlog_alpha)) return -1;
    if (a.K == 64) with_rows(a.rows, [&](auto rag) { hipLaunchKernelGGL((bwd_post_kernel<T, 64, GV, PW, decltype(rag)::value>), grid, block, 0, st, a); });
    else if (a.K == 128) with_rows(a.rows, [&](auto rag) { hipLaunchKernelGGL((bwd_post_kernel<T, 128, GV, PW, decltype(rag)::value>), grid, block, 0, st, a); });
    else return -1;
    return 0;
}
int launch_bwd_post(const ChunkArgs &a, bool bf16_io, hipStream_t st) {
    if (a.gate_vec) return bf16_io ? launch_post_t<bf16, true>(a, st) : launch_post_t<float, true>(a, st);
    return bf16_io ? launch_post_t<bf16, false>(a, st) : launch_post_t<float, false>(a, st);
}

// ---------------------------------------------------------------- unfold ----
// One state gate per key channel: phase 2 worked on Qg = Gamma . Q, Kg = Gamma . K and
// Kd = K~ / Gamma (Gamma = e^{G}, G the cumulative log-decay of every channel inside the
// chunk), and on gamma_C = Gamma's last row.  Per chunk this kernel rebuilds G and maps
//     dq = Gamma . dQg,   dk_read = Gamma . dKg,   dk~ = dKd / Gamma             (in place)
//     dG = dq . q + dk_read . k - dk~ . k~   (elementwise: G reaches the loss through the three
//          folded operands only),  dG[last token] += gamma_C . dgamma_C,
//     dlog_alpha = suffix sum of dG over the tokens of the chunk, channel by channel.
template <typename T, int K, bool RAG>
__global__ __launch_bounds__(NT) void unfold_kernel(UnfoldArgs a) {
    constexpr int GLD = K + 4, VN = 16 / sizeof(T);
    __shared__ __attribute__((aligned(16))) float Gt[C * GLD];     // G, then dG, then dlog_alpha
    const int n = a.n0 + blockIdx.x / a.H, h = blockIdx.x % a.H, b = blockIdx.y, tid = threadIdx.x;
    const size_t bhn = ((size_t)b * a.N + n) * a.H + h;
    const size_t tok0 = a.rows.first<RAG>(b, n) * a.H + h;
    const int rows = a.rows.count<RAG>(n);                               // (tokens that do not exist: gate 1, every gradient zero)
    const size_t rs = (size_t)a.H * K;                              // elements between consecutive tokens
    const float *gp = a.log_alpha + tok0 * K;
    for (int v = tid; v < C * K / 4; v += NT) {
        const int i = v / (K / 4), c = (v % (K / 4)) * 4;
        const f32x4 g4 = *reinterpret_cast<const f32x4 *>(gp + (size_t)min(i, rows - 1) * rs + c);
        *reinterpret_cast<f32x4 *>(Gt + i * GLD + c) = i < rows ? g4 : f32x4{0.f, 0.f, 0.f, 0.f};
    }
    __syncthreads();
    if (tid < K) {
        float G = 0.f;
#pragma unroll 16
        for (int i = 0; i < C; ++i) {
            G += Gt[i * GLD + tid];
            Gt[i * GLD + tid] = G;
        }
    }
    __syncthreads();
    const T *qp = static_cast<const T *>(a.q) + tok0 * K, *kp = static_cast<const T *>(a.k) + tok0 * K,
            *tp = static_cast<const T *>(a.kt) + bhn * C * K;
    T *dqp = static_cast<T *>(a.dq) + tok0 * K, *dkp = static_cast<T *>(a.dk_read) + bhn * C * K,
      *dtp = static_cast<T *>(a.dkt) + bhn * C * K;
    for (int v = tid; v < C * K / VN; v += NT) {
        const int i = v / (K / VN), c = (v % (K / VN)) * VN;
        if (i >= rows) {                                                // (dk~ and dk of the tile are not read there)
#pragma unroll
            for (int e = 0; e < VN; ++e) Gt[i * GLD + c + e] = 0.f;
            continue;
        }
        const size_t o = (size_t)i * rs + c, ot_ = i * K + c;            // caller's tensors, workspace tiles
        const u32x4 qv = *reinterpret_cast<const u32x4 *>(qp + o), kv = *reinterpret_cast<const u32x4 *>(kp + o),
                    tv = *reinterpret_cast<const u32x4 *>(tp + ot_);
        const u32x4 gq = *reinterpret_cast<const u32x4 *>(dqp + o), gk = *reinterpret_cast<const u32x4 *>(dkp + ot_),
                    gt = *reinterpret_cast<const u32x4 *>(dtp + ot_);
        float oq[VN], ok[VN], ot[VN];
#pragma unroll
        for (int e = 0; e < VN; ++e) {
            const float G = Gt[i * GLD + c + e];
            const float gam = __expf(G), inv = __expf(-G);
            oq[e] = vec_get<T>(gq, e) * gam;
            ok[e] = vec_get<T>(gk, e) * gam;
            ot[e] = vec_get<T>(gt, e) * inv;
            Gt[i * GLD + c + e] = oq[e] * vec_get<T>(qv, e) + ok[e] * vec_get<T>(kv, e) - ot[e] * vec_get<T>(tv, e);
        }
        store_vec_t(dqp + o, oq);
        store_vec_t(dkp + ot_, ok);
        store_vec_t(dtp + ot_, ot);
    }
    __syncthreads();
    if (tid < K) {
        float acc = a.dgamC[bhn * K + tid];
#pragma unroll 16
        for (int i = C - 1; i >= 0; --i) {
            acc += Gt[i * GLD + tid];
            Gt[i * GLD + tid] = acc;
        }
    }
    __syncthreads();
    float *dg = a.dlog_alpha + tok0 * K;
    for (int v = tid; v < C * K / 4; v += NT) {
        const int i = v / (K / 4), c = (v % (K / 4)) * 4;
        if (i < rows) *reinterpret_cast<f32x4 *>(dg + (size_t)i * rs + c) = *reinterpret_cast<const f32x4 *>(Gt + i * GLD + c);
    }
}

template <typename T>
static int launch_unfold_t(const UnfoldArgs &a, hipStream_t st) {
    dim3 grid((a.n1 - a.n0) * a.H, a.B), block(NT);
    if (a.K == 64) with_rows(a.rows, [&](auto rag) { hipLaunchKernelGGL((unfold_kernel<T, 64, decltype(rag)::value>), grid, block, 0, st, a); });
    else if (a.K == 128) with_rows(a.rows, [&](auto rag) { hipLaunchKernelGGL((unfold_kernel<T, 128, decltype(rag)::value>), grid, block, 0, st, a); });
    else return -1;
    return 0;
}
int launch_unfold(const UnfoldArgs &a, bool bf16_io, hipStream_t st) {
    if (!a.log_alpha || !a.q || !a.k || !a.kt || !a.dq || !a.dk_read || !a.dkt || !a.dgamC || !a.dlog_alpha)
        return -1;
    return bf16_io ? launch_unfold_t<bf16>(a, st) : launch_unfold_t<float>(a, st);
}

}  // namespace osdn
