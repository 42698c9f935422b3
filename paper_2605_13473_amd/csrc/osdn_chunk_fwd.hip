// Phase 2 forward of OSDN in chunkwise WY/UT form (Appendix A.2; gated, decay-ratio gauge
// of Appendix B.1), chunk length C = 64.  With G the in-chunk cumulative log-decay,
// gamma_i = e^{G_i}, rho_i = e^{G_C - G_i}, Gamma_ij = e^{G_i - G_j} (only j <= i is formed):
//
//   chunk_prep   (parallel over chunks):  A = tril(beta_i Gamma_ij <k_i, k~_j>, -1),
//                T = (I + A)^-1 in fp32,  W = T (beta gamma . K),  U = T (beta . V)
//   state_fwd    (sequential over chunks, parallel over (b, h, slice of V)):
//                E = U - W S^T ;  S <- gamma_C S + (rho . E)^T K~      (S fp32 in registers)
//   output_fwd   (parallel over chunks):  O = scale [ gamma . (Q S^T) + P E ],  P = tril(Gamma . Q K~^T)
//                (P is also written out when a backward pass follows)
//
// All contractions run on MFMA with fp32 accumulation; operands are staged in LDS in the
// I/O element type.
#include "osdn_kernels.h"
#include "osdn_tile.h"

namespace osdn {

// ------------------------------------------------------------ chunk_prep ----
// Leaves per chunk -W (natural layout), T diag(beta), the cumulative log-decay G, and T itself when
// a backward pass follows.  The row scalings of the right-hand sides move into T: W = (T diag(beta
// gamma)) K and U = (T diag(beta)) V; U is never stored: the state kernel adds (T diag(beta)) V to
// its product with the state, and scales E (not K~) for the write.  So V, U and a
// scaled copy of K~ stay out of this kernel's traffic.
//
// Bound by its phases' latency and memory: three workgroups share a CU (52 KB of LDS each at K =
// 128 in bf16: A, K~'s space reused for (I + A)^-1 and then for the outgoing W, the block products
// of the inverse in A's empty upper blocks).  4096 chunk-heads, K = V = 128 in bf16: 57 us and 269 MB;
// writing U^T and (rho K~)^T for the chain as well, two workgroups per CU: 104 us and 446 MB.
//
// GV: one state gate per key channel (the chunkwise UT form of online-scaled KDA, appendix
// section on Kimi Delta Attention with online scaling).  The cumulative channel decays
// Gamma [64 x K] do not factor out of the Gram matrix as a 64 x 64 mask, so they are folded
// into the operands: K <- Gamma . K and K~ <- K~ / Gamma in LDS before anything else, after
// which the kernel runs as with no gate at all; it also leaves Gamma . Q, K~ / Gamma, the chunk's
// total decay per channel gamma_C, and gamma_C . K~ / Gamma (from k~, rounded once) for the chain
// kernels.  1 / Gamma grows like e^{|G|}: the cumulative log-decay of a channel inside a chunk has
// to stay above about -80.
constexpr int CP_ = 512;        // threads of a chunk_prep workgroup (8 wavefronts)
template <typename T, int K, bool GV, bool RAG>
__global__ __launch_bounds__(CP_) void chunk_prep_kernel(ChunkArgs a) {
    constexpr int PAD = Pad<T>::v, LDK = K + PAD, LDC = C + PAD, LDF = C + 1;
    constexpr int NW = CP_ / 64, VN = 16 / sizeof(T);
    constexpr int X2_F = (C * LDK * (int)sizeof(T) / 4 > C * LDF ? C * LDK * (int)sizeof(T) / 4 : C * LDF + 3) & ~3;
    constexpr int TW_F = C * LDC * (int)sizeof(T) / 4, GLD = K + 4;
    constexpr int AF_F0 = C * LDF > TW_F ? C * LDF : TW_F;
    constexpr int AF_F = ((GV && C * GLD > AF_F0 ? C * GLD : AF_F0) + 3) & ~3;
    __shared__ __attribute__((aligned(16))) T X1[C * LDK];      // K
    __shared__ __attribute__((aligned(16))) float X2f[X2_F];    // K~, then (I + A)^-1 (fp32), then -W on its way out
    __shared__ __attribute__((aligned(16))) float Af[AF_F];     // (GV: the channel decays,) A (fp32), then T diag(beta gamma)
    T *X2 = reinterpret_cast<T *>(X2f);
    float *Ti = X2f;
    T *Tw = reinterpret_cast<T *>(Af);                          // [64][LDC], once A is dead
    __shared__ float Gs[C], Bs[C], BGs[C];

    const int n = a.n0 + blockIdx.x / a.H, h = blockIdx.x % a.H, b = blockIdx.y;
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const size_t tstride = a.H;                                           // tokens are H rows apart
    const size_t bhn = ((size_t)b * a.N + n) * a.H + h;
    const size_t tok0 = a.rows.first<RAG>(b, n) * a.H + h;                     // (b, first token, h)
    const int last = a.rows.count<RAG>(n) - 1;                                 // (rows of K behind it: their columns of T diag(beta) are zero)
    {
        TileRegs<T, C, K, CP_> r_K, r_Kt;
        float g = 0.f, bt = 0.f;
        r_K.fetch(static_cast<const T *>(a.k) + tok0 * K, tstride * K, tid, last);
        r_Kt.fetch(static_cast<const T *>(a.kt) + bhn * C * K, (size_t)K, tid);
        if (wave == 0) {
            const size_t th = tok0 + (size_t)min(lane, last) * tstride;
            if (!GV && a.log_alpha) g = lane <= last ? a.log_alpha[th] : 0.f;      // GV: the gates go into the operands
            bt = lane <= last ? a.beta[th] : 0.f;
            const float G = wave_cumsum(g, lane);
            Gs[lane] = G;
            Bs[lane] = bt;
            BGs[lane] = bt * __expf(G);
            if (!GV) {                          // the chunk's gates for everyone else: G, gamma = e^G, rho = e^(G_C - G)
                float *gr = a.gates + bhn * 3 * C;
                gr[lane] = G;
                gr[C + lane] = __expf(G);
                gr[2 * C + lane] = __expf(lane_bcast63(G) - G);
            }
        }
        r_K.put(X1, LDK, tid);
        r_Kt.put(X2, LDK, tid);
    }
    __syncthreads();
    if (GV) {
        // cumulative log-decay of every channel, G [64 x K] in fp32, in A's space: loaded with vector
        // reads, summed down the columns by one thread per channel, then K <- e^{G} K and K~ <- e^{-G}
        // K~ in LDS and Gamma . Q straight to memory, all threads on 16-byte vectors
        float *Gt = Af;
        const size_t rs = tstride * K;
        const float *gp = a.log_alpha + tok0 * K;
        for (int v = tid; v < C * K / 4; v += CP_) {
            const int i = v / (K / 4), c = (v % (K / 4)) * 4;
            const f32x4 g4 = *reinterpret_cast<const f32x4 *>(gp + (size_t)min(i, last) * rs + c);
            *reinterpret_cast<f32x4 *>(Gt + i * GLD + c) = i <= last ? g4 : f32x4{0.f, 0.f, 0.f, 0.f};
        }
        __syncthreads();
        if (tid < K) {
            float G = 0.f;
#pragma unroll 16
            for (int i = 0; i < C; ++i) {
                G += Gt[i * GLD + tid];
                Gt[i * GLD + tid] = G;
            }
            a.gamC[bhn * K + tid] = __expf(G);
        }
        __syncthreads();
        const T *qp = static_cast<const T *>(a.q) + tok0 * K;
        T *qg = static_cast<T *>(a.Qg) + bhn * C * K, *kw = static_cast<T *>(a.Kw) + bhn * C * K;
        for (int v = tid; v < C * K / VN; v += CP_) {
            const int i = v / (K / VN), c = (v % (K / VN)) * VN;
            const u32x4 kv = *reinterpret_cast<const u32x4 *>(X1 + i * LDK + c);
            const u32x4 tv = *reinterpret_cast<const u32x4 *>(X2 + i * LDK + c);
            u32x4 qv = *reinterpret_cast<const u32x4 *>(qp + (size_t)min(i, last) * rs + c);
            if (i > last) qv = u32x4{0u, 0u, 0u, 0u};
            float ko[VN], to[VN], qo[VN], wo[VN];
#pragma unroll
            for (int e = 0; e < VN; ++e) {
                const float G = Gt[i * GLD + c + e];
                wo[e] = vec_get<T>(tv, e) * __expf(Gt[(C - 1) * GLD + c + e] - G);
                const float gam = __expf(G), inv = __expf(-G);
                ko[e] = vec_get<T>(kv, e) * gam;
                to[e] = vec_get<T>(tv, e) * inv;
                qo[e] = vec_get<T>(qv, e) * gam;
            }
            store_vec_t(X1 + i * LDK + c, ko);
            store_vec_t(X2 + i * LDK + c, to);
            store_vec_t(qg + i * K + c, qo);
            store_vec_t(kw + i * K + c, wo);
        }
        __syncthreads();            // (the decays' space is handed over to A)
        store_tile_global(static_cast<T *>(a.Kg) + bhn * C * K, (size_t)K, X1, LDK, C, K, tid, CP_);
        store_tile_global(static_cast<T *>(a.Kd) + bhn * C * K, (size_t)K, X2, LDK, C, K, tid, CP_);
    }

    // ---- A = tril(beta_i Gamma_ij <k_i, k~_j>, -1): the ten lower 16x16 tiles ----
    for (int idx = wave; idx < 10; idx += NW) {
        const int ib = idx < 1 ? 0 : idx < 3 ? 1 : idx < 6 ? 2 : 3;
        const int jb = idx - (ib * (ib + 1)) / 2;
        const f32x4 acc = mma_tile0<T, true, true>(X1 + ib * 16 * LDK, LDK, X2 + jb * 16 * LDK, LDK, K, lane);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int i = ib * 16 + acc_row(lane, r), j = jb * 16 + acc_col(lane);
            Af[i * LDF + j] = (j < i) ? Bs[i] * __expf(Gs[i] - Gs[j]) * acc[r] : 0.f;
        }
    }
    __syncthreads();                // A is complete, K~ is dead: (I + A)^-1 is built in its place
    // ---- T = (I + A)^-1 in fp32, blocked ----
    ut_inverse64<LDF, LDF>(Af, Ti, Af + 16, 16, wave, lane);
    // ---- T in the I/O type, up to three times: as it is (for a backward pass), with the columns scaled
    //      by beta (for E) and by beta gamma (for W); the upper triangle is exactly zero ----
    {
        T *tg = a.Tm ? static_cast<T *>(a.Tm) + bhn * C * C : nullptr;
        T *ug = static_cast<T *>(a.Tu) + bhn * C * C;
        for (int v = tid; v < C * C / VN; v += CP_) {
            const int i = v / (C / VN), j0 = (v % (C / VN)) * VN;
            float plain[VN], tu[VN], tw[VN];
#pragma unroll
            for (int e = 0; e < VN; ++e) {
                const int j = j0 + e;
                const float t = j <= i ? Ti[i * LDF + j] : 0.f;
                plain[e] = t;
                tu[e] = t * Bs[j];
                tw[e] = t * BGs[j];
            }
            if (tg) store_vec_t(tg + i * C + j0, plain);
            store_vec_t(ug + i * C + j0, tu);
            store_vec_t(Tw + i * LDC + j0, tw);
        }
    }
    __syncthreads();                // (I + A)^-1 is dead from here on: its space is the staging tile
    // ---- -W = -(T diag(beta gamma)) K ----
    for (int t = wave; t < (K / 16) * 4; t += NW) {
        const int nb = t >> 2, ib = t & 3;
        const int kdim = min(C, ((ib + 1) * 16 + Mfma<T>::KSTEP - 1) / Mfma<T>::KSTEP * Mfma<T>::KSTEP);
        f32x4 acc = mma_tile0<T, false, true>(X1 + nb * 16, LDK, Tw + ib * 16 * LDC, LDC, kdim, lane);
#pragma unroll
        for (int r = 0; r < 4; ++r) acc[r] = -acc[r];
        store_tile_t(X2 + ib * 16 * LDK + nb * 16, LDK, acc, lane);       // rows = tokens
    }
    __syncthreads();
    store_tile_global(static_cast<T *>(a.Wn) + bhn * C * K, (size_t)K, X2, LDK, C, K, tid, CP_);
}

// ------------------------------------------------------------- state_fwd ----
// Sequential over the chunks of one (batch, head), one workgroup per slice of VS rows of S.  Eight
// wavefronts carry the chain  S_n -> E_n -> S_{n+1}  (two barriers per chunk):
//   A  S, rounded to the I/O type, into LDS                                   | barrier 1
//   B  E = (T diag(beta)) V - W S^T, one 16x16 tile per wavefront; E and rho E (the operand of the
//      write) into LDS                                                        | barrier 2
//   C  S <- gamma_C S + (rho E)^T K~ in the MFMA accumulators (fp32)
// With bf16 I/O everything a phase needs besides S or E is in registers when its barrier opens: the
// fragments of -W and the product with V are prepared in phase C of the chunk before, those of K~ in phase
// B.  (fp32 fragments would not fit the registers: there the product with V alone, at K = 64.)
// Four more wavefronts move data.  Two load, directly from global memory into three LDS rings
// (osdn_tile.h): -W; X, what the product with V takes (T diag(beta), the slice of V) and the gates; what
// phase C multiplies (K~; per-channel gates: the chunk's decays).  Two store the checkpoint of S and E^T.  They are
// wavefronts of their own because a memory instruction stalls its wavefront until the CU's address
// unit takes it (64 bytes per clock: 700 cycles for a chunk's tiles), which adds to the chain when the
// same wavefronts do both, and because a wavefront's accesses retire in order: a load issued behind a
// store is only known to be there when the store is acknowledged, about 1 us later.
// Bound by what a CU has in flight from HBM (46 KB in and 12 KB out per chunk with slices of 32): 64
// chains of 64 chunks, V = 128: 115 us, 3.8 TB/s; without the stores 73 us, without any traffic 52 us.
// With fp32 I/O bound by what the slices of a chain read over again (84 KB in per chunk at K = 128 with
// slices of 16, 88 with 32): many chains take slices of 32 there too, although -W alone then has a second
// slot.  256 chains of 16 chunks: K = V = 128 412 -> 314 us (the product with V a phase ahead, X and K~ both in
// flight during phase B alone: 390; one slot for -W too: 447), V = 256 799 -> 604, K = 64, V = 128 316 -> 222.
constexpr int CW_ = 8;          // wavefronts of a chain workgroup that compute
constexpr int CM_ = 2;          // ... that load
constexpr int CS_ = 2;          // ... that store
constexpr int CT_ = (CW_ + CM_ + CS_) * 64;
// Ring depths (chunks of operands in LDS) of -W, of T diag(beta), V and the gates, and of K~, from what fits.
template <typename T, int K, int VS> constexpr int SF_NSW = sizeof(T) == 2 ? 3 : 2;
template <typename T, int K, int VS> constexpr int SF_NSX = sizeof(T) == 2 ? 3 : (K == 64 || VS == 16 ? 2 : 1);
template <typename T, int K, int VS> constexpr int SF_NSC = sizeof(T) == 2 || K == 64 ? 2 : 1;

// GV: one state gate per key channel: the operands carry the decays inside the chunk, and every
// coordinate of the state its own gamma_C; K~ is gamma_C . K~ / Gamma.
// VS: rows of S (values) owned by one workgroup, 32 or 16.  With few chains the narrow slice
// gives twice the workgroups, each with half the work on the dependent path per chunk.
template <typename T, int K, bool GV, int VS, bool RAG>
__global__ __launch_bounds__(CT_) void state_fwd_kernel(ChunkArgs a) {
    constexpr int ES = sizeof(T), RK = K * ES, RC = C * ES, RV = VS * ES;      // bytes per row of a tile
    constexpr int NVT = VS / 16, NFB = K / 16;
    constexpr int NTC = NFB * NVT, TPW = NTC > CW_ ? NTC / CW_ : 1;            // state tiles, ... per wavefront
    constexpr int KS = Mfma<T>::KSTEP, NKK = K / KS, NKC = C / KS;
    typedef typename Mfma<T>::Frag Frag;
    constexpr bool PRE = sizeof(T) == 2;        // operands in registers ahead of their phase (fp32: they would not fit)
    constexpr int NSW = SF_NSW<T, K, VS>, NSX = SF_NSX<T, K, VS>, NSC = SF_NSC<T, K, VS>;
    constexpr bool AHEAD = NSC > 1;             // the product with V one phase ahead (else phase B has to cover the loads of K~)
    static_assert(!PRE || (AHEAD && NSW == NSX), "what phase B multiplies comes at once");
    constexpr int X_T = 0, X_V = X_T + C * RC, X_G = X_V + C * RV, X_BYTES = X_G + 2 * C * 4;
    constexpr int C_K = 0, C_D = C_K + C * RK, C_BYTES = C_D + (GV ? K * 4 : 0);
    __shared__ __attribute__((aligned(1024))) char ringW[NSW * C * RK];
    __shared__ __attribute__((aligned(1024))) char ringX[NSX * X_BYTES];
    __shared__ __attribute__((aligned(1024))) char ringC[NSC * C_BYTES];
    __shared__ __attribute__((aligned(1024))) char Sb[VS * RK];         // S in the I/O type [v][kf]
    __shared__ __attribute__((aligned(1024))) char Eo[VS * RC];         // E^T  [v][i]
    __shared__ __attribute__((aligned(1024))) char Ew[GV ? 16 : VS * RC];   // (rho E)^T

    int chain, slice;
    chain_slice_of(blockIdx.x, a.V / VS, (a.seq_chunks ? a.n_seqs : a.B) * a.H, chain, slice);
    const int vs = slice * VS, h = chain % a.H, b = chain / a.H;   // b: batch entry, or packed sequence
    int bt = b;                                 // batch entry of the token tensors
    if (a.seq_chunks) {
        bool begins, ends;
        if (!clip_to_sequence(a.seq_chunks, b, a.n0, a.n1, begins, ends)) return;
        a.S_in = begins ? a.S_first : a.S_out;
        bt = 0;
    }
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const bool loader = wave >= CW_ && wave < CW_ + CM_, storer = wave >= CW_ + CM_;
    const int mw = wave - CW_, mt = tid - (CW_ + CM_) * 64;     // loader wavefront, storer thread
    const size_t bh = (size_t)b * a.H + h;      // the chain: indexes S_in / S_out
    const uint32_t gV = (uint32_t)a.H * (uint32_t)a.V * ES;        // bytes between tokens of v
    const ChainRows<RAG> rows(a.rows, a.seq_chunks, b, a.n0);
    const bool wideV = (reinterpret_cast<uintptr_t>(a.v) & 15) == 0;

    LdsLoad<RK, C, CM_> lK;
    LdsLoad<RC, C, CM_> lT;
    LdsLoad<RV, C, CM_> lV;
    lK.init(RK, mw, lane); lT.init(RC, mw, lane); lV.init(gV, mw, lane);
    auto loadW = [&](int n, int slot) {
        lK.issue(ringW + slot * C * RK, static_cast<const char *>(a.Wn) + (((size_t)bt * a.N + n) * a.H + h) * C * RK, RK, mw, lane, slice);
    };
    auto loadX = [&](int n, int slot) {
        const size_t bhn = ((size_t)bt * a.N + n) * a.H + h;
        char *s = ringX + slot * X_BYTES;
        lT.issue(s + X_T, static_cast<const char *>(a.Tu) + bhn * C * RC, RC, mw, lane, slice);
        lV.issue(s + X_V, static_cast<const char *>(a.v) + (rows.first(n) * a.H + h) * a.V * ES + (size_t)vs * ES,
                 gV, mw, lane, 0, wideV, rows.count(n) - 1);      // (rows behind the last: their columns of T diag(beta) are zero)
        if (!GV && mw < 2) {                    // gamma (loader 0) and rho (1)
            const int w = mw;
            load_lds4(a.gates + (bhn * 3 + 1 + w) * C, lane * 4, lds_offset(s + X_G + w * C * 4));
        }
    };
    auto loadC = [&](int n, int slot) {
        char *s = ringC + slot * C_BYTES;
        lK.issue(s + C_K, static_cast<const char *>(a.kt) + (((size_t)bt * a.N + n) * a.H + h) * C * RK, RK, mw, lane, slice);
        if (GV && mw < K / 64) load_lds4(a.gamC + (((size_t)bt * a.N + n) * a.H + h) * K, mw * 256 + lane * 4, lds_offset(s + C_D + mw * 256));
    };
    // Loads of a loader that are newer than the tiles it waits for (at least).  A chunk asks behind barrier 1
    // for -W and X (PRE), for K~ and X (AHEAD), or for K~, and behind barrier 2 for the others in this order.
    constexpr int LW = LdsLoad<RK, C, CM_>::MIN, LX = LdsLoad<RC, C, CM_>::MIN + LdsLoad<RV, C, CM_>::MIN, LC = LW, LA = LW + LX + LC;
    constexpr int NMAX = NSW > NSX ? (NSW > NSC ? NSW : NSC) : (NSX > NSC ? NSX : NSC);
    constexpr int NEWER_W = (NSW - 1) * LA + (AHEAD ? 0 : LX), NEWER_X = (NSX - 1) * LA, NEWER_C = (NSC - 1) * LA + (AHEAD && !PRE ? LX : 0);
    constexpr int NEWER_1 = PRE ? NEWER_C : AHEAD || NEWER_W < NEWER_X ? NEWER_W : NEWER_X;
    constexpr int NEWER_2 = PRE ? NEWER_X : !AHEAD || NEWER_C < NEWER_X ? NEWER_C : NEWER_X;
    static_assert(NEWER_1 < 64 && NEWER_2 < 64, "the counter has six bits");
#pragma unroll
    for (int j = 0; j < NMAX; ++j) {
        if (loader && j < NSW && a.n0 + j < a.n1) loadW(a.n0 + j, j);
        if (loader && j < NSX && a.n0 + j < a.n1) loadX(a.n0 + j, j);
        if (loader && j < (PRE ? NSC : NSC - 1) && a.n0 + j < a.n1) loadC(a.n0 + j, j);
    }

    // ---- state slice, transposed: St[q] rows = features, cols = values ----
    // this wavefront's tiles of S (feature block fb, value blocks vtC ..) and of E (row block rb, value block vtB)
    const bool inC = wave * TPW < NTC, inB = wave < 4 * NVT;
    const int fb = wave % NFB, vtC = wave / NFB;
    const int rb = wave & 3, vtB = wave >> 2;
    f32x4 St[TPW] = {};
    if (inC) {
#pragma unroll
        for (int q = 0; q < TPW; ++q) {
            const int v = vs + (vtC + q) * 16 + acc_col(lane), c0 = fb * 16 + acc_row(lane, 0);
            if (a.S_in) St[q] = *reinterpret_cast<const f32x4 *>(a.S_in + (bh * a.V + v) * K + c0);
        }
    }
    if (loader) wait_vm<0>();
    __syncthreads();
    int sw = 0, sx = 0, sc = 0;                 // ring slots of chunk n
    auto next = [](int slot, int depth) { return slot + 1 == depth ? 0 : slot + 1; };
    if (loader) {
        // (all is there; said to the compiler too, which does not count wait_vm: it would wait for the state's loads where
        // their registers are used again in the loop, and with them for every tile on its way: 122 -> 142 us)
        __builtin_amdgcn_s_waitcnt(0x0f70);     // vmcnt(0)
        for (int n = a.n0; n < a.n1; ++n) {
            const bool full = n + NMAX < a.n1;  // everything counted as newer has been asked for
            // a slot is refilled as soon as its operands have been read: ahead of their phase (X; PRE: all), or in it
            if (full) wait_vm<NEWER_1>(); else wait_vm<0>();        // K~ (PRE), -W, X (not AHEAD)
            __syncthreads();                                        // barrier 1
            if (PRE && n + NSW < a.n1) loadW(n + NSW, sw);
            if (!PRE && n - 1 + NSC < a.n1) loadC(n - 1 + NSC, sc == 0 ? NSC - 1 : sc - 1);
            if (AHEAD && n + NSX < a.n1) loadX(n + NSX, sx);
            if (full) wait_vm<NEWER_2>(); else wait_vm<0>();        // -W and X of the next chunk (PRE), X of the next chunk (AHEAD) and K~
            __syncthreads();                                        // barrier 2
            if (PRE && n + NSC < a.n1) loadC(n + NSC, sc);
            if (!PRE && n + NSW < a.n1) loadW(n + NSW, sw);
            if (!AHEAD && n + NSX < a.n1) loadX(n + NSX, sx);
            sw = next(sw, NSW); sx = next(sx, NSX); sc = next(sc, NSC);
        }
        return;
    }
    if (storer) {
        for (int n = a.n0; n < a.n1; ++n) {
            const size_t bhn = ((size_t)bt * a.N + n) * a.H + h;
            __syncthreads();                                        // barrier 1
            tile_to_global<RK, VS>(static_cast<char *>(a.S_ckpt) + (bhn * a.V + vs) * RK, RK, Sb, mt, CS_ * 64);
            __syncthreads();                                        // barrier 2
            tile_to_global<RC, VS>(static_cast<char *>(a.Et) + (bhn * a.V + vs) * RC, RC, Eo, mt, CS_ * 64);
        }
        return;
    }
    TileFrag<T, RK> fK;
    TileFrag<T, RC> fT;
    TileFrag<T, RV> fV;
    fK.init(lane); fT.init(lane); fV.init(lane);
    // operands of phase B of one chunk: fragments of -W (PRE), the product with V, rho of this lane's rows, gamma_C
    Frag wf[NKK];
    f32x4 uacc = {}, rho = {1.f, 1.f, 1.f, 1.f};
    float gC = 1.f;
    auto fetchB = [&](const char *tW, const char *tX) {
        if (inB) {
            if (PRE) {
#pragma unroll
                for (int kk = 0; kk < NKK; ++kk) wf[kk] = fK.kc(tW, rb * 16, kk * KS);
            }
            uacc = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int kk = 0; kk < NKC; ++kk)
                if (kk * KS < (rb + 1) * 16)                    // T is lower triangular
                    uacc = Mfma<T>::mma(fT.kc(tX + X_T, rb * 16, kk * KS), fV.tr(tX + X_V, kk * KS, vtB * 16), uacc);
            if (!GV) rho = *reinterpret_cast<const f32x4 *>(tX + X_G + (rb * 16 + acc_row(lane, 0)) * 4 + C * 4);
        }
        if (!GV) gC = *reinterpret_cast<const float *>(tX + X_G + (C - 1) * 4);
    };
    if (AHEAD) fetchB(ringW, ringX);
    for (int n = a.n0; n < a.n1; ++n) {
        const char *tW = ringW + sw * C * RK, *tC = ringC + sc * C_BYTES;
        // ---- phase A ----
        if (inC) {
#pragma unroll
            for (int q = 0; q < TPW; ++q) fK.put(Sb, (vtC + q) * 16, fb * 16, St[q]);
        }
        __syncthreads();                                            // barrier 1
        // ---- phase B ----
        Frag sf[NKK], kf[NKC];
        f32x4 dc = {};
        if (!AHEAD) fetchB(tW, ringX + sx * X_BYTES);
        if (inB) {
#pragma unroll
            for (int kk = 0; kk < NKK; ++kk) sf[kk] = fK.kc(Sb, vtB * 16, kk * KS);
        }
        if (PRE && inC) {
#pragma unroll
            for (int kk = 0; kk < NKC; ++kk) kf[kk] = fK.tr(tC + C_K, kk * KS, fb * 16);
            if (GV) dc = *reinterpret_cast<const f32x4 *>(tC + C_D + (fb * 16 + acc_row(lane, 0)) * 4);
        }
        if (inB) {
            f32x4 acc = {0.f, 0.f, 0.f, 0.f}, acc2 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int kk = 0; kk < NKK; kk += 2) {
                acc = Mfma<T>::mma(PRE ? wf[kk] : fK.kc(tW, rb * 16, kk * KS), sf[kk], acc);
                acc2 = Mfma<T>::mma(PRE ? wf[kk + 1] : fK.kc(tW, rb * 16, (kk + 1) * KS), sf[kk + 1], acc2);
            }
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[r] = uacc[r] + (acc[r] + acc2[r]);     // (last: begun with U, every step would round at its size)
            if (!GV) {
                f32x4 ew;
#pragma unroll
                for (int r = 0; r < 4; ++r) ew[r] = acc[r] * rho[r];
                fT.put(Ew, vtB * 16, rb * 16, ew);
            }
            fT.put(Eo, vtB * 16, rb * 16, acc);
        }
        const float g = gC;
        __syncthreads();                                            // barrier 2
        // ---- phase C ----
        if (inC) {
            Frag fe[TPW][NKC];
            if (!PRE && GV) dc = *reinterpret_cast<const f32x4 *>(tC + C_D + (fb * 16 + acc_row(lane, 0)) * 4);
#pragma unroll
            for (int q = 0; q < TPW; ++q)
#pragma unroll
                for (int kk = 0; kk < NKC; ++kk) fe[q][kk] = fT.kc(GV ? Eo : Ew, (vtC + q) * 16, kk * KS);
#pragma unroll
            for (int q = 0; q < TPW; ++q) {
#pragma unroll
                for (int r = 0; r < 4; ++r) St[q][r] *= GV ? dc[r] : g;
#pragma unroll
                for (int kk = 0; kk < NKC; ++kk) St[q] = Mfma<T>::mma(PRE ? kf[kk] : fK.tr(tC + C_K, kk * KS, fb * 16), fe[q][kk], St[q]);
            }
        }
        sw = next(sw, NSW); sx = next(sx, NSX); sc = next(sc, NSC);
        if (AHEAD && n + 1 < a.n1) fetchB(ringW + sw * C * RK, ringX + sx * X_BYTES);
    }
    if (inC) {
#pragma unroll
        for (int q = 0; q < TPW; ++q) {
            const int v = vs + (vtC + q) * 16 + acc_col(lane), c0 = fb * 16 + acc_row(lane, 0);
            *reinterpret_cast<f32x4 *>(a.S_out + (bh * a.V + v) * K + c0) = St[q];
        }
    }
}

// ------------------------------------------------------------ output_fwd ----
constexpr int OT_ = 512;        // threads of an output_fwd workgroup: 8 wavefronts, (row block, half of the value tiles)
template <typename T, int K, bool RAG>
__global__ __launch_bounds__(OT_) void output_fwd_kernel(ChunkArgs a) {
    constexpr int PAD = sizeof(T) == 2 ? 16 : Pad<T>::v, LDK = K + PAD, LDC = C + PAD;   // bf16: rows 32 bytes apart modulo 128 (every operand read here is 16 bytes per lane along k)
    constexpr int NW = OT_ / 64;
    __shared__ __attribute__((aligned(16))) T Qs[C * LDK];
    __shared__ __attribute__((aligned(16))) T Kts[C * LDK];     // K~, later the output staging tile
    __shared__ __attribute__((aligned(16))) T Ss[C * LDK];      // 64 rows of the chunk-start state
    __shared__ __attribute__((aligned(16))) T Ps[C * LDC];      // tril(Gamma . Q K~^T)
    __shared__ __attribute__((aligned(16))) T Ets[C * LDC];     // 64 rows of E^T
    __shared__ float Gs[C];

    const int n = a.n0 + blockIdx.x / a.H, h = blockIdx.x % a.H, b = blockIdx.y;
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const size_t bhn = ((size_t)b * a.N + n) * a.H + h;
    const size_t tok0 = a.rows.first<RAG>(b, n) * a.H + h;
    const int rows = a.rows.count<RAG>(n);
    const size_t tstride = a.H;

    if (wave == 0) {
        Gs[lane] = a.log_alpha ? a.gates[bhn * 3 * C + lane] : 0.f;
    }
    load_tile(Qs, LDK, static_cast<const T *>(a.q) + (a.gate_vec ? bhn * C : tok0) * K, a.gate_vec ? (size_t)K : tstride * K, C, K, tid, OT_,
              a.gate_vec ? C - 1 : rows - 1);
    load_tile(Kts, LDK, static_cast<const T *>(a.kt) + bhn * C * K, (size_t)K, C, K, tid, OT_);
    // the slabs of S and E^T travel through registers, one slab ahead of the products
    TileRegs<T, C, K, OT_> r_S;
    TileRegs<T, C, C, OT_> r_E;
    r_S.fetch(static_cast<const T *>(a.S_ckpt) + bhn * a.V * K, (size_t)K, tid);
    r_E.fetch(static_cast<const T *>(a.Et) + bhn * a.V * C, (size_t)C, tid);
    __syncthreads();
    // P^T tiles (rows j, columns i) so that the store lands k-contiguous in Ps[i][j]
    for (int idx = wave; idx < 16; idx += NW) {
        const int ib = idx >> 2, jb = idx & 3;
        f32x4 acc = {0.f, 0.f, 0.f, 0.f};
        if (jb <= ib) {
            mma_tile<T, true, true>(acc, Kts + jb * 16 * LDK, LDK, Qs + ib * 16 * LDK, LDK, K, lane);
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int j = jb * 16 + acc_row(lane, r), i = ib * 16 + acc_col(lane);
                acc[r] = (j <= i) ? __expf(Gs[i] - Gs[j]) * acc[r] : 0.f;
            }
        }
        store_tile_t(Ps + ib * 16 * LDC + jb * 16, LDC, acc, lane);
    }
    T *Os = Kts;
    for (int v0 = 0; v0 < a.V; v0 += C) {
        __syncthreads();
        // P is kept for the backward pass (its chain kernel forms scale P^T dO from it)
        if (v0 == 0 && a.Pm) store_tile_global(static_cast<T *>(a.Pm) + bhn * C * C, (size_t)C, Ps, LDC, C, C, tid, OT_);
        r_S.put(Ss, LDK, tid);
        r_E.put(Ets, LDC, tid);
        if (v0 + C < a.V) {
            r_S.fetch(static_cast<const T *>(a.S_ckpt) + (bhn * a.V + v0 + C) * K, (size_t)K, tid);
            r_E.fetch(static_cast<const T *>(a.Et) + (bhn * a.V + v0 + C) * C, (size_t)C, tid);
        }
        __syncthreads();
        const int rb = wave & 3;                    // row block of this wavefront; the other bit: which value tiles
        const int kdim = min(C, ((rb + 1) * 16 + Mfma<T>::KSTEP - 1) / Mfma<T>::KSTEP * Mfma<T>::KSTEP);
#pragma unroll
        for (int vq = 0; vq < 4 / (NW / 4); ++vq) {
            const int vt = (wave >> 2) * (4 / (NW / 4)) + vq;
            f32x4 a1 = {0.f, 0.f, 0.f, 0.f}, a2 = {0.f, 0.f, 0.f, 0.f};
            mma_tile<T, true, true>(a1, Qs + rb * 16 * LDK, LDK, Ss + vt * 16 * LDK, LDK, K, lane);
            mma_tile<T, true, true>(a2, Ps + rb * 16 * LDC, LDC, Ets + vt * 16 * LDC, LDC, kdim, lane);
#pragma unroll
            for (int r = 0; r < 4; ++r)
                a1[r] = a.scale * (__expf(Gs[rb * 16 + acc_row(lane, r)]) * a1[r] + a2[r]);
            store_tile(Os + rb * 16 * LDC + vt * 16, LDC, a1, lane);
        }
        __syncthreads();
        T *og = static_cast<T *>(a.o) + tok0 * a.V + v0;
        if (rows == C) store_tile_global(og, tstride * a.V, Os, LDC, C, C, tid, OT_);      // (a constant count: unrolled)
        else store_tile_global(og, tstride * a.V, Os, LDC, rows, C, tid, OT_);
    }
}

// -------------------------------------------------------------- launchers ----
template <typename T, bool GV>
static int launch_prep_t(const ChunkArgs &a, hipStream_t st) {
    dim3 grid((a.n1 - a.n0) * a.H, a.B), block(CP_);
    if (GV && (!a.log_alpha || !a.Qg || !a.Kg || !a.Kd || !a.Kw || !a.gamC)) return -1;
    if (a.K == 64) with_rows(a.rows, [&](auto rag) { hipLaunchKernelGGL((chunk_prep_kernel<T, 64, GV, decltype(rag)::value>), grid, block, 0, st, a); });
    else if (a.K == 128) with_rows(a.rows, [&](auto rag) { hipLaunchKernelGGL((chunk_prep_kernel<T, 128, GV, decltype(rag)::value>), grid, block, 0, st, a); });
    else return -1;
    return 0;
}
int launch_chunk_prep(const ChunkArgs &a, bool bf16_io, hipStream_t st) {
    if (a.gate_vec) return bf16_io ? launch_prep_t<bf16, true>(a, st) : launch_prep_t<float, true>(a, st);
    return bf16_io ? launch_prep_t<bf16, false>(a, st) : launch_prep_t<float, false>(a, st);
}
template <typename T, bool GV, int VS>
static int launch_state_t(const ChunkArgs &a, hipStream_t st) {
    dim3 grid((a.V / VS) * a.H * (a.seq_chunks ? a.n_seqs : a.B)), block(CT_);
    if (GV && !a.gamC) return -1;
    if (a.K == 64) with_rows(a.rows, [&](auto rag) { hipLaunchKernelGGL((state_fwd_kernel<T, 64, GV, VS, decltype(rag)::value>), grid, block, 0, st, a); });
    else if (a.K == 128) with_rows(a.rows, [&](auto rag) { hipLaunchKernelGGL((state_fwd_kernel<T, 128, GV, VS, decltype(rag)::value>), grid, block, 0, st, a); });
    else return -1;
    return 0;
}
// Slices of 16 values when the caller asks for them (few chains: see osdn_fwd), else of 32.
template <typename T, bool GV>
static int launch_state_v(const ChunkArgs &a, hipStream_t st) {
    return a.narrow_slices ? launch_state_t<T, GV, 16>(a, st) : launch_state_t<T, GV, 32>(a, st);
}
int launch_state_fwd(const ChunkArgs &a, bool bf16_io, hipStream_t st) {
    if (a.gate_vec) return bf16_io ? launch_state_v<bf16, true>(a, st) : launch_state_v<float, true>(a, st);
    return bf16_io ? launch_state_v<bf16, false>(a, st) : launch_state_v<float, false>(a, st);
}
template <typename T>
static int launch_output_t(const ChunkArgs &a, hipStream_t st) {
    dim3 grid((a.n1 - a.n0) * a.H, a.B), block(OT_);
    if (a.K == 64) with_rows(a.rows, [&](auto rag) { hipLaunchKernelGGL((output_fwd_kernel<T, 64, decltype(rag)::value>), grid, block, 0, st, a); });
    else if (a.K == 128) with_rows(a.rows, [&](auto rag) { hipLaunchKernelGGL((output_fwd_kernel<T, 128, decltype(rag)::value>), grid, block, 0, st, a); });
    else return -1;
    return 0;
}
int launch_output_fwd(const ChunkArgs &a, bool bf16_io, hipStream_t st) {
    return bf16_io ? launch_output_t<bf16>(a, st) : launch_output_t<float>(a, st);
}

}  // namespace osdn
