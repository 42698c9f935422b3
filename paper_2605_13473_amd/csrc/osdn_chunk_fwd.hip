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
// Sequential over the chunks of one (batch, head), one workgroup per slice of VS rows of S: state_fwd_kernel with fp32
// I/O, state_fwd_run_kernel (below) with bf16.  Eight wavefronts carry the chain  S_n -> E_n -> S_{n+1}  (two barriers per chunk):
//   A  S into LDS                                                             | barrier 1
//   B  E = (T diag(beta)) V - W S^T, one 16x16 tile per wavefront; E and rho E (the operand of the
//      write) into LDS                                                        | barrier 2
//   C  S <- gamma_C S + (rho E)^T K~ in the MFMA accumulators
// Four more wavefronts move data.  Two load, directly from global memory into three LDS rings
// (osdn_tile.h): -W; X, what the product with V takes (T diag(beta), the slice of V) and the gates; what
// phase C multiplies (K~; per-channel gates: the chunk's decays).  Two store the checkpoint of S and E^T.  They are
// wavefronts of their own because a memory instruction stalls its wavefront until the CU's address
// unit takes it, which adds to the chain when the
// same wavefronts do both, and because a wavefront's accesses retire in order: a load issued behind a
// store is only known to be there when the store is acknowledged, about 1 us later.
// Bound by what the slices of a chain read over again (84 KB in per chunk at K = 128 with
// slices of 16, 88 with 32): many chains take slices of 32, although -W alone then has a second
// slot.  256 chains of 16 chunks: K = V = 128 412 -> 314 us (the product with V a phase ahead, X and K~ both in
// flight during phase B alone: 390; one slot for -W too: 447), V = 256 799 -> 604, K = 64, V = 128 316 -> 222.
constexpr int CW_ = 8;          // wavefronts of a chain workgroup that compute
constexpr int CM_ = 2;          // ... that load
constexpr int CS_ = 2;          // ... that store
constexpr int CT_ = (CW_ + CM_ + CS_) * 64;
// Ring depths (chunks of operands in LDS) of -W, of T diag(beta), V and the gates, and of K~, from what fits.
constexpr int SF_NSW = 2;
template <int K, int VS> constexpr int SF_NSX = K == 64 || VS == 16 ? 2 : 1;
template <int K, int VS> constexpr int SF_NSC = K == 64 ? 2 : 1;

// GV: one state gate per key channel: the operands carry the decays inside the chunk, and every
// coordinate of the state its own gamma_C; K~ is gamma_C . K~ / Gamma.
// VS: rows of S (values) owned by one workgroup, 32 or 16.  With few chains the narrow slice
// gives twice the workgroups, each with half the work on the dependent path per chunk.
template <int K, bool GV, int VS, bool RAG>
__global__ __launch_bounds__(CT_) void state_fwd_kernel(ChunkArgs a) {
    typedef float T;
    constexpr int ES = sizeof(T), RK = K * ES, RC = C * ES, RV = VS * ES;      // bytes per row of a tile
    constexpr int NVT = VS / 16, NFB = K / 16;
    constexpr int NTC = NFB * NVT, TPW = NTC > CW_ ? NTC / CW_ : 1;            // state tiles, ... per wavefront
    constexpr int KS = Mfma<T>::KSTEP, NKK = K / KS, NKC = C / KS;
    typedef typename Mfma<T>::Frag Frag;
    constexpr int NSW = SF_NSW, NSX = SF_NSX<K, VS>, NSC = SF_NSC<K, VS>;
    constexpr bool AHEAD = NSC > 1;             // the product with V one phase ahead (else phase B has to cover the loads of K~)
    constexpr int X_T = 0, X_V = X_T + C * RC, X_G = X_V + C * RV, X_BYTES = X_G + 2 * C * 4;
    constexpr int C_K = 0, C_D = C_K + C * RK, C_BYTES = C_D + (GV ? K * 4 : 0);
    __shared__ __attribute__((aligned(1024))) char ringW[NSW * C * RK];
    __shared__ __attribute__((aligned(1024))) char ringX[NSX * X_BYTES];
    __shared__ __attribute__((aligned(1024))) char ringC[NSC * C_BYTES];
    __shared__ __attribute__((aligned(1024))) char Sb[VS * RK];         // S in the I/O type [v][kf]
    __shared__ __attribute__((aligned(1024))) char Eo[VS * RC];         // E^T  [v][i]
    __shared__ __attribute__((aligned(1024))) char Ew[GV ? 16 : VS * RC];   // (rho E)^T

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
    // for K~ and X (AHEAD), or for K~, and behind barrier 2 for the others in this order.
    constexpr int LW = LdsLoad<RK, C, CM_>::MIN, LX = LdsLoad<RC, C, CM_>::MIN + LdsLoad<RV, C, CM_>::MIN, LC = LW, LA = LW + LX + LC;
    constexpr int NMAX = NSW > NSX ? (NSW > NSC ? NSW : NSC) : (NSX > NSC ? NSX : NSC);
    constexpr int NEWER_W = (NSW - 1) * LA + (AHEAD ? 0 : LX), NEWER_X = (NSX - 1) * LA, NEWER_C = (NSC - 1) * LA + (AHEAD ? LX : 0);
    constexpr int NEWER_1 = AHEAD || NEWER_W < NEWER_X ? NEWER_W : NEWER_X;
    constexpr int NEWER_2 = !AHEAD || NEWER_C < NEWER_X ? NEWER_C : NEWER_X;
    static_assert(NEWER_1 < 64 && NEWER_2 < 64, "the counter has six bits");
#pragma unroll
    for (int j = 0; j < NMAX; ++j) {
        if (loader && j < NSW && a.n0 + j < a.n1) loadW(a.n0 + j, j);
        if (loader && j < NSX && a.n0 + j < a.n1) loadX(a.n0 + j, j);
        if (loader && j < NSC - 1 && a.n0 + j < a.n1) loadC(a.n0 + j, j);
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
            // a slot is refilled as soon as its operands have been read: ahead of their phase (X), or in it
            if (full) wait_vm<NEWER_1>(); else wait_vm<0>();        // -W, X (not AHEAD)
            __syncthreads();                                        // barrier 1
            if (n - 1 + NSC < a.n1) loadC(n - 1 + NSC, sc == 0 ? NSC - 1 : sc - 1);
            if (AHEAD && n + NSX < a.n1) loadX(n + NSX, sx);
            if (full) wait_vm<NEWER_2>(); else wait_vm<0>();        // X of the next chunk (AHEAD) and K~
            __syncthreads();                                        // barrier 2
            if (n + NSW < a.n1) loadW(n + NSW, sw);
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
    // operands of phase B of one chunk: the product with V, rho of this lane's rows, gamma_C
    f32x4 uacc = {}, rho = {1.f, 1.f, 1.f, 1.f};
    float gC = 1.f;
    auto fetchB = [&](const char *tX) {
        if (inB) {
            uacc = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int kk = 0; kk < NKC; ++kk)
                if (kk * KS < (rb + 1) * 16)                    // T is lower triangular
                    uacc = Mfma<T>::mma(fT.kc(tX + X_T, rb * 16, kk * KS), fV.tr(tX + X_V, kk * KS, vtB * 16), uacc);
            if (!GV) rho = *reinterpret_cast<const f32x4 *>(tX + X_G + (rb * 16 + acc_row(lane, 0)) * 4 + C * 4);
        }
        if (!GV) gC = *reinterpret_cast<const float *>(tX + X_G + (C - 1) * 4);
    };
    if (AHEAD) fetchB(ringX);
    for (int n = a.n0; n < a.n1; ++n) {
        const char *tW = ringW + sw * C * RK, *tC = ringC + sc * C_BYTES;
        // ---- phase A ----
        if (inC) {
#pragma unroll
            for (int q = 0; q < TPW; ++q) fK.put(Sb, (vtC + q) * 16, fb * 16, St[q]);
        }
        __syncthreads();                                            // barrier 1
        // ---- phase B ----
        Frag sf[NKK];
        if (!AHEAD) fetchB(ringX + sx * X_BYTES);
        if (inB) {
#pragma unroll
            for (int kk = 0; kk < NKK; ++kk) sf[kk] = fK.kc(Sb, vtB * 16, kk * KS);
        }
        if (inB) {
            f32x4 acc = {0.f, 0.f, 0.f, 0.f}, acc2 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int kk = 0; kk < NKK; kk += 2) {
                acc = Mfma<T>::mma(fK.kc(tW, rb * 16, kk * KS), sf[kk], acc);
                acc2 = Mfma<T>::mma(fK.kc(tW, rb * 16, (kk + 1) * KS), sf[kk + 1], acc2);
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
            f32x4 dc = {};
            if (GV) dc = *reinterpret_cast<const f32x4 *>(tC + C_D + (fb * 16 + acc_row(lane, 0)) * 4);
#pragma unroll
            for (int q = 0; q < TPW; ++q)
#pragma unroll
                for (int kk = 0; kk < NKC; ++kk) fe[q][kk] = fT.kc(GV ? Eo : Ew, (vtC + q) * 16, kk * KS);
#pragma unroll
            for (int q = 0; q < TPW; ++q) {
#pragma unroll
                for (int r = 0; r < 4; ++r) St[q][r] *= GV ? dc[r] : g;
#pragma unroll
                for (int kk = 0; kk < NKC; ++kk) St[q] = Mfma<T>::mma(fK.tr(tC + C_K, kk * KS, fb * 16), fe[q][kk], St[q]);
            }
        }
        sw = next(sw, NSW); sx = next(sx, NSX); sc = next(sc, NSC);
        if (AHEAD && n + 1 < a.n1) fetchB(ringX + sx * X_BYTES);
    }
    if (inC) {
#pragma unroll
        for (int q = 0; q < TPW; ++q) {
            const int v = vs + (vtC + q) * 16 + acc_col(lane), c0 = fb * 16 + acc_row(lane, 0);
            *reinterpret_cast<f32x4 *>(a.S_out + (bh * a.V + v) * K + c0) = St[q];
        }
    }
}

// ------------------------------------------------------- state_fwd, bf16 ----
// The same chain with bf16 I/O.  Two wavefronts own 16 values, each half of the features of S and, in E, 32 of the 64 tokens.  The
// accumulator tiles of S (and of rho E) are laid out so that their rounded values are the next product's operand as they stand
// (RunFrag in osdn_tile.h): through LDS go only the half that the other wavefront holds and what is stored.
//   A  S, rounded, into LDS                                                                         | barrier 1
//   B  E = (T diag(beta)) V - W S^T of 32 tokens; E and rho E into LDS                              | barrier 2
//   C  S <- gamma_C S + (rho E)^T K~ in the MFMA accumulators, half of the features
// A third wavefront forms (T diag(beta)) V of the chunk after; two load (two LDS rings, three chunks deep: -W, T diag(beta) and
// V; K~ and the gates), two store the checkpoint of S and E^T.
// What bounds it (cycles a chunk, measured with the clock in every wavefront; 16 chains of 512 chunks, K = V = 128, slices of
// 16): the chain itself takes 1050 of 1980; the rest is waiting for the loaders, whose accesses (22 of 1 KB each) are
// taken the slower the more lines are on their way from HBM, and by the stores beside them (without stores 1500; with both
// out of the L2 1650).  Hence the lines that the slices of a chain share are asked for PF chunks ahead where they sit on one XCD and
// come from HBM (asks_ahead in osdn_plan.h), each slice a share of them, 4 bytes a line: without that 2360.  Eight wavefronts with a tile of 16 x 16 each, S and E all
// through LDS, read 82 KB of LDS a chunk instead of 44 (at 64 bytes a clock) and took 2250: state_fwd 535 -> 467 us; 16 chains
// of 128 chunks, V = 256 155 -> 139; in all 1026 -> 944 and 862 -> 845 us.  With -W and T diag(beta) straight from memory
// to registers, 16 rows of 64 bytes an access, 2750.
// Slices of 32 (many chains) are bound by HBM, at 4.0 of the 5.3 TB/s that a copy reaches: 1072 chains, 486 -> 471 us, 64 of 32
// chunks 53.1 -> 52.5; asking ahead only costs there (66).
constexpr int RM_ = 2, RS_ = 2;      // wavefronts that load, that store
template <int VS> constexpr int RT_ = (3 * (VS / 16) + RM_ + RS_) * 64;      // threads
template <int K, bool GV, int VS, bool RAG>
__global__ __launch_bounds__(RT_<VS>, 1) void state_fwd_run_kernel(ChunkArgs a) {
    typedef bf16 T;
    typedef Mfma<T>::Frag Frag;
    constexpr int NV = VS / 16, ES = sizeof(T), RK = K * ES, RC = C * ES, RV = VS * ES;      // bytes per row of a tile
    constexpr int NF = K / 32, NFW = NF / 2, NT = C / 32;     // blocks of 32 features, those of a wavefront, blocks of 32 tokens
    constexpr int NSW = 3, NSC = 3;             // ring depths (chunks)
    constexpr int PF = 8;                       // chunks by which the lines are asked for ahead
    constexpr int W_T = C * RK, W_V = W_T + C * RC, W_BYTES = W_V + C * RV;
    constexpr int C_G = C * RK, C_BYTES = C_G + (GV ? K : 2 * C) * 4;
    __shared__ __attribute__((aligned(1024))) char ringW[NSW * W_BYTES];
    __shared__ __attribute__((aligned(1024))) char ringC[NSC * C_BYTES];
    __shared__ __attribute__((aligned(1024))) char Sb[VS * RK];             // S in the I/O type [v][kf]
    __shared__ __attribute__((aligned(1024))) char Eo[VS * RC];             // E^T  [v][i]
    __shared__ __attribute__((aligned(1024))) char Ew[GV ? 16 : VS * RC];   // (rho E)^T
    __shared__ __attribute__((aligned(1024))) f32x4 Ub[NV][4][64];          // (T diag(beta)) V as accumulator tiles
    __shared__ __attribute__((aligned(1024))) char dump[256];

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
        a.S_in = begins ? a.S_first : a.S_out;
        bt = 0;
    }
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const bool loader = wave >= 3 * NV && wave < 3 * NV + RM_, storer = wave >= 3 * NV + RM_;
    const int mw = wave - 3 * NV, mt = tid - (3 * NV + RM_) * 64;     // loader wavefront, storer thread
    const size_t bh = (size_t)b * a.H + h;      // the chain: indexes S_in / S_out
    const uint32_t gV = (uint32_t)a.H * (uint32_t)a.V * ES;        // bytes between tokens of v
    const ChainRows<RAG> rows(a.rows, a.seq_chunks, b, a.n0);
    const bool wideV = (reinterpret_cast<uintptr_t>(a.v) & 15) == 0;
    auto tile_of = [&](int n) { return ((size_t)bt * a.N + n) * a.H + h; };
    auto next = [](int slot, int depth) { return slot + 1 == depth ? 0 : slot + 1; };

    if (loader) {
        LdsLoad<RK, C, RM_> lW;
        LdsLoad<RK, C, RM_, SwzRun<RK>> lK;
        LdsLoad<RC, C, RM_> lT;
        LdsLoad<RV, C, RM_> lV;
        lW.init(RK, mw, lane); lK.init(RK, mw, lane); lT.init(RC, mw, lane); lV.init(gV, mw, lane);
        auto loadW = [&](int n, int slot) {
            char *s = ringW + slot * W_BYTES;
            lW.issue(s, static_cast<const char *>(a.Wn) + tile_of(n) * C * RK, RK, mw, lane, slice);
        };
        auto loadU = [&](int n, int slot) {
            char *s = ringW + slot * W_BYTES;
            lT.issue(s + W_T, static_cast<const char *>(a.Tu) + tile_of(n) * C * RC, RC, mw, lane, slice);
            lV.issue(s + W_V, static_cast<const char *>(a.v) + (rows.first(n) * a.H + h) * a.V * ES + (size_t)vs * ES,
                     gV, mw, lane, 0, wideV, rows.count(n) - 1);      // (rows behind the last: their columns of T diag(beta) are zero)
        };
        auto loadC = [&](int n, int slot) {
            char *s = ringC + slot * C_BYTES;
            lK.issue(s, static_cast<const char *>(a.kt) + tile_of(n) * C * RK, RK, mw, lane, slice);
            const int w = mw;
            if (!GV) load_lds4(a.gates + (tile_of(n) * 3 + 1 + w) * C, lane * 4, lds_offset(s + C_G + w * C * 4));     // gamma, rho
            else if (w < K / 64) load_lds4(a.gamC + tile_of(n) * K, w * 256 + lane * 4, lds_offset(s + C_G + w * 256));
        };
        static_assert(RM_ == 2, "gamma and rho");
        constexpr int LW = LdsLoad<RK, C, RM_>::MIN + LdsLoad<RC, C, RM_>::MIN + LdsLoad<RV, C, RM_>::MIN;
        constexpr int LC = LdsLoad<RK, C, RM_>::MIN + (!GV || K / 64 >= RM_ ? 1 : 0);
        for (int j = 0; j < NSW && a.n0 + j < a.n1; ++j) {
            loadU(a.n0 + j, j); loadW(a.n0 + j, j);
            if (j < NSC - 1) loadC(a.n0 + j, j);
        }
        wait_vm<0>();
        __builtin_amdgcn_s_waitcnt(0x0f70);     // vmcnt(0), said to the compiler too
        __syncthreads();
        int sw = 0, sc = NSC - 1;               // slots of -W of chunk n, of K~ of chunk n + 2
        for (int n = a.n0; n < a.n1; ++n) {
            // K~ of this chunk, -W of the next: all that was asked for two chunks ago
            if (n + 2 < a.n1) wait_vm<LW + LC>();
            else if (n + 1 < a.n1) wait_vm<LC>();
            else wait_vm<0>();
            __syncthreads();                                        // barrier 1
            if (n + 2 < a.n1) loadC(n + 2, sc);
            if (n + 3 < a.n1) loadU(n + 3, sw);
            __syncthreads();                                        // barrier 2
            if (n + 3 < a.n1) loadW(n + 3, sw);
            sw = next(sw, NSW); sc = next(sc, NSC);
        }
        return;
    }
    if (storer) {
        constexpr int NS = VS * RK / 16 / (RS_ * 64), G = RK / 16;      // accesses of a thread for S; 16-byte groups of a row
        static_assert(NS >= 1 && VS * RK % (RS_ * 64 * 16) == 0, "S by 16 bytes a thread");
        __syncthreads();
        for (int n = a.n0; n < a.n1; ++n) {
            char *sg = static_cast<char *>(a.S_ckpt) + (tile_of(n) * a.V + vs) * RK;
            __syncthreads();                                        // barrier 1
            u32x4 x[NS];
#pragma unroll
            for (int i = 0; i < NS; ++i) {
                const uint32_t v = (mt + i * RS_ * 64) / G, c = (mt + i * RS_ * 64) % G;
                x[i] = *reinterpret_cast<const u32x4 *>(Sb + Swz<RK>::at(v, c));
            }
#pragma unroll
            for (int i = 0; i < NS; ++i) {
                if (i == (NS + 1) / 2) __syncthreads();             // barrier 2
                *reinterpret_cast<u32x4 *>(sg + (mt + i * RS_ * 64) * 16) = x[i];
            }
            if (NS == 1) __syncthreads();                           // barrier 2
            tile_to_global<RC, VS>(static_cast<char *>(a.Et) + (tile_of(n) * a.V + vs) * RC, RC, Eo, mt, RS_ * 64);
        }
        return;
    }
    const int m = lane & 15, q = lane >> 4;
    if (wave >= 2 * NV) {                       // (T diag(beta)) V of the chunk after
        const int vt = wave - 2 * NV;
        RunFrag<RC> fT;
        TileFrag<T, RV> fV;
        fT.init(lane); fV.init(lane);
        f32x4 u[4];
        auto product = [&](const char *s) {
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                u[t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int kk = 0; kk <= t / 2; ++kk)                     // T is lower triangular
                    u[t] = Mfma<T>::mma(fT.rows(s + W_T, t / 2 * 32, t & 1, kk * 32), fV.tr(s + W_V, kk * 32, vt * 16), u[t]);
            }
        };
        auto keep = [&] {
#pragma unroll
            for (int t = 0; t < 4; ++t) Ub[vt][t][lane] = u[t];
        };
        // This slice's share of the lines of a chunk's operands, in the order -W, K~, T diag(beta), gates, V: lane l asks for the
        // l-th and the (64 + l)-th, whose addresses step from chunk to chunk.
        constexpr int GS = (GV ? K : 3 * C) * 4;                        // bytes from one chunk's gates to the next's
        constexpr int LK = C * RK / LINE, LT = C * RC / LINE, LG = (GV ? K : 2 * C) * 4 / LINE, L0 = 2 * LK + LT + LG;
        const int lpr = a.V * ES / LINE, all = L0 + C * lpr, share = (all + a.V / VS - 1) / (a.V / VS);
        const char *lp[2];
        uint32_t ls[2];
        int lr[2];                              // the row of V, or 0
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int i = lane + 64 * j, l = slice * share + i;
            const size_t t0 = tile_of(a.n0);
            lr[j] = i < share && l < all ? 0 : C;                       // (no row: nothing to ask for)
            if (l < LK) { lp[j] = static_cast<const char *>(a.Wn) + t0 * C * RK + l * LINE; ls[j] = C * RK; }
            else if (l < 2 * LK) { lp[j] = static_cast<const char *>(a.kt) + t0 * C * RK + (l - LK) * LINE; ls[j] = C * RK; }
            else if (l < 2 * LK + LT) { lp[j] = static_cast<const char *>(a.Tu) + t0 * C * RC + (l - 2 * LK) * LINE; ls[j] = C * RC; }
            else if (l < L0) { lp[j] = reinterpret_cast<const char *>(GV ? a.gamC : a.gates + C) + t0 * GS + (l - 2 * LK - LT) * LINE; ls[j] = GS; }
            else {
                const int r = (l - L0) / lpr;
                lp[j] = static_cast<const char *>(a.v) + ((rows.first(a.n0) + r) * a.H + h) * a.V * ES + (l - L0) % lpr * LINE;
                ls[j] = C * a.V * ES;
                if (lr[j] == 0) lr[j] = r;
            }
        }
        int pf = a.n0;                          // the chunk that lp stands at
        auto ahead = [&](int n) {
            const uint32_t step = (uint32_t)(n - pf) * (uint32_t)a.H;
            pf = n;
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                if (64 * j >= share) break;
                lp[j] += (size_t)step * ls[j];
                if (lr[j] < rows.count(n)) touch(lp[j], lds_offset(dump));
            }
        };
        __syncthreads();
        product(ringW);
        keep();
        int sw = 1;
        for (int n = a.n0; n < a.n1; ++n) {
            __syncthreads();                                        // barrier 1
            product(ringW + sw * W_BYTES);      // (behind the last chunk: in vain)
            sw = next(sw, NSW);
            __syncthreads();                                        // barrier 2
            keep();
            if (VS == 16 && a.asks_ahead && n + PF < a.n1) ahead(n + PF);
        }
        wait_vm<0>();
        return;
    }
    // ---- the chain: two wavefronts per 16 values, each with half of the features ----
    const int half = wave & 1, vt = wave >> 1, f0 = half * NFW;
    RunFrag<RK> fK;
    fK.init(lane);
    f32x4 St[NFW][2] = {};                      // transposed: rows = features, cols = values
    const size_t at = (bh * a.V + vs + vt * 16 + m) * K + f0 * 32 + q * 8;
    if (a.S_in) {
#pragma unroll
        for (int f = 0; f < NFW; ++f)
#pragma unroll
            for (int e = 0; e < 2; ++e) St[f][e] = *reinterpret_cast<const f32x4 *>(a.S_in + at + f * 32 + e * 4);
    }
    auto sb_at = [&](int f) { return reinterpret_cast<Frag *>(Sb + (Swz<RK>::at(vt * 16 + m, q) ^ (uint32_t)(f << 6))); };
    auto e_at = [&](char *E, int t) { return reinterpret_cast<Frag *>(E + (Swz<RC>::at(vt * 16 + m, q) ^ (uint32_t)(t << 6))); };
    Frag wf[2][NF];                             // -W: the 32 tokens that this wavefront forms E of
    auto readW = [&](const char *s) {
#pragma unroll
        for (int kk = 0; kk < NF; ++kk)
#pragma unroll
            for (int e = 0; e < 2; ++e) wf[e][kk] = fK.rows(s, half * 32, e, kk * 32);
    };
    __syncthreads();
    readW(ringW);
    int sw = 1, sc = 0;                         // slots of -W of chunk n + 1, of K~ of chunk n
    for (int n = a.n0; n < a.n1; ++n) {
        const char *s = ringC + sc * C_BYTES;
        // ---- phase A ----
        Frag sf[NF];
#pragma unroll
        for (int f = 0; f < NFW; ++f) *sb_at(f0 + f) = RunFrag<RK>::pack(St[f][0], St[f][1]);
        __syncthreads();                                            // barrier 1
        // ---- phase B ----
#pragma unroll
        for (int f = 0; f < NF; ++f) sf[f] = *sb_at(f);
        f32x4 u[2], rho[2], dc[NFW][2];
        float g = 1.f;
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            u[e] = Ub[vt][half * 2 + e][lane];
            if (!GV) rho[e] = *reinterpret_cast<const f32x4 *>(s + C_G + (C + half * 32 + q * 8 + e * 4) * 4);
        }
        if (!GV) g = *reinterpret_cast<const float *>(s + C_G + (C - 1) * 4);
        Frag kf[NFW][2][NT];
#pragma unroll
        for (int f = 0; f < NFW; ++f)
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                if (GV) dc[f][e] = *reinterpret_cast<const f32x4 *>(s + C_G + ((f0 + f) * 32 + q * 8 + e * 4) * 4);
#pragma unroll
                for (int t = 0; t < NT; ++t) kf[f][e][t] = fK.tr(s, t * 32, (f0 + f) * 32, e);
            }
        f32x4 acc[2] = {}, acc2[2] = {};
#pragma unroll
        for (int kk = 0; kk < NF; kk += 2)
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                acc[e] = Mfma<T>::mma(wf[e][kk], sf[kk], acc[e]);
                acc2[e] = Mfma<T>::mma(wf[e][kk + 1], sf[kk + 1], acc2[e]);
            }
        f32x4 ew[2];
#pragma unroll
        for (int e = 0; e < 2; ++e)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                acc[e][r] = u[e][r] + (acc[e][r] + acc2[e][r]);     // (last: begun with U, every step would round at its size)
                if (!GV) ew[e][r] = acc[e][r] * rho[e][r];
            }
        if (!GV) *e_at(Ew, half) = RunFrag<RC>::pack(ew[0], ew[1]);
        *e_at(Eo, half) = RunFrag<RC>::pack(acc[0], acc[1]);
        __syncthreads();                                            // barrier 2
        // ---- phase C ----
        Frag ef[NT];
#pragma unroll
        for (int t = 0; t < NT; ++t) ef[t] = *e_at(GV ? Eo : Ew, t);
        readW(ringW + sw * W_BYTES);            // (behind the last chunk: in vain)
#pragma unroll
        for (int f = 0; f < NFW; ++f)
#pragma unroll
            for (int e = 0; e < 2; ++e) {
#pragma unroll
                for (int r = 0; r < 4; ++r) St[f][e][r] *= GV ? dc[f][e][r] : g;
            }
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int f = 0; f < NFW; ++f)
#pragma unroll
                for (int e = 0; e < 2; ++e) St[f][e] = Mfma<T>::mma(kf[f][e][t], ef[t], St[f][e]);
        sw = next(sw, NSW); sc = next(sc, NSC);
    }
#pragma unroll
    for (int f = 0; f < NFW; ++f)
#pragma unroll
        for (int e = 0; e < 2; ++e) *reinterpret_cast<f32x4 *>(a.S_out + at + f * 32 + e * 4) = St[f][e];
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
template <bool BF16, bool GV, int VS>
static int launch_state_t(const ChunkArgs &a, hipStream_t st) {
    ChunkArgs b = a;
    b.map = slice_map(a.V / VS, a.H * (long long)(a.seq_chunks ? a.n_seqs : a.B), VS == 16);
    dim3 grid(chain_workgroups(b.map)), block(BF16 ? RT_<VS> : CT_);
    if (GV && !a.gamC) return -1;
    auto launch = [&](auto k) {
        constexpr int K = decltype(k)::value;
        with_rows(a.rows, [&](auto rag) {
            constexpr bool RAG = decltype(rag)::value;
            if constexpr (BF16) hipLaunchKernelGGL((state_fwd_run_kernel<K, GV, VS, RAG>), grid, block, 0, st, b);
            else hipLaunchKernelGGL((state_fwd_kernel<K, GV, VS, RAG>), grid, block, 0, st, b);
        });
    };
    if (a.K == 64) launch(std::integral_constant<int, 64>{});
    else if (a.K == 128) launch(std::integral_constant<int, 128>{});
    else return -1;
    return 0;
}
// Slices of 16 values when the caller asks for them (few chains: see osdn_fwd), else of 32.
template <bool BF16, bool GV>
static int launch_state_v(const ChunkArgs &a, hipStream_t st) {
    return a.narrow_slices ? launch_state_t<BF16, GV, 16>(a, st) : launch_state_t<BF16, GV, 32>(a, st);
}
int launch_state_fwd(const ChunkArgs &a, bool bf16_io, hipStream_t st) {
    if (a.gate_vec) return bf16_io ? launch_state_v<true, true>(a, st) : launch_state_v<false, true>(a, st);
    return bf16_io ? launch_state_v<true, false>(a, st) : launch_state_v<false, false>(a, st);
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
