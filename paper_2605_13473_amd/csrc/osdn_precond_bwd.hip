// Reverse sweep over the projected affine recurrence of the preconditioner (Section 4.5),
// split so that only what is sequential stays on the sequential path.
//
// With  abar_t = mask_t (.) a_{t+1},  sigma_t = <s_t, abar_t>,  s_t = k_t (.) k_t,
//       a_t    = k_t (.) dL/dk~_t + r_t abar_t - ca_t sigma_t s_t        (ca_t = eta b'^2 / n_t)
// the only coupling between chunks is the K-vector a at the chunk boundary, and inside a chunk
// the only coupling between coordinates is the scalar sigma_t.  Three kernels:
//   precond_mask   one workgroup per (chain, chunk), all chunks in parallel: replays d from the
//                  stored chunk-start value and step scalars and records, per coordinate, the
//                  64-bit mask of tokens whose unprojected update stayed inside the box
//   precond_chain  one workgroup per chain, chunks right to left: finds sigma by fixed-point
//                  sweeps (as the forward kernel finds <d, s>), keeps the adjoint at every chunk
//                  boundary and the 64 sigmas of every chunk, nothing else
//   precond_post   one workgroup per (chain, chunk), all chunks in parallel, one thread per
//                  coordinate: replays d, re-runs the adjoint recurrence of its chunk from the
//                  stored boundary value, sigmas and masks, and writes dk, dbeta, dretention
// The retention gate is absent, one value per (token, head), or one per coordinate (RET).
//
// Without retention, on a chunk in which no coordinate met the box (every mask bit set), the
// recurrence is linear with constant coefficients:  abar_i = g + sum_{j>i} (lambda_j - ca_j
// sigma_j s_j)  (g = the adjoint at the chunk's right end, lambda_j = k_j (.) dL/dk~_j), hence
//     (I + U) sigma = S g + rho0,   U_ij = <s_i, s_j> ca_j (j > i),   rho0_i = <s_i, sum_{j>i} lambda_j>,
//     a_left = g + sum_j lambda_j - S^T (ca (.) sigma).
//   precond_lin_m  one workgroup per (chain, chunk), all chunks in parallel, needs the forward
//                  pass only: writes the chunk's masks (in place of precond_mask, which is not
//                  launched when this form is on), decides whether the chunk qualifies and, if
//                  so, leaves (I + U)^-1 (Gram matrix and blocked inverse on the fp32 MFMA), kept
//                  in the I/O type;
//   precond_lin_r  the same grid, once dL/dk~ of the chunk is there: rho0 and sum_j lambda_j;
// on such a chunk precond_chain_lin only has the three matrix-vector products left (osdn_precond.h,
// "a chunk of the recurrence in solved form"); on any other chunk it runs its sweeps.
#include "osdn_precond.h"

namespace osdn {

// ---------------------------------------------------------------- precond_mask ----
// RET (all three kernels): 0 = no retention, 1 = one gate per (token, head), 2 = one per coordinate
template <typename T, int K, int RET, bool RAG>
__global__ __launch_bounds__(K) void precond_mask_kernel(PrecondBwdArgs a) {
    constexpr bool HAS_RET = RET != 0, RET_VEC = RET == 2;
    __shared__ __attribute__((aligned(16))) float steps[C];
    __shared__ __attribute__((aligned(16))) float rs[C];
    const int n = a.n0 + blockIdx.x / a.H, h = blockIdx.x % a.H, b = blockIdx.y, tid = threadIdx.x;
    const int N = a.T / C;
    const size_t bh = (size_t)b * a.H + h;
    const size_t tokc = ((size_t)b * a.T + (size_t)n * C) * a.H + h;
    // Without retention, a chunk that the forward sweep marked (mark_bound; its last run says): every bit is set, and neither k nor d is read (no chunk near
    // the box: 1072 chains, 78 us of 3346; 64 chains of 64 chunks, beside bwd_chain, training step 1011 -> 998).
    if (!HAS_RET && __builtin_bit_cast(int, a.tok_scalars[(tokc + (size_t)(C - 1) * a.H) * 4 + 2]) < 0) {
        a.masks[(bh * N + n) * K + tid] = make_uint2(0xffffffffu, 0xffffffffu);
        return;
    }
    const ChunkIn<T, K, RET, RAG> in(a, b, n, h);
    const bool project = a.d_min <= a.d_max;
    const float lo = project ? a.d_min : -INFINITY, hi = project ? a.d_max : INFINITY;
    if (tid < C) {
        const size_t th = tokc + (size_t)tid * a.H;
        steps[tid] = a.tok_scalars[th * 4];
        rs[tid] = (HAS_RET && !RET_VEC) ? in.ret[(size_t)tid * a.H] : 1.f;
    }
    const T *kp = in.k;
    const float *rp = in.ret;
    const uint32_t kstride = (uint32_t)a.H * K;
    float kv[C], rvv[RET_VEC ? C : 1];
#pragma unroll
    for (int i = 0; i < C; ++i) {
        kv[i] = to_f32(kp[(uint32_t)tid + (uint32_t)i * kstride]);
        if (RET_VEC) rvv[RET_VEC ? i : 0] = rp[(uint32_t)tid + (uint32_t)i * kstride];
    }
    float d = a.d_ckpt[(bh * N + n) * K + tid];
    __syncthreads();
    uint32_t mlo = 0u, mhi = 0u;
#pragma unroll
    for (int i = 0; i < C; ++i) {
        const float sq = kv[i] * kv[i];
        const float r = RET_VEC ? rvv[RET_VEC ? i : 0] : rs[i];
        const uint32_t bit = lands_inside<HAS_RET>(r, d, steps[i], sq, lo, hi) ? (1u << (i & 31)) : 0u;
        d = clip3(d_bar<HAS_RET>(r, d, steps[i], sq), lo, hi);
        if (i < 32) mlo |= bit; else mhi |= bit;
    }
    a.masks[(bh * N + n) * K + tid] = make_uint2(mlo, mhi);
}

// ----------------------------------------------------------------- precond_lin ----
// Two kernels, both one workgroup per (chain, chunk).  precond_lin_m needs the forward pass only
// (keys, step scalars, d at the chunk start): it replays d over the chunk for the box masks (what
// precond_mask does when this form is off: the same arithmetic, from the s tile it builds anyway),
// decides from them whether the chunk qualifies, and inverts the system.
// precond_lin_r needs dL/dk~ of the chunk as well: rho0 and the sum of lambda.
template <typename T, int K, bool RAG>
__global__ __launch_bounds__(P1T) void precond_lin_m_kernel(PrecondBwdArgs a) {
    typedef Lin<K> LN;
    constexpr int EPT = LN::EPT, VN = 16 / sizeof(T), NVK = EPT / VN;
    constexpr int LDT = K + 4;                   // s tile: MFMA fragment reads (row = lane % 16, k = lane / 16) spread over the banks
    constexpr int LDF = C + 1;
    constexpr int TI_F = C * LDF + 3 * 16 * 17;  // (I + A)^-1 and the block products: in the s tile's space once A is built
    static_assert(TI_F <= C * LDT || K == 64, "the inverse reuses the s tile");
    __shared__ __attribute__((aligned(16))) float Ss[C * LDT > TI_F ? C * LDT : TI_F];
    __shared__ __attribute__((aligned(16))) float Af[C * LDF];
    __shared__ float cas[C];
    __shared__ float steps[C];
    float *Ti = Ss, *Xs = Ss + C * LDF;

    const int n = a.n0 + blockIdx.x / a.H, h = blockIdx.x % a.H, b = blockIdx.y;
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int N = a.T / C;
    const size_t bhn = ((size_t)b * a.H + h) * N + n;
    const size_t tokc = ((size_t)b * a.T + (size_t)n * C) * a.H + h;
    const ChunkIn<T, K, 0, RAG> src(a, b, n, h);
    const int i = tid >> 3, part = tid & 7;
    const uint32_t kstride = (uint32_t)a.H * K;
    u32x4 kv[NVK];
    {
        const uint32_t off = ((uint32_t)i * kstride + (uint32_t)(part * EPT)) * (uint32_t)sizeof(T);
        const u32x4 *kp = reinterpret_cast<const u32x4 *>(src.k);
#pragma unroll
        for (int m = 0; m < NVK; ++m) kv[m] = at_byte(kp, off + 16 * m);
    }
    const bool project = a.d_min <= a.d_max;
    float nraw = 1.f, bet = 0.f, d = 1.f;
    if (tid < C) {
        const size_t th = tokc + (size_t)tid * a.H;
        const float4 sc = *reinterpret_cast<const float4 *>(a.tok_scalars + th * 4);
        steps[tid] = sc.x;
        nraw = sc.z;
        bet = src.beta[(size_t)tid * a.H];
    }
    if (project && tid < K) d = a.d_ckpt[bhn * K + tid];
#pragma unroll
    for (int m = 0; m < NVK; ++m)
#pragma unroll
        for (int e4 = 0; e4 < VN; e4 += 4) {
            float sq[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float kf = vec_get<T>(kv[m], e4 + e);
                sq[e] = kf * kf;
            }
            store_vec(Ss + i * LDT + part * EPT + m * VN + e4, sq);
        }
    __syncthreads();
    // ---- the box masks of the chunk; does it qualify?  (no coordinate met the box at any token) ----
    bool ok = true;
    if (project && tid < K) {
        uint32_t mlo = 0u, mhi = 0u;
#pragma unroll 8
        for (int t = 0; t < C; ++t) {
            const float sq = Ss[t * LDT + tid], st = steps[t];
            const uint32_t in = lands_inside<false>(1.f, d, st, sq, a.d_min, a.d_max) ? (1u << (t & 31)) : 0u;
            d = clip3(d_bar<false>(1.f, d, st, sq), a.d_min, a.d_max);
            if (t < 32) mlo |= in; else mhi |= in;
        }
        a.masks[bhn * K + tid] = make_uint2(mlo, mhi);
        ok = (mlo & mhi) == 0xffffffffu;
    }
    const int clean = __syncthreads_and(ok ? 1 : 0);
    if (tid == 0) a.lin_clean[bhn] = clean;
    if (!clean) return;
    if (tid < C) {
        const float nn = fmaxf(fabsf(nraw), a.eps);
        const float bp = a.beta_aware ? bet : 1.f;
        cas[tid] = a.eta * bp / nn * bp;
    }
    __syncthreads();
    // ---- A = tril(ca_i <s_i, s_j>, -1): the transpose of U; (I + A)^-1 = ((I + U)^-1)^T ----
    for (int idx = wave; idx < 10; idx += P1W) {
        const int ib = idx < 1 ? 0 : idx < 3 ? 1 : idx < 6 ? 2 : 3;
        const int jb = idx - (ib * (ib + 1)) / 2;
        const f32x4 acc = mma_tile0<float, true, true>(Ss + ib * 16 * LDT, LDT, Ss + jb * 16 * LDT, LDT, K, lane);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int ii = ib * 16 + acc_row(lane, r), jj = jb * 16 + acc_col(lane);
            Af[ii * LDF + jj] = (jj < ii) ? cas[ii] * acc[r] : 0.f;
        }
    }
    __syncthreads();                                             // the s tile is dead: its space takes the inverse
    ut_inverse64<LDF, 17>(Af, Ti, Xs, 16 * 17, wave, lane);
    // ---- (I + U)^-1, row i: entries j >= i are column i of the lower inverse ----
    // (kept in the I/O type: its diagonal is 1 and the rest is of the size of the step, so with
    // bf16 I/O the rounding is far inside what that I/O type's other operands carry)
    {
        T *mg = static_cast<T *>(a.lin_M) + bhn * C * C + i * C + part * 8;
        constexpr int VNM = 16 / sizeof(T);
#pragma unroll
        for (int e4 = 0; e4 < 8; e4 += VNM) {
            float o[VNM];
#pragma unroll
            for (int e = 0; e < VNM; ++e) {
                const int j = part * 8 + e4 + e;
                o[e] = j >= i ? Ti[j * LDF + i] : 0.f;
            }
            store_vec(mg + e4, o);
        }
    }
}

// rho0_i = <s_i, sum_{j > i} lambda_j> and sum_j lambda_j, lambda_j = k_j (.) dL/dk~_j: thread
// (c = tid % K, tg = tid / K) keeps TS consecutive tokens of coordinate c in registers; the suffix
// sums run down its tokens and across the runs through LDS; the row dots are folded over the lanes
// as in the sweeps of precond_chain.
template <typename T, int K, bool RAG>
__global__ __launch_bounds__(P1T) void precond_lin_r_kernel(PrecondBwdArgs a) {
    constexpr int NSEG = P1T / K, TS = C / NSEG, WPS = K / 64, NPART = K / TS;
    __shared__ float tot[NSEG * K];
    __shared__ float part[P1W * 64];
    const int n = a.n0 + blockIdx.x / a.H, h = blockIdx.x % a.H, b = blockIdx.y;
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int c = tid % K, sg = tid / K;
    const int N = a.T / C;
    const size_t bhn = ((size_t)b * a.H + h) * N + n;
    if (!a.lin_clean[bhn]) return;                               // (uniform)
    const uint32_t kstride = (uint32_t)a.H * K;
    const ChunkIn<T, K, 0, RAG> src(a, b, n, h);
    const T *kp = src.k, *gp = static_cast<const T *>(a.dkt) + (((size_t)b * N + n) * a.H + h) * C * K;
    float sv[TS], lam[TS];
#pragma unroll
    for (int u = 0; u < TS; ++u) {
        const float kf = to_f32(lane_elem(kp, (uint32_t)(sg * TS + u) * kstride + (uint32_t)c));
        sv[u] = kf * kf;
        lam[u] = kf * to_f32(lane_elem(gp, (sg * TS + u) * K + c));
    }
    float acc = 0.f;
#pragma unroll
    for (int u = TS - 1; u >= 0; --u) {                          // exclusive suffix sums inside the run
        const float t = lam[u];
        lam[u] = acc;
        acc += t;
    }
    tot[sg * K + c] = acc;
    __syncthreads();
    float offs = 0.f;
#pragma unroll
    for (int g2 = NSEG - 1; g2 > 0; --g2)
        if (g2 > sg) offs += tot[g2 * K + c];
    if (sg == 0) a.lin_t0[bhn * K + c] = acc + offs;
    float prod[TS];
#pragma unroll
    for (int u = 0; u < TS; ++u) prod[u] = sv[u] * (lam[u] + offs);
    part[wave * 64 + lane] = lane_fold<TS>(prod, lane);
    __syncthreads();
    if (tid < C) {
        const int w0 = (tid / TS) * WPS, u = tid % TS;
        float r = 0.f;
#pragma unroll
        for (int j = 0; j < NPART; ++j) r += part[(w0 + j / (64 / TS)) * 64 + (j % (64 / TS)) * TS + u];
        a.lin_r0[bhn * C + tid] = r;
    }
}

// --------------------------------------------------------------- precond_chain ----
// The adjoint recurrence is linear in a (the masks are data of the forward pass).  A chunk is cut into
// runs of 8 tokens, one wavefront per run, K / 64 adjacent coordinates per lane, everything in registers,
// as in the forward kernel.  Per coordinate a run maps the adjoint at its right end to P a + L at its left:
// P (mask bits and retentions) is a property of the chunk, L depends on the run's sigma.  A sweep
// composes L from its sigma, publishes it, chains the runs to its right (one fma each), replays its
// tokens and folds the products s_i abar_i over the lanes of the wavefront: the next sigma.
//
// The first sweep takes sigma = 0, the second what the first found; what the second finds is accepted
// if it moved by so little that the next would move by less than the tolerance (differences shrink by the
// ratio just seen); the adjoint at the chunk's left end is the one that gave it.  Two barriers a chunk: the
// verdict on sigma is published together with the first maps of the next chunk (which need no adjoint); a
// chunk that is then found not to have settled is done again with three sweeps before the verdict, and so are
// the chunks after it, until eight in a row would have settled in two.  One that does not settle in three either is
// done again with a barrier for every verdict, and so are those after it until eight in a row take no more than three.
// (One chunk that needs three sweeps among others that need two costs more than all of them with three: back after one chunk,
// beta about 0.95 without retention took 4.22 us a chunk, with every verdict waited for 3.75, as it is 3.24.)  With retention a
// chunk whose coordinates the box holds at every token has sigma = 0: no sweep (gates of 0.97: 2.5 -> 1.7).
//
// Bound by the issue of one CU's vector instructions (two wavefronts per SIMD) and the latency of its two
// barriers.  Chains of 64 chunks of 128 coordinates, bf16, us per chunk: no retention 3.43 -> 2.43, one gate per head
// 2.97 -> 2.45, per coordinate 3.26 -> 2.99 against three barriers a sweep, one coordinate and 16 tokens per thread,
// and results stored behind the next chunk's loads; with three sweeps 4.19 -> 3.24, 3.70 -> 3.29, 3.89 -> 3.75.
//
// PIECES: for few long chains the chain is cut into pieces, one workgroup each, as in the forward kernel: every
// piece is swept from a guess of the adjoint at its right end, and the sweeps over all pieces repeat until
// no such value of the chain moves.  A piece that began at x and ended at y is left as the map
//     x' -> y + P (x' - x - g <g, x' - x> / <1, g>),
// P per coordinate, g = sum over the piece's tokens of ca_t <1, s_t> s_t:
// exact where nothing moved, and as good as the sweeps need it elsewhere.  The term in g is the coupling of the
// coordinates along (1, .., 1), which is nearly all of it (sum ca_t s_t s_t^T = g g^T / <1, g> for equal keys); one gate per token
// multiplies it as it does the rest.  How many sweeps it takes goes by how much the gates fade, and without the term in g also by
// eta and beta (16 chains of 128 chunks, K = 64, gates of 1, beta about 0.95: more than the limit, 900 us; 350 with it).
// With gates of 0.999 two sweeps do and a third finds that nothing moved, with 0.9999 or 1 three to five (16 chains, K = V = 128,
// backward pass against segments: 128 chunks 567 and 437 us, with gates of 1 571 and 503; 512 1927 and 1602, 1954 and 1802).
template <typename T, int K, int RET, bool PIECES, bool RAG>
__global__ __launch_bounds__(P1F) void precond_chain_kernel(PrecondBwdArgs a) {
    static_assert(!PIECES || RET != 0, "without retention a chain is not cut");
    constexpr bool HAS_RET = RET != 0, RET_VEC = RET == 2;
    constexpr int CPT = K / 64;                  // coordinates per thread (adjacent)
    constexpr int NRUN = C / RUN;                // = wavefronts of the workgroup
    typedef Pack<T, CPT> Pk;
    typedef Pack<float, CPT> Pr;
    __shared__ __attribute__((aligned(16))) float mapP[2][NRUN * K];     // chunks in turn
    __shared__ __attribute__((aligned(16))) float mapL[3][NRUN * K];     // 0: of sigma = 0; 1, 2: of later sweeps, in turn
    __shared__ __attribute__((aligned(16))) float wmax[2][2 * NRUN];           // per wavefront: largest change of sigma, largest sigma
    // per wavefront: 1: the chunk before has not settled, 2: nor would it have in two sweeps; 4: some coordinate of this chunk is
    // not held by the box throughout
    __shared__ __attribute__((aligned(16))) int flags[NRUN];

    const int tid = threadIdx.x, run = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int c0 = lane * CPT;                   // first coordinate of this thread
    const int u_own = fold_token(lane);          // the token of the run whose scalars this lane keeps
    const int piece = PIECES ? blockIdx.x % a.pieces : 0;
    const int chain = PIECES ? blockIdx.x / a.pieces : blockIdx.x;
    const int h = chain % a.H;
    int b = chain / a.H;                                      // batch entry, or packed sequence
    if (a.settled && !(PIECES && a.sweep == 0) && a.settled[chain]) return;
    if (PIECES) {
        a.n0 += piece * a.piece_chunks;
        a.n1 = min(a.n1, a.n0 + a.piece_chunks);
        if (a.n0 >= a.n1) return;
    }
    int bt = b;                                               // batch entry of the token tensors
    if (a.seq_chunks) {
        b = sequence_of(a.seq_chunks, a.n_seqs, b);
        bool begins, ends;
        if (!clip_to_sequence(a.seq_chunks, b, a.n0, a.n1, begins, ends)) return;
        a.dd_out = ends ? a.dd_last : a.dd_in;
        bt = 0;
    }
    const size_t bh = (size_t)b * a.H + h;                    // the chain: indexes dd_out / dd_in
    const size_t bth = (size_t)bt * a.H + h;                  // indexes the per-chunk buffers
    const bool project = a.d_min <= a.d_max;
    const int N = a.T / C;
    const uint32_t kstride = (uint32_t)a.H * K;               // elements between consecutive tokens
    const ChainIn<T, K, RET, RAG> in(a, b, a.n0, h);

    float ga[CPT];                               // adjoint of d at the right end of the chunk (the same in every wavefront)
#pragma unroll
    for (int e = 0; e < CPT; ++e) ga[e] = a.dd_out ? a.dd_out[bh * K + c0 + e] : 0.f;

    auto put_map = [&](float *m, const float (&v)[CPT]) {
        *reinterpret_cast<typename Pr::Raw *>(m + run * K + c0) = Pr::pack(v);
    };
    auto get_map = [&](const float *m, int j, float (&v)[CPT]) {
        Pr::unpack(*reinterpret_cast<const typename Pr::Raw *>(m + j * K + c0), v);
    };
    float PP[CPT], gacc[PIECES ? CPT : 1] = {}, start[CPT];  // the piece so far: P, g; where it began
    if (PIECES) {
        // The adjoint at this piece's right end: the chain's own carried through the maps that the sweep before left
        // (first sweep: the chain's own, as a guess).  Every workgroup of a chain walks all its pieces and so sees
        // whether any of those values moved; if none did, what the sweep before wrote stands.
        const size_t buf = (size_t)gridDim.x * K;
        const float4 *prev = a.piece_map + ((a.sweep & 1) ? 0 : buf) + bh * a.pieces * K;
        if (run == 0) {
            float x[CPT], xs[CPT];
            bool moved = a.sweep == 0;
#pragma unroll
            for (int e = 0; e < CPT; ++e) x[e] = xs[e] = ga[e];
            // (WALK records at a time, asked for together: as in the forward kernel)
            constexpr int WALK = 8;
            for (int q0 = a.sweep > 0 ? a.pieces - 1 : -1; q0 >= 0; q0 -= WALK) {
                float4 m[WALK][CPT];
#pragma unroll
                for (int j = 0; j < WALK; ++j)
#pragma unroll
                    for (int e = 0; e < CPT; ++e) m[j][e] = prev[(size_t)max(q0 - j, 0) * K + c0 + e];
#pragma unroll
                for (int j = 0; j < WALK; ++j) {
                    if (q0 - j < 0) break;
                    float dx[CPT], dot = 0.f, big = 0.f;
#pragma unroll
                    for (int e = 0; e < CPT; ++e) {
                        if (q0 - j == piece) { xs[e] = x[e]; gacc[PIECES ? e : 0] = m[j][e].w; }
                        dx[e] = x[e] - m[j][e].x;
                        big = fmaxf(big, fabsf(x[e]));
                        dot = __builtin_fmaf(m[j][e].w, dx[e], dot);
                    }
                    big = wave_max(big);
#pragma unroll
                    for (int e = 0; e < CPT; ++e) moved = moved || !(fabsf(dx[e]) <= PIECE_TOL_BWD * big);   // (not a number: moved)
                    dot = wave_sum(dot);
#pragma unroll
                    for (int e = 0; e < CPT; ++e) dx[e] = __builtin_fmaf(-dot, m[j][e].w, dx[e]);
#pragma unroll
                    for (int e = 0; e < CPT; ++e) x[e] = __builtin_fmaf(m[j][e].z, dx[e], m[j][e].y);
                }
            }
            if (__any(moved)) moved = true;
            if (lane == 0) flags[0] = moved ? 1 : 0;
            put_map(mapL[0], xs);
        }
        __syncthreads();
        const int any = flags[0];
        if (piece == 0 && tid == 0) a.settled[chain] = any ? 0 : 1;
        if (!any) return;
        get_map(mapL[0], 0, ga);
        __syncthreads();
#pragma unroll
        for (int e = 0; e < CPT; ++e) { PP[e] = 1.f; start[e] = ga[e]; }
        a.piece_map += (a.sweep & 1) ? buf : 0;
    }

    typename Pk::Raw kreg[RUN], greg[RUN];       // this thread's k and dL/dk~ of the next chunk
    typename Pr::Raw rreg[RET_VEC ? RUN : 1];    // ... its per-coordinate retention
    uint32_t mreg[CPT];                          // ... half of its mask bits
    float nrawreg = 1.f, betreg = 0.f, retreg = 1.f;          // ... and the scalars of token (run, u_own)
    // (per-chunk buffers, like the caller's rows, lie a constant step apart from chunk to chunk)
    const T *const gc = static_cast<const T *>(a.dkt) + (((size_t)bt * N * a.H + h) * C + run * RUN) * K;
    float *const tc = a.tok_scalars + ((size_t)bt * a.T * a.H + h) * 4;
    const uint32_t *const mc = reinterpret_cast<const uint32_t *>(a.masks + bth * N * K) + run / (32 / RUN);
    float *const ac = a.a_ckpt + bth * N * K;
#define OSDN_P1_BLOAD(n_)                                                                        \
    {                                                                                            \
        const size_t off_ = (size_t)(n_) * in.chunk_rows;                                        \
        const int fl_ = fresh_lane(lane);                                                        \
        const T *kp_ = in.k_of(n_) + (uint32_t)(run * RUN) * kstride, *gp_ = gc + off_ * K;      \
        const float *rp_ = HAS_RET ? in.ret_of(n_) : nullptr;                                    \
        _Pragma("unroll") for (int u = 0; u < RUN; ++u) {                                        \
            kreg[u] = row_elem(reinterpret_cast<const typename Pk::Raw *>(kp_ + (size_t)u * kstride), fl_); \
            greg[u] = row_elem(reinterpret_cast<const typename Pk::Raw *>(gp_ + u * K), fl_);    \
            if (RET_VEC)                                                                         \
                rreg[RET_VEC ? u : 0] = row_elem(reinterpret_cast<const typename Pr::Raw *>(     \
                    rp_ + (size_t)(run * RUN + u) * kstride), fl_);                              \
        }                                                                                        \
        _Pragma("unroll") for (int e = 0; e < CPT; ++e) mreg[e] = lane_elem(mc + (size_t)(n_) * K * 2, (c0 + e) * 2); \
        const int i_ = (run * RUN + u_own) * a.H;                                                \
        nrawreg = lane_elem(tc + off_ * 4 + 2, i_ * 4);                                          \
        betreg = lane_elem(in.beta_of(n_), i_);                                                  \
        if (HAS_RET && !RET_VEC) retreg = lane_elem(rp_, i_);                                    \
    }
    // The adjoint g of the chunk's right end carried to the right end of this run (returned in at) and, if
    // OUT, on to the chunk's left end (in g).  The run is the same for the whole wavefront: scalar branches.
    auto carry = [&](auto out, const float *mP, const float *mL, float (&g)[CPT], float (&at)[CPT]) {
        constexpr bool OUT = decltype(out)::value;
        float P[NRUN][CPT], L[NRUN][CPT];
        int r = run;
        asm volatile("" : "+s"(r));              // (compared here: eight conditions kept for the whole kernel would spill)
#pragma unroll
        for (int j = NRUN - 1; j >= (OUT ? 0 : 1); --j) { get_map(mP, j, P[j]); get_map(mL, j, L[j]); }
        float x[CPT];
#pragma unroll
        for (int e = 0; e < CPT; ++e) x[e] = g[e];
#pragma unroll
        for (int j = NRUN - 1; j >= 0; --j) {
            if (j == r) {
#pragma unroll
                for (int e = 0; e < CPT; ++e) at[e] = x[e];
                if (!OUT) return;
            }
            if (!OUT && j == 0) return;
#pragma unroll
            for (int e = 0; e < CPT; ++e) x[e] = __builtin_fmaf(P[j][e], x[e], L[j][e]);
        }
#pragma unroll
        for (int e = 0; e < CPT; ++e) {
            g[e] = x[e];
            if (PIECES) {
#pragma unroll
                for (int j = 0; j < NRUN; ++j) PP[e] *= P[j][e];
            }
        }
    };
    // (largest of values >= 0, compared as their bit patterns)
    auto max8 = [](const float *v) {
        typedef __attribute__((__vector_size__(16))) uint32_t U;
        const U x = *reinterpret_cast<const U *>(v), y = *reinterpret_cast<const U *>(v + 4);
        uint32_t m = 0u;
#pragma unroll
        for (int i = 0; i < 4; ++i) m = max(m, max(x[i], y[i]));
        return __builtin_bit_cast(float, m);
    };
    // P1_TOL_BWD to the 1/2 and 2/3: a second (third) sweep that moved sigma by this share of what the first one did (from
    // zero) settles it, with differences that shrink by one ratio
    constexpr float SECOND_OK = 3.16e-4f, THIRD_OK = 2.15e-5f;
    constexpr int CALM = 8;                      // chunks in a row that needed less before less is tried again

    OSDN_P1_BLOAD(a.n1 - 1)
    // what the next pass stores: chunk, adjoint at its right end, sigma (at first nothing to keep: stored again by the second pass)
    int done = a.n1 - 1;
    float gdone[CPT], sdone = 0.f, PPdone[PIECES ? CPT : 1] = {};
#pragma unroll
    for (int e = 0; e < CPT; ++e) gdone[e] = ga[e];
    // Sweeps of a chunk whose verdict waits for the next chunk's maps: two (three: deep).  Careful: as many as it takes, with a
    // barrier for every verdict.  pending: the chunk before awaits its verdict; again: it is done once more
    bool deep = false, careful = false, pending = false, refetch = false, again = false;
    int calm = 0, verdict = 0;
    for (int n = a.n1 - 1;; --n) {
        // ---- this thread's s = k^2, lambda = k . dL/dk~, masks and retention (past the end: of the last chunk, in vain) ----
        float sv[RUN][CPT], lam[RUN][CPT], rv[RUN][RET_VEC ? CPT : 1];
        uint32_t mb[CPT];
#pragma unroll
        for (int e = 0; e < CPT; ++e) mb[e] = project ? mreg[e] >> (run % (32 / RUN) * RUN) & ((1u << RUN) - 1) : (1u << RUN) - 1;
#pragma unroll
        for (int u = 0; u < RUN; ++u) {
            float kf[CPT], gf[CPT];
            Pk::unpack(kreg[u], kf);
            Pk::unpack(greg[u], gf);
#pragma unroll
            for (int e = 0; e < CPT; ++e) {
                sv[u][e] = kf[e] * kf[e];
                lam[u][e] = kf[e] * gf[e];
            }
            if constexpr (RET_VEC) Pr::unpack(rreg[RET_VEC ? u : 0], rv[u]);
            else rv[u][0] = HAS_RET ? lane_bcast(retreg, fold_lane(u)) : 1.f;
        }
        bool whole = true;
#pragma unroll
        for (int e = 0; e < CPT; ++e) whole = whole && mb[e] == (1u << RUN) - 1;
        const bool clean = __all(whole);            // no coordinate of this wavefront met the box in its run
        float ca, cn = 0.f;
        {
            const float nn = fmaxf(fabsf(nrawreg), a.eps), bp = a.beta_aware ? betreg : 1.f;
            ca = a.eta * bp / nn * bp;
            if (PIECES) cn = ca * nrawreg;
        }
        // (all that was loaded has been used when its registers are refilled: else the loop's end copies them, and waits)
        asm volatile("" : "+v"(ca), "+v"(cn));
        if constexpr (RET == 1) {
#pragma unroll
            for (int u = 0; u < RUN; ++u) asm volatile("" : "+s"(rv[u][0]));
        }
#pragma unroll
        for (int e = 0; e < CPT; ++e) {
            asm volatile("" : "+v"(mb[e]));
#pragma unroll
            for (int u = 0; u < RUN; ++u) {
                asm volatile("" : "+v"(sv[u][e]), "+v"(lam[u][e]));
                if constexpr (RET_VEC) asm volatile("" : "+v"(rv[u][e]));
            }
        }
        // the results of the chunk before, ahead of the loads: behind them, the wait for the loads would be one for
        // these stores too (every wavefront stores the same adjoint, eight lanes the same sigma)
        lane_elem(reinterpret_cast<typename Pr::Raw *>(ac + (size_t)done * K), lane) = Pr::pack(gdone);
        lane_elem(tc + (size_t)done * in.chunk_rows * 4 + 3, (run * RUN + u_own) * a.H * 4) = sdone;
        OSDN_P1_BLOAD(max(n - 1, a.n0))
        int mk[RUN][CPT];                        // all ones where the projection of the token lets the coordinate pass
#pragma unroll
        for (int u = 0; u < RUN; ++u)
#pragma unroll
            for (int e = 0; e < CPT; ++e) {
                mk[u][e] = (int)(mb[e] << (31 - u)) >> 31;
                asm volatile("" : "+v"(mk[u][e]));       // (formed once, not at every use)
            }
        auto through = [&](float x, int u, int e) { return __builtin_bit_cast(float, __builtin_bit_cast(int, x) & mk[u][e]); };
        // the run's L for lambda - ca sigma s = src
        auto compose = [&](const float (&src)[RUN][CPT], float *m) {
            float L[CPT];
#pragma unroll
            for (int e = 0; e < CPT; ++e) {
                float x = src[RUN - 1][e];
                if (clean) {
#pragma unroll
                    for (int u = RUN - 2; u >= 0; --u) x = HAS_RET ? __builtin_fmaf(rv[u][RET_VEC ? e : 0], x, src[u][e]) : x + src[u][e];
                } else {
#pragma unroll
                    for (int u = RUN - 2; u >= 0; --u) {
                        const float t = through(x, u, e);
                        x = HAS_RET ? __builtin_fmaf(rv[u][RET_VEC ? e : 0], t, src[u][e]) : t + src[u][e];
                    }
                }
                L[e] = x;
            }
            put_map(m, L);
        };
        float P[CPT];
#pragma unroll
        for (int e = 0; e < CPT; ++e) {
            float x = rv[0][0];
            if (HAS_RET) {
                x = rv[0][RET_VEC ? e : 0];
#pragma unroll
                for (int u = 1; u < RUN; ++u) x *= rv[u][RET_VEC ? e : 0];
            }
            P[e] = mb[e] == (1u << RUN) - 1 ? x : 0.f;
        }
        float *const mP = mapP[n & 1];
        put_map(mP, P);
        {
            uint32_t some = mb[0];
#pragma unroll
            for (int e = 1; e < CPT; ++e) some |= mb[e];
            if (!HAS_RET || __any(some != 0u)) verdict |= 4;
            if (lane == 0) flags[run] = verdict;
        }
        compose(lam, mapL[0]);
        __syncthreads();
        int all;
        {
            typedef __attribute__((__vector_size__(16))) int I;
            const I x = *reinterpret_cast<const I *>(flags) | *reinterpret_cast<const I *>(flags + 4);
            all = __builtin_amdgcn_readfirstlane(x[0] | x[1] | x[2] | x[3]);
        }
        verdict = 0;
        if (pending) {
            pending = false;
            calm = all & 2 ? 0 : calm + 1;
            if (all & 1) {                       // (uniform) the chunk before, once more from the same adjoint
                careful = deep;
                deep = refetch = again = true;
                calm = 0;
                n += 3;                          // (the next pass only fetches chunk n + 1)
#pragma unroll
                for (int e = 0; e < CPT; ++e) {
                    ga[e] = gdone[e];
                    if (PIECES) PP[e] = PPdone[PIECES ? e : 0];
                }
                __syncthreads();                 // (the flags have been read)
                continue;
            }
            if (calm >= CALM) deep = false;
        }
        if (refetch) {
            refetch = false;
            continue;
        }
        if (n < a.n0) break;
#pragma unroll
        for (int e = 0; e < CPT; ++e) {
            gdone[e] = ga[e];
            if (PIECES) PPdone[PIECES ? e : 0] = PP[e];
        }
        if (PIECES && a.sweep == 0 && !again) {
#pragma unroll
            for (int u = 0; u < RUN; ++u) {
                const float c = lane_bcast(cn, fold_lane(u));
#pragma unroll
                for (int e = 0; e < CPT; ++e) gacc[PIECES ? e : 0] = __builtin_fmaf(c, sv[u][e], gacc[PIECES ? e : 0]);
            }
        }
        again = false;
        if (HAS_RET && !(all & 4)) {                 // the box holds every coordinate at every token: sigma is zero
            float at[CPT];
            carry(std::true_type{}, mP, mapL[0], ga, at);
            sdone = 0.f;
            done = n;
            __syncthreads();                     // (maps and flags have been read)
            continue;
        }
        // the tokens of the run replayed from the adjoint x at its right end: their sigma
        auto replay = [&](const float (&at)[CPT], const float (&src)[RUN][CPT]) {
            float vp[RUN];
#pragma unroll
            for (int e = 0; e < CPT; ++e) {
                float x = at[e];
                if (clean) {
#pragma unroll
                    for (int u = RUN - 1; u >= 0; --u) {
                        vp[u] = e == 0 ? sv[u][e] * x : __builtin_fmaf(sv[u][e], x, vp[u]);
                        x = HAS_RET ? __builtin_fmaf(rv[u][RET_VEC ? e : 0], x, src[u][e]) : x + src[u][e];
                    }
                } else {
#pragma unroll
                    for (int u = RUN - 1; u >= 0; --u) {
                        const float t = through(x, u, e);
                        vp[u] = e == 0 ? sv[u][e] * t : __builtin_fmaf(sv[u][e], t, vp[u]);
                        x = HAS_RET ? __builtin_fmaf(rv[u][RET_VEC ? e : 0], t, src[u][e]) : t + src[u][e];
                    }
                }
            }
            return fold_tokens(vp);
        };
        float src[RUN][CPT];
        auto sources = [&](float sigma) {
            const float cs = ca * sigma;
#pragma unroll
            for (int u = 0; u < RUN; ++u) {
                const float c = -lane_bcast(cs, fold_lane(u));
#pragma unroll
                for (int e = 0; e < CPT; ++e) src[u][e] = __builtin_fmaf(c, sv[u][e], lam[u][e]);
            }
        };
        float at[CPT];
        carry(std::false_type{}, mP, mapL[0], ga, at);
        float sig0 = replay(at, lam);
        // in lane 63, the largest |x| of the wavefront (a lane holds one of eight tokens, by its upper three bits; what is not a
        // number is left out: it has no say in whether the others have settled)
        auto largest = [](float x) {
            uint32_t m = __builtin_bit_cast(uint32_t, fmaxf(fabsf(x), 0.f));
            m = max(m, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)m, 0x128, 0xF, 0xF, true));       // row_ror:8
            m = max(m, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)m, 0x142, 0xA, 0xF, false));      // row_bcast:15
            m = max(m, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)m, 0x143, 0xC, 0xF, false));      // row_bcast:31
            return __builtin_bit_cast(float, m);
        };
        {
            const float m = largest(sig0);
            if (lane == 63) wmax[0][NRUN + run] = m;
        }
        sources(sig0);
        compose(src, mapL[1]);
        __syncthreads();
        const float first = max8(wmax[0] + NRUN);
        carry(std::true_type{}, mP, mapL[1], ga, at);
        float sig = replay(at, src);
        if (!careful) {
            verdict = __any(fabsf(sig - sig0) > SECOND_OK * first) ? 3 : 0;
            if (deep) {
                sources(sig);
                compose(src, mapL[2]);
                __syncthreads();
                sig0 = sig;
#pragma unroll
                for (int e = 0; e < CPT; ++e) {
                    ga[e] = gdone[e];
                    if (PIECES) PP[e] = PPdone[PIECES ? e : 0];
                }
                carry(std::true_type{}, mP, mapL[2], ga, at);
                sig = replay(at, src);
                verdict = (verdict & 2) | (__any(fabsf(sig - sig0) > THIRD_OK * first) ? 1 : 0);
            }
            pending = true;
        } else {
            float dprev = first;
            int sweeps = 2, buf = 2, row = 1;
            for (;;) {
                const float d = largest(sig - sig0), x = largest(sig);
                if (lane == 63) { wmax[row][run] = d; wmax[row][NRUN + run] = x; }
                sources(sig);
                compose(src, mapL[buf]);
                __syncthreads();
                const float dcur = max8(wmax[row]), mx = max8(wmax[row] + NRUN);
                // converged, or the observed contraction ratio says that the next difference would be below the tolerance
                if (dcur <= P1_TOL_BWD * mx || (dcur <= 0.1f * dprev && dcur * dcur <= P1_TOL_BWD * mx * dprev) || sweeps >= P1_MAX_SWEEPS) break;
                dprev = dcur;
                sig0 = sig;
#pragma unroll
                for (int e = 0; e < CPT; ++e) {
                    ga[e] = gdone[e];
                    if (PIECES) PP[e] = PPdone[PIECES ? e : 0];
                }
                carry(std::true_type{}, mP, mapL[buf], ga, at);
                sig = replay(at, src);
                buf = 3 - buf;
                row ^= 1;
                ++sweeps;
            }
            calm = sweeps > 3 ? 0 : calm + 1;
            if (calm >= CALM) {
                careful = false;
                calm = 0;
            }
        }
        sdone = sig;
        done = n;
    }
    if (PIECES && a.sweep == 0) {                // g of the piece, the sum over its runs, over sqrt(<1, g>) (the same for every sweep)
        float v[CPT];
#pragma unroll
        for (int e = 0; e < CPT; ++e) v[e] = gacc[PIECES ? e : 0];
        __syncthreads();
        put_map(mapL[0], v);
        __syncthreads();
#pragma unroll
        for (int e = 0; e < CPT; ++e) gacc[PIECES ? e : 0] = 0.f;
#pragma unroll
        for (int j = 0; j < NRUN; ++j) {
            get_map(mapL[0], j, v);
#pragma unroll
            for (int e = 0; e < CPT; ++e) gacc[PIECES ? e : 0] += v[e];
        }
        float sum = 0.f;
#pragma unroll
        for (int e = 0; e < CPT; ++e) sum += gacc[PIECES ? e : 0];
        sum = wave_sum(sum);
        const float r = sum > 0.f ? rsqrtf(sum) : 0.f;
#pragma unroll
        for (int e = 0; e < CPT; ++e) gacc[PIECES ? e : 0] *= r;
    }
    if (run == 0) {
#pragma unroll
        for (int e = 0; e < CPT; ++e) {
            if (!PIECES || piece == 0) a.dd_in[bh * K + c0 + e] = ga[e];
            if (PIECES) a.piece_map[(bh * a.pieces + piece) * K + c0 + e] = make_float4(start[e], ga[e], PP[e], gacc[PIECES ? e : 0]);
        }
    }
#undef OSDN_P1_BLOAD
}

// --------------------------------------------------------------- precond_chain_lin ----
// The chain where chunks that qualify take the solved form (no retention; see the top of this file).  Any
// other chunk is swept: NSEG = 512 / K runs of TS tokens, one coordinate of one run per thread, abar_i kept as
// L_i + P_i * carry; the runs are chained through LDS, the products s_i abar_i folded over the lanes, three
// barriers a sweep.  Which calls come here goes by sizes alone, not by d: with the default box such chunks are few, also where
// the d that is carried in lies on a face, which it leaves within the chunk (16 chains of 64 chunks of 128 coordinates, backward
// pass: 273 us, from d = d_max 276); a box so narrow that d keeps meeting it makes every chunk one of them.
template <typename T, int K, bool RAG>
__global__ __launch_bounds__(P1T) void precond_chain_lin_kernel(PrecondBwdArgs a) {
    constexpr int NSEG = P1T / K;                 // runs per chunk
    constexpr int TS = C / NSEG;                  // tokens per run
    constexpr int WPS = K / 64;                   // wavefronts per run
    constexpr int NPART = K / TS;                 // partial sums per token
    __shared__ float ga[K];                      // adjoint of d at the right end of the chunk
    __shared__ float segL[NSEG * K], segP[NSEG * K];
    __shared__ float cas[C], sig[C];
    __shared__ __attribute__((aligned(16))) float casig[C];
    __shared__ float part[P1W * 64];
    __shared__ int done;
    // chunks in solved form (see the top of this file)
    typedef Lin<K> LN;
    constexpr int EPT = LN::EPT, VN = 16 / sizeof(T), NVK = EPT / VN, NG = LN::NG;
    __shared__ __attribute__((aligned(16))) float Sl[C * LN::LD];       // s = k^2 of the chunk
    __shared__ __attribute__((aligned(16))) float gp[8 * LN::VSTR];     // copy of ga, sliced per thread of the row layout
    __shared__ __attribute__((aligned(16))) float xs[8 * LN::XSTR];     // S g + rho0
    __shared__ float ws[C];                                             // ca (.) sigma

    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int c = tid % K, sg = tid / K;          // coordinate and run of this thread
    const int li = tid >> 3, lpart = tid & 7;     // row layout of the solved form: token, slice
    const int lc = tid / NG, ltg = tid % NG;      // column layout: coordinate, token group
    const int h = blockIdx.x % a.H;
    int b = blockIdx.x / a.H;                                 // batch entry, or packed sequence
    int bt = b;                                               // batch entry of the token tensors
    if (a.seq_chunks) {
        b = sequence_of(a.seq_chunks, a.n_seqs, b);
        bool begins, ends;
        if (!clip_to_sequence(a.seq_chunks, b, a.n0, a.n1, begins, ends)) return;
        a.dd_out = ends ? a.dd_last : a.dd_in;
        bt = 0;
    }
    const size_t bh = (size_t)b * a.H + h;                    // the chain: indexes dd_out / dd_in
    const size_t bth = (size_t)bt * a.H + h;                  // indexes the per-chunk buffers
    const bool project = a.d_min <= a.d_max;
    const int N = a.T / C;
    const uint32_t kstride = (uint32_t)a.H * K;   // elements between consecutive tokens
    const ChainIn<T, K, 0, RAG> src(a, b, a.n0, h);

    if (tid < K) {
        const float g0 = a.dd_out ? a.dd_out[bh * K + tid] : 0.f;
        ga[tid] = g0;
        gp[LN::vidx(tid)] = g0;
    }

    T kreg[TS], greg[TS];
    float nrawreg = 1.f, betreg = 0.f;
    uint2 mreg = make_uint2(0xffffffffu, 0xffffffffu);
#define OSDN_P1_BLOAD(n_)                                                                        \
    {                                                                                            \
        const size_t tokc_ = ((size_t)bt * a.T + (size_t)(n_) * C) * a.H + h;                    \
        const T *kp_ = src.k_of(n_);                                                             \
        const T *gp_ = static_cast<const T *>(a.dkt) + (((size_t)bt * N + (n_)) * a.H + h) * C * K; \
        uint32_t ok_ = (uint32_t)(sg * TS) * kstride + (uint32_t)c, og_ = (uint32_t)(sg * TS * K + c); \
        asm volatile("" : "+v"(ok_), "+v"(og_));             /* (seldom run: no addresses kept for it) */ \
        _Pragma("unroll") for (int u = 0; u < TS; ++u) {                                         \
            const uint32_t o_ = ok_ + (uint32_t)u * kstride;                                     \
            kreg[u] = lane_elem(kp_, o_); greg[u] = lane_elem(gp_, og_ + u * K);                 \
        }                                                                                        \
        if (tid < C) {                                                                           \
            const size_t th = tokc_ + (size_t)tid * a.H;                                         \
            nrawreg = a.tok_scalars[th * 4 + 2];                                                 \
            betreg = src.beta_of(n_)[(size_t)tid * a.H];                                         \
        }                                                                                        \
        if (project) mreg = a.masks[(bth * N + (n_)) * K + c];                                   \
    }
    // Registers of a chunk in solved form: the thread's slice of its key row and of its row of
    // the inverse, the token's scalars (slice 0 only), the coordinate's sum of lambda (group 0 only).
    struct LinRegs {
        u32x4 kq[NVK];
        u32x4 mq[8 * sizeof(T) / 16];
        float rho, nraw, beta, t0;
    };
#define OSDN_P1_LLOAD(n_, R)                                                                     \
    {                                                                                            \
        __builtin_amdgcn_sched_barrier(0);     /* the sets are requested in program order */     \
        const size_t tokc_ = ((size_t)bt * a.T + (size_t)(n_) * C) * a.H + h;                    \
        const size_t bhn_ = bth * N + (n_);                                                      \
        const uint32_t off_ = ((uint32_t)li * kstride + (uint32_t)(lpart * EPT)) * (uint32_t)sizeof(T); \
        const u32x4 *kp_ = reinterpret_cast<const u32x4 *>(src.k_of(n_));                        \
        _Pragma("unroll") for (int m_ = 0; m_ < NVK; ++m_) R.kq[m_] = at_byte(kp_, off_ + 16 * m_); \
        const u32x4 *mp_ = reinterpret_cast<const u32x4 *>(static_cast<const T *>(a.lin_M) + bhn_ * C * C + li * C + lpart * 8); \
        _Pragma("unroll") for (int m_ = 0; m_ < (int)(8 * sizeof(T) / 16); ++m_) R.mq[m_] = mp_[m_]; \
        const size_t th = tokc_ + (size_t)li * a.H;      /* (every lane of a token loads its scalars) */ \
        R.nraw = a.tok_scalars[th * 4 + 2];                                                      \
        R.beta = src.beta_of(n_)[(size_t)li * a.H];                                              \
        R.rho = a.lin_r0[bhn_ * C + li];                                                         \
        R.t0 = a.lin_t0[bhn_ * K + lc];                                                          \
        __builtin_amdgcn_sched_barrier(0);                                                       \
    }
    // One chunk in solved form from the registers R (a step outside the run [m_lo, n_hi] does
    // nothing but the refill); when they have been read, they are refilled with the chunk three
    // further on (clamped to the run: past its end a harmless reload of its last chunk).  No load or store of the step sits under a branch, and lanes that hold the
    // same value all store it: the loads of the other two register sets then stay in flight
    // across the step (behind a branch the compiler can no longer count what is outstanding and
    // waits for everything).
#define OSDN_P1_LSTEP(n_, R, m_lo, n_hi)                                                         \
    {                                                                                            \
        const bool act_ = (n_) <= (n_hi) && (n_) >= (m_lo);       /* uniform */                  \
        float pre_ = 0.f;                                                                        \
        if (act_) {                                                                              \
        const size_t tokc_s = ((size_t)bt * a.T + (size_t)(n_) * C) * a.H + h;                   \
        a.a_ckpt[(bth * N + (n_)) * K + c] = ga[c];                                              \
        /* x = S g + rho0, and the s tile into LDS for the product with S^T */                   \
        float y = 0.f;                                                                           \
        _Pragma("unroll") for (int m_ = 0; m_ < NVK; ++m_)                                       \
            _Pragma("unroll") for (int e4 = 0; e4 < VN; e4 += 4) {                               \
                const f32x4 gv = *reinterpret_cast<const f32x4 *>(gp + lpart * LN::VSTR + m_ * VN + e4); \
                float sq[4];                                                                     \
                _Pragma("unroll") for (int e = 0; e < 4; ++e) {                                  \
                    const float kf = vec_get<T>(R.kq[m_], e4 + e);                               \
                    sq[e] = kf * kf;                                                             \
                    y = __builtin_fmaf(sq[e], gv[e], y);                                         \
                }                                                                                \
                store_vec(Sl + li * LN::LD + LN::swz(lpart * EPT + m_ * VN + e4), sq);                    \
            }                                                                                    \
        y = sum_lanes8(y);                                                                       \
        const float nn_ = fmaxf(fabsf(R.nraw), a.eps);                                                  \
        const float bp_ = a.beta_aware ? R.beta : 1.f;                                           \
        const float ca_i = a.eta * bp_ / nn_ * bp_;                                              \
        xs[LN::xidx(li)] = y + R.rho;                                                            \
        __syncthreads();                                                                         \
        /* sigma = (I + U)^-1 x */                                                               \
        float sgm = 0.f;                                                                         \
        _Pragma("unroll") for (int h4 = 0; h4 < 2; ++h4) {                                       \
            const f32x4 xv = *reinterpret_cast<const f32x4 *>(xs + lpart * LN::XSTR + 4 * h4);   \
            _Pragma("unroll") for (int e = 0; e < 4; ++e)                                        \
                sgm = __builtin_fmaf(vec_get<T>(R.mq[(4 * h4 + e) / VN], (4 * h4 + e) % VN), xv[e], sgm); \
        }                                                                                        \
        sgm = sum_lanes8(sgm);                                                                   \
        ws[li] = ca_i * sgm;                                                                     \
        a.tok_scalars[(tokc_s + (size_t)li * a.H) * 4 + 3] = sgm;                                \
        pre_ = ga[lc] + R.t0;                   /* (no loaded value is kept past the refill, */  \
        asm volatile("" : "+v"(pre_));          /*  and this sum is not moved behind it)     */  \
        }                                                                                        \
        OSDN_P1_LLOAD(min(max((n_) - 3, (m_lo)), (n_hi)), R)                                     \
        if (act_) {                                                                              \
        __syncthreads();                                                                         \
        /* a_left = g + sum lambda - S^T (ca (.) sigma) */                                       \
        float acc_ = 0.f;                                                                        \
        _Pragma("unroll") for (int u = 0; u < C / NG; ++u)                                       \
            acc_ = __builtin_fmaf(Sl[(u * NG + ltg) * LN::LD + LN::swz(lc)], ws[u * NG + ltg], acc_);     \
        acc_ = NG == 4 ? sum_lanes4(acc_) : sum_lanes8(acc_);                                    \
        const float gn = pre_ - acc_;                                                            \
        ga[lc] = gn;                                                                             \
        gp[LN::vidx(lc)] = gn;                                                                   \
        __syncthreads();                                                                         \
        }                                                                                        \
    }
    // Which chunks take the solved form: the flags precond_lin left, as bits in LDS (bit n - n0;
    // chunks past the table's reach sweep).  Only the solved form prefetches (three
    // chunks deep, inside a run of such chunks); a chunk that has to sweep fetches its operands
    // when it starts: keeping both sets of registers alive across the loop would spill.
    constexpr int FLAG_WORDS = 512;
    __shared__ uint32_t flagw[FLAG_WORDS];
    {
        for (int base = 0; base < a.n1 - a.n0 && base < FLAG_WORDS * 32; base += P1T) {
            const int nn = a.n0 + base + tid;
            const int f = nn < a.n1 ? a.lin_clean[bth * N + nn] : 0;
            const unsigned long long bits = __ballot(f != 0);
            if (lane == 0) {
                flagw[(base >> 5) + 2 * wave] = (uint32_t)bits;
                flagw[(base >> 5) + 2 * wave + 1] = (uint32_t)(bits >> 32);
            }
        }
    }
    __syncthreads();
    auto solved = [&](int nn) -> bool {            // uniform
        const int r = nn - a.n0;
        return r < FLAG_WORDS * 32 && ((flagw[r >> 5] >> (r & 31)) & 1u) != 0;
    };

    for (int n = a.n1 - 1; n >= a.n0; --n) {
        const size_t tokc = ((size_t)bt * a.T + (size_t)n * C) * a.H + h;
        if (solved(n)) {
            // the run [m, n] of chunks in solved form, three chunks in flight
            int m = n;
            while (m > a.n0 && solved(m - 1)) --m;
            // (the first three steps only request operands: with nothing requested ahead of the
            // loop, the compiler's count of what is outstanding at the top of the loop is exact)
            LinRegs r0, r1, r2;
            for (int j = n + 3; j >= m; j -= 3) {
                OSDN_P1_LSTEP(j, r0, m, n)
                OSDN_P1_LSTEP(j - 1, r1, m, n)
                OSDN_P1_LSTEP(j - 2, r2, m, n)
            }
            n = m;                                  // (the loop's own decrement moves past the run)
            continue;
        }
        // ---- this thread's (s, lambda) = (k^2, k . dL/dk~) and mask bits ----
        OSDN_P1_BLOAD(n)
        float sv[TS], lam[TS];
#pragma unroll
        for (int u = 0; u < TS; ++u) {
            const float kv = to_f32(kreg[u]);
            sv[u] = kv * kv;
            lam[u] = kv * to_f32(greg[u]);
        }
        const uint32_t mword = (sg * TS) < 32 ? mreg.x : mreg.y;
        const uint32_t mbits = (mword >> ((sg * TS) & 31)) & ((1u << TS) - 1u);
        if (tid < C) {
            const float nn = fmaxf(fabsf(nrawreg), a.eps);
            const float bp = a.beta_aware ? betreg : 1.f;
            cas[tid] = a.eta * bp / nn * bp; sig[tid] = 0.f; casig[tid] = 0.f;
        }
        if (tid < K) a.a_ckpt[(bth * N + n) * K + tid] = ga[tid];
        __syncthreads();
        // a wavefront whose coordinates never touched the box in this run: P stays 1 and L is a plain running sum
        const bool plain = __all(mbits == ((1u << TS) - 1u));
        // ---- sweeps for sigma_i = <s_i, abar_i> ----
        float dprev = 0.f, a_left = 0.f;
        for (int sweep = 0; sweep < P1_MAX_SWEEPS; ++sweep) {
            float abL[TS], abP[TS];
            float loc = 0.f, P = 1.f;
            if (plain) {
#pragma unroll
                for (int u = TS - 1; u >= 0; --u) {
                    abL[u] = loc;
                    loc += __builtin_fmaf(-casig[sg * TS + u], sv[u], lam[u]);
                }
            } else {
#pragma unroll
                for (int u = TS - 1; u >= 0; --u) {
                    const bool in = (mbits >> u) & 1u;
                    abL[u] = in ? loc : 0.f;
                    abP[u] = in ? P : 0.f;
                    const float src = __builtin_fmaf(-casig[sg * TS + u], sv[u], lam[u]);
                    loc = abL[u] + src;
                    P = abP[u];
                }
            }
            segL[sg * K + c] = loc;
            segP[sg * K + c] = P;
            __syncthreads();
            // value of a at the right end of this run: chain the runs to its right
            float carry = ga[c];
#pragma unroll
            for (int s2 = NSEG - 1; s2 > 0; --s2)
                if (s2 > sg) carry = __builtin_fmaf(segP[s2 * K + c], carry, segL[s2 * K + c]);
            a_left = __builtin_fmaf(P, carry, loc);      // (meaningful in run 0: left end of the chunk)
            float prod[TS];
            if (plain) {
#pragma unroll
                for (int u = 0; u < TS; ++u) prod[u] = sv[u] * (abL[u] + carry);
            } else {
#pragma unroll
                for (int u = 0; u < TS; ++u) prod[u] = sv[u] * __builtin_fmaf(abP[u], carry, abL[u]);
            }
            part[wave * 64 + lane] = lane_fold<TS>(prod, lane);
            __syncthreads();
            if (tid < C) {
                const int i = tid, w0 = (i / TS) * WPS, u = i % TS;
                float sg_ = 0.f;
#pragma unroll
                for (int j = 0; j < NPART; ++j)     // fixed order: wavefronts of the run, lane groups
                    sg_ += part[(w0 + j / (64 / TS)) * 64 + (j % (64 / TS)) * TS + u];
                const float mx = wave_max(fabsf(sg_));
                const float dcur = wave_max(fabsf(sg_ - sig[i]));
                // converged, or (from the second pass on) the observed contraction ratio says
                // that the next difference would be below the tolerance
                const bool all_ok = dcur <= P1_TOL_BWD * mx ||
                                    (sweep >= 1 && dcur <= 0.1f * dprev && dcur * dcur <= P1_TOL_BWD * mx * dprev);
                dprev = dcur;
                sig[i] = sg_;
                casig[i] = cas[i] * sg_;
                if (tid == 0) done = all_ok ? 1 : 0;
            }
            __syncthreads();
            if (done) break;
        }
        // ---- accepted: sig generated a_left ----
        if (tid < C) a.tok_scalars[(tokc + (size_t)tid * a.H) * 4 + 3] = sig[tid];
        if (sg == 0) { ga[c] = a_left; gp[LN::vidx(c)] = a_left; }
        __syncthreads();
    }
    if (tid < K) a.dd_in[bh * K + tid] = ga[tid];
}
#undef OSDN_P1_BLOAD

// ---------------------------------------------------------------- precond_post ----
//   in : k, beta, retention, d_ckpt, tok_scalars (step, <d,s>, sum s, sigma per token),
//        a_ckpt (adjoint of d at the right end of every chunk), dkt (dL/dk~),
//        dk_read (read-side dL/dk), dbeta (partial, from phase 2)
//   out: dk (io type) = dk_read + d_t . dkt + 2 k_t (step_t abar_t + g_p d_t + g_nraw),
//        dbeta += sigma_t eta (1 - 2 b' p_t)/n_t,  dretention_t = <abar_t, d_t>
template <typename T, int K, int RET, bool RAG>
__global__ __launch_bounds__(K) __attribute__((amdgpu_waves_per_eu(2, 8))) void precond_post_kernel(PrecondBwdArgs a) {
    constexpr bool HAS_RET = RET != 0, RET_VEC = RET == 2;
    constexpr int LD = K + 1;
    __shared__ __attribute__((aligned(16))) float st_s[C];
    __shared__ __attribute__((aligned(16))) float r_s[C];
    __shared__ __attribute__((aligned(16))) float casig_s[C];
    __shared__ __attribute__((aligned(16))) float gp_s[C];
    __shared__ __attribute__((aligned(16))) float gn_s[C];
    // the scalar gate's dL/dr_i = sum over the coordinates of abar_i d_i: folded over the lanes of a
    // wavefront eight tokens at a time, one partial per wavefront and token here
    __shared__ float rpart[(HAS_RET && !RET_VEC) ? (K / 64) * C : 1];
    static_assert(PB == 8, "the fold takes eight values per lane");
    const int n = a.n0 + blockIdx.x / a.H, h = blockIdx.x % a.H, b = blockIdx.y, tid = threadIdx.x;
    const int N = a.T / C;
    const size_t bh = (size_t)b * a.H + h;
    const size_t tokc = ((size_t)b * a.T + (size_t)n * C) * a.H + h;
    const ChunkIn<T, K, RET, RAG> in(a, b, n, h);
    const size_t out0 = a.rows.first<RAG>(b, n) * a.H + h;
    const int rows = a.rows.count<RAG>(n);
    const bool project = a.d_min <= a.d_max;
    const float lo = project ? a.d_min : -INFINITY, hi = project ? a.d_max : INFINITY;
    if (tid < C) {
        const size_t th = tokc + (size_t)tid * a.H;
        const float4 sc = *reinterpret_cast<const float4 *>(a.tok_scalars + th * 4);
        const float step = sc.x, p = sc.y, n_raw = fabsf(sc.z), sg = sc.w;
        const float bet = in.beta[(size_t)tid * a.H];
        const float nn = fmaxf(n_raw, a.eps);
        const float bp = a.beta_aware ? bet : 1.f;
        const float ca = a.eta * bp / nn * bp;
        st_s[tid] = step;
        r_s[tid] = (HAS_RET && !RET_VEC) ? in.ret[(size_t)tid * a.H] : 1.f;
        casig_s[tid] = ca * sg;
        gp_s[tid] = -sg * ca;
        gn_s[tid] = (n_raw >= a.eps) ? -sg * step / nn : 0.f;
        if (a.beta_aware && tid < rows) a.dbeta[out0 + (size_t)tid * a.H] += sg * a.eta * (1.f - 2.f * bp * p) / nn;
    }
    // uniform bases + 32-bit per-thread offsets (64 rows of H*K elements: below 2^31)
    const T *kp = in.k;
    const size_t tile = (((size_t)b * N + n) * a.H + h) * C * K;        // dkt and dk_read: one tile per chunk and head
    const T *gp = static_cast<const T *>(a.dkt) + tile, *rp = static_cast<const T *>(a.dk_read) + tile;
    T *op = static_cast<T *>(a.dk) + out0 * K;
    const float *retp = RET_VEC ? in.ret : nullptr;     // per-coordinate retention and its gradient
    float *dretp = (RET_VEC && a.dretention) ? a.dretention + out0 * K : nullptr;
    const uint32_t kstride = (uint32_t)a.H * K;
    float Dv[C];
    // which steps landed inside the box: decided once, by precond_mask (or precond_lin_m)
    const uint2 mbits = project ? a.masks[(bh * N + n) * K + tid] : make_uint2(0xffffffffu, 0xffffffffu);
    const uint32_t mlo = mbits.x, mhi = mbits.y;
    {   // ---- replay d over the chunk (same arithmetic as the forward kernel) ----
        float kv[C];
#pragma unroll
        for (int i = 0; i < C; ++i) kv[i] = to_f32(lane_elem(kp + (size_t)i * kstride, tid));
        float d = a.d_ckpt[(bh * N + n) * K + tid];
        __syncthreads();
#pragma unroll
        for (int i = 0; i < C; ++i) {
            Dv[i] = d;
            const float r = RET_VEC ? lane_elem(retp + (size_t)i * kstride, tid) : r_s[i];
            d = clip3(d_bar<HAS_RET>(r, d, st_s[i], kv[i] * kv[i]), lo, hi);
        }
    }
    // ---- the chunk's adjoint recurrence, right to left, and the elementwise outputs ----
    float av = a.a_ckpt[(bh * N + n) * K + tid];
    // (the per-token scalars are read again through pointers the compiler cannot identify with
    // the arrays, so that it does not keep the replay's 128 values in registers)
    const float *st_p = st_s, *r_p = r_s, *casig_p = casig_s, *gp_p = gp_s, *gn_p = gn_s;
    asm volatile("" : "+v"(st_p), "+v"(r_p), "+v"(casig_p), "+v"(gp_p), "+v"(gn_p));
    float kb[2][PB], gb[2][PB], rb[2][PB], rrb[RET_VEC ? 2 : 1][RET_VEC ? PB : 1];
    // byte offsets (in units of T) of the next row to fetch and of the next row to write
    constexpr uint32_t FS = sizeof(float) / sizeof(T);
    const uint32_t rowb = kstride * (uint32_t)sizeof(T);
    uint32_t lofs = ((uint32_t)tid + (uint32_t)(C - 1) * kstride) * (uint32_t)sizeof(T);
    asm volatile("" : "+v"(lofs));
    // Pad tokens are stored to the last row that exists, which the same thread overwrites later: the
    // count of stores in flight stays known, where a branch would make every load behind it wait for all.
    uint32_t sofs = ((uint32_t)tid + (uint32_t)(rows - 1) * kstride) * (uint32_t)sizeof(T);
#define OSDN_PLOAD(buf, ih_)                                                                     \
    _Pragma("unroll") for (int u = 0; u < PB; ++u) {                                             \
        const uint32_t tofs = (uint32_t)(((ih_) - u) * K + tid) * (uint32_t)sizeof(T);           \
        kb[buf][u] = to_f32(at_byte(kp, lofs)); gb[buf][u] = to_f32(at_byte(gp, tofs));          \
        rb[buf][u] = to_f32(at_byte(rp, tofs));                                                  \
        if (RET_VEC) rrb[RET_VEC ? buf : 0][RET_VEC ? u : 0] = at_byte(retp, lofs * FS);         \
        lofs -= rowb;                                                                            \
    }
    OSDN_PLOAD(0, C - 1)
#pragma unroll
    for (int blk = 0; blk < C / PB; ++blk) {
        const int ih = C - 1 - blk * PB;
        if (blk + 1 < C / PB) OSDN_PLOAD((blk + 1) & 1, ih - PB)
        float pr[PB];
#pragma unroll
        for (int u = 0; u < PB; ++u) {
            const int i = ih - u;
            const uint32_t bit = (i < 32 ? mlo : mhi) & (1u << (i & 31));
            const float ab = bit ? av : 0.f;
            const float kv = kb[blk & 1][u], g = gb[blk & 1][u], Di = Dv[i];
            const float gsum = st_p[i] * ab + gp_p[i] * Di + gn_p[i];
            at_byte(op, sofs) = from_f32<T>(rb[blk & 1][u] + Di * g + 2.f * kv * gsum);
            if (RET_VEC) { if (dretp) at_byte(dretp, sofs * FS) = ab * Di; }
            pr[u] = ab * Di;
            sofs -= i < rows ? rowb : 0u;
            const float src = __builtin_fmaf(-casig_p[i], kv * kv, kv * g);
            const float r = RET_VEC ? rrb[RET_VEC ? blk & 1 : 0][RET_VEC ? u : 0] : r_p[i];
            av = HAS_RET ? __builtin_fmaf(r, ab, src) : ab + src;
        }
        if (HAS_RET && !RET_VEC) {
            const int lane = tid & 63;
            const float tot = lane_fold8_all(pr, lane);     // lane l: token ih - l % 8, summed over the wavefront
            if (lane < PB) rpart[(HAS_RET && !RET_VEC) ? (tid >> 6) * C + ih - lane : 0] = tot;
        }
    }
    if (HAS_RET && !RET_VEC) {
        __syncthreads();
        if (tid < rows && a.dretention) {
            float s = 0.f;
#pragma unroll
            for (int w = 0; w < K / 64; ++w) s += rpart[(HAS_RET && !RET_VEC) ? w * C + tid : 0];
            a.dretention[out0 + (size_t)tid * a.H] = s;
        }
    }
}

// -------------------------------------------------------------------- launchers ----
template <typename T, int K, int RET>
static void launch_chain_k(const PrecondBwdArgs &a, int nchains, hipStream_t st) {
    if constexpr (RET == 0) {
        if (a.lin_clean) {
            with_rows(a.rows, [&](auto rag) { hipLaunchKernelGGL((precond_chain_lin_kernel<T, K, decltype(rag)::value>), dim3(nchains), dim3(P1T), 0, st, a); });
            return;
        }
    }
    if constexpr (RET != 0) {
        if (a.pieces) {
            with_rows(a.rows, [&](auto rag) { hipLaunchKernelGGL((precond_chain_kernel<T, K, RET, true, decltype(rag)::value>), dim3(nchains * a.pieces), dim3(P1F), 0, st, a); });
            return;
        }
    }
    with_rows(a.rows, [&](auto rag) { hipLaunchKernelGGL((precond_chain_kernel<T, K, RET, false, decltype(rag)::value>), dim3(nchains), dim3(P1F), 0, st, a); });
}
template <typename T, int RET>
static int launch_precond_bwd_t(const PrecondBwdArgs &a, int which, hipStream_t st) {
    const dim3 per_chunk((a.n1 - a.n0) * a.H, a.B);
    const int nchains = (a.seq_chunks ? a.n_seqs : a.B) * a.H;
    if (a.K == 64) {
        if (which == 0) with_rows(a.rows, [&](auto rag) { hipLaunchKernelGGL((precond_mask_kernel<T, 64, RET, decltype(rag)::value>), per_chunk, dim3(64), 0, st, a); });
        else if (which == 1) launch_chain_k<T, 64, RET>(a, nchains, st);
        else with_rows(a.rows, [&](auto rag) { hipLaunchKernelGGL((precond_post_kernel<T, 64, RET, decltype(rag)::value>), per_chunk, dim3(64), 0, st, a); });
    } else if (a.K == 128) {
        if (which == 0) with_rows(a.rows, [&](auto rag) { hipLaunchKernelGGL((precond_mask_kernel<T, 128, RET, decltype(rag)::value>), per_chunk, dim3(128), 0, st, a); });
        else if (which == 1) launch_chain_k<T, 128, RET>(a, nchains, st);
        else with_rows(a.rows, [&](auto rag) { hipLaunchKernelGGL((precond_post_kernel<T, 128, RET, decltype(rag)::value>), per_chunk, dim3(128), 0, st, a); });
    } else {
        return -1;
    }
    return 0;
}
static int launch_precond_bwd_any(const PrecondBwdArgs &a, bool bf16_io, int which, hipStream_t st) {
    const int ret = a.retention ? (a.ret_vec ? 2 : 1) : 0;
    if (ret == 2)
        return bf16_io ? launch_precond_bwd_t<bf16, 2>(a, which, st) : launch_precond_bwd_t<float, 2>(a, which, st);
    if (ret == 1)
        return bf16_io ? launch_precond_bwd_t<bf16, 1>(a, which, st) : launch_precond_bwd_t<float, 1>(a, which, st);
    return bf16_io ? launch_precond_bwd_t<bf16, 0>(a, which, st) : launch_precond_bwd_t<float, 0>(a, which, st);
}
template <typename T>
static int launch_precond_lin_t(const PrecondBwdArgs &a, bool m_part, hipStream_t st) {
    const dim3 per_chunk((a.n1 - a.n0) * a.H, a.B);
    if (a.K == 64) {
        if (m_part) with_rows(a.rows, [&](auto rag) { hipLaunchKernelGGL((precond_lin_m_kernel<T, 64, decltype(rag)::value>), per_chunk, dim3(P1T), 0, st, a); });
        else with_rows(a.rows, [&](auto rag) { hipLaunchKernelGGL((precond_lin_r_kernel<T, 64, decltype(rag)::value>), per_chunk, dim3(P1T), 0, st, a); });
    } else if (a.K == 128) {
        if (m_part) with_rows(a.rows, [&](auto rag) { hipLaunchKernelGGL((precond_lin_m_kernel<T, 128, decltype(rag)::value>), per_chunk, dim3(P1T), 0, st, a); });
        else with_rows(a.rows, [&](auto rag) { hipLaunchKernelGGL((precond_lin_r_kernel<T, 128, decltype(rag)::value>), per_chunk, dim3(P1T), 0, st, a); });
    } else {
        return -1;
    }
    return 0;
}
// only without retention.  m_part: flags and inverses of the chunks [n0, n1) (needs the masks when
// there is a box); else rho0 and the sums of lambda (needs the flags and dL/dk~ of those chunks)
int launch_precond_lin_bwd(const PrecondBwdArgs &a, bool bf16_io, bool m_part, hipStream_t st) {
    if (a.retention || !a.lin_clean || !a.lin_M || !a.lin_r0 || !a.lin_t0) return -1;
    return bf16_io ? launch_precond_lin_t<bf16>(a, m_part, st) : launch_precond_lin_t<float>(a, m_part, st);
}
int launch_precond_mask(const PrecondBwdArgs &a, bool bf16_io, hipStream_t st) { return launch_precond_bwd_any(a, bf16_io, 0, st); }
int launch_precond_chain(const PrecondBwdArgs &a, bool bf16_io, hipStream_t st) { return launch_precond_bwd_any(a, bf16_io, 1, st); }
int launch_precond_post(const PrecondBwdArgs &a, bool bf16_io, hipStream_t st) { return launch_precond_bwd_any(a, bf16_io, 2, st); }

}  // namespace osdn
