// Phase 1 of OSDN: the online preconditioner sweep (Algorithm 1, Eq. (dt_update) and its
// retention form Eq. (dt_update_apf)).
//
// The recurrence  d_{t+1} = clip(r_t d_t + c_t s_t),  s_t = k_t (.) k_t,
//                 c_t = eta b'(1 - b' p_t)/n_t,  p_t = <d_t, s_t>
// couples the K coordinates only through the scalar p_t.  One workgroup owns one
// (batch, head) chain and walks it in chunks of 64 tokens.  Inside a chunk it solves for the
// 64 scalars p by fixed-point sweeps: given p (first guess: <d_0, s_t>) the recurrence
// separates into K independent scalar recurrences; from the resulting trajectory the 64 inner
// products are recomputed; the sweep repeats until they reproduce themselves.  Sweep m fixes
// at least the first m tokens exactly, so 64 sweeps always suffice; because the coupling is
// O(eta) two do in practice, also when coordinates sit on a face of the box.  With one retention per
// token the first guess takes what the gates of the tokens before leave of d_0 (a prefix product over
// the chunk, every wavefront its own): without it a third sweep is needed where d still fades, as it does over the first ten
// chunks of a sequence with gates of 0.999 (2 x 384 tokens, 8 heads of 128 x 128: 52.8 -> 46.9 us).  Once d lies on the lower face
// the gates change nothing, and a guess that fades is what needs one sweep more (16 heads of 64 chunks of 128 coordinates, bf16, us
// a chunk, without a fading guess, with one throughout, and as it is: gates of 0.97 2.71, 3.84, 2.72, of 0.999 3.39, 3.86, 3.30).
//
// A sweep does not walk the 64 tokens one after the other.  The chunk is cut into 8 runs of
// 8 tokens, one wavefront per run, a lane per coordinate (pair): everything a thread needs of
// the chunk (its k, s, d) stays in registers.  One token maps d to clip(r d + c s), and maps
// of that form compose to x -> clip3(A x + B, L, H) with
//     A' = r A,  B' = r B + c s,  L' = clip(r L + c s),  H' = clip(r H + c s)      (r >= 0),
// so a thread first composes the map of its run, the runs are chained through LDS (one
// fma + median-of-three per run), and with its run's starting value known the thread replays
// its 8 tokens.  The products s d are folded over the lanes of the wavefront.  All arithmetic is fp32; k~ is
// rounded once, from fp32 d k.
//
// Without retention the box is left out of a sweep as long as it cannot matter: with every c >= 0 the
// trajectory of a run only rises, so it met no face if it starts at or above the lower one and ends at
// or below the upper one (checked by every sweep).  The map of a run is then x + B and a replayed
// token one fma, the same one as in the full form.  A chunk that fails the check is done again with the box;
// one that begins with a coordinate on a face is not tried without it.
//
// One barrier per sweep: a sweep's verdict (did p reproduce itself?) is published together with the run
// maps of the sweep that would follow, which are dropped if there is none; the value of d at the
// chunk's end travels with them.  The kernel is bound by the issue of one CU's vector instructions (about
// 500 a wavefront and chunk, two wavefronts per SIMD) and by these barriers: 64 tokens of 128
// coordinates take 2.8 us at the paper's step size (two sweeps; 3.9 us with the box always in, separate
// barriers for maps and verdicts, selects instead of register swaps in the folds and 64-bit row addresses
// in vector registers: 4 x 16 chains of 4096 tokens 250 -> 179 us).  4 runs of 16 tokens fold with fewer
// instructions but leave one wavefront per SIMD and nothing to cover latency: 210 us.
//
// For few long chains the same composition is taken one level up: the chain is cut into pieces,
// one workgroup per piece walks its chunks from a start value it is given and also composes the
// accepted run maps into one map for the piece; the next sweep carries the chain's start value
// through those maps to get its start values, and the sweeps over all pieces repeat until no
// start value of a chain moves (the caller launches them ahead of time; the workgroups of a
// settled chain return at once).
#include "osdn_precond.h"

namespace osdn {

// RET: 0 = no retention, 1 = one gate per (token, head), 2 = one per coordinate (diag(r_t))
// PIECES: one workgroup per piece of a chain (sweeps over the whole sequence) instead of one per chain
// TILES: part of a forward pass: whole chunks, k~ as one contiguous [64 x K] tile per chunk and head, the
// checkpoints and token scalars wanted.  Then no access of the loop sits under a branch (lanes without
// an element of their own repeat another's), and the wait for the next chunk's keys, which the compiler
// counts in accesses, does not become one for the stores behind them.
// Registers: with one gate per token, K = 128 in bf16 the compiler is held to 128, which it would pass by four: two workgroups
// to a CU, which the pieces are laid out for (16 chains of 256 chunks, forward pass: 873 us with 132 registers, 753 with 128).
template <typename T, int K, int RET, bool PIECES, bool TILES, bool RAG>
__global__ __launch_bounds__(P1F, K == 128 && RET == 1 && sizeof(T) == 2 ? 4 : 1) void precond_fwd_kernel(PrecondArgs a) {
    constexpr bool HAS_RET = RET != 0, RET_VEC = RET == 2;
    constexpr int RE = RET_VEC ? K / 64 : 1;      // retention values a thread keeps per token
    constexpr int CPT = K / 64;                   // coordinates per thread (adjacent)
    constexpr int NRUN = C / RUN;                 // = wavefronts of the workgroup
    static_assert(K <= P1F, "one thread per coordinate, for the pieces");
    typedef Pack<T, CPT> Pk;
    constexpr bool FAST = RET == 0 && !PIECES;    // sweeps without the box while it does not matter
    constexpr int NBUF = PIECES ? 3 : 2;          // map buffers, used in turn (a piece reads the accepted maps once more)
    __shared__ float dnext[K];                   // d at the end of the chunk
    // per run and coordinate B, L, H and, with one retention per coordinate, A (else A is one number per
    // run); without the box B alone
    constexpr int NCOMP = RET_VEC ? 4 : 3;
    __shared__ __attribute__((aligned(16))) float maps[NBUF][NCOMP][NRUN * K];
    __shared__ __attribute__((aligned(16))) float runA[2][NRUN];      // (chunks in turn)
    __shared__ int flags[2][NRUN];

    const int tid = threadIdx.x, run = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int c0 = lane * CPT;                    // first coordinate of this thread
    const int u_own = fold_token(lane);      // the token of the run whose scalars this lane keeps
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
        a.d_in = begins ? a.d_first : a.d_out;
        bt = 0;
    }
    const size_t bh = (size_t)b * a.H + h;                    // the chain: indexes d_in / d_out
    const size_t bth = (size_t)bt * a.H + h;                  // indexes the per-chunk buffers
    const bool project = a.d_min <= a.d_max;
    const float lo = project ? a.d_min : -INFINITY, hi = project ? a.d_max : INFINITY;
    const int N = (a.T + C - 1) / C;
    const uint32_t kstride = (uint32_t)a.H * K;   // elements between consecutive tokens
    const ChainRows<RAG> rows(a.rows, a.seq_chunks, b, a.n0);

    if (!PIECES) {
        if (tid < K) dnext[tid] = a.d_in ? a.d_in[bh * K + tid] : 1.f;
    } else {
        // The start value of this piece: the chain's own start value carried through the maps
        // that the previous sweep left for the pieces before this one (first sweep: the chain's
        // start value itself, as a guess).  Every workgroup of the chain walks all its pieces and
        // so sees whether any start value moved by more than the tolerance of the sweeps; if
        // none did, what the previous sweep wrote stands and the chain is settled.
        const size_t buf = (size_t)gridDim.x * K;                 // elements of one buffer
        const size_t cur = (a.sweep & 1) * buf, prev = buf - cur;
        float x = 1.f, xs = 1.f;
        bool moved = a.sweep == 0;
        if (tid < K) {
            // WALK records at a time, asked for together (past the end: the last one again): one by one every piece cost the walk
            // a memory latency of 0.45 us, once a sweep and once more to find that the chain is settled (16 chains, forward pass:
            // 12 pieces, three sweeps 106.7 -> 102.2 us; 32 pieces, two sweeps 1026 -> 1014; 16 at a time: two registers too many for
            // two workgroups a CU with fp32 I/O)
            constexpr int WALK = 8;
            x = xs = a.d_in ? a.d_in[bh * K + tid] : 1.f;
            for (int q0 = 0; q0 < (a.sweep > 0 ? a.pieces : 0); q0 += WALK) {
                float old[WALK];
                float4 m[WALK];
#pragma unroll
                for (int j = 0; j < WALK; ++j) {
                    const size_t i = prev + (bh * a.pieces + min(q0 + j, a.pieces - 1)) * K + tid;
                    old[j] = a.piece_start[i];
                    m[j] = a.piece_map[i];
                }
#pragma unroll
                for (int j = 0; j < WALK; ++j) {
                    if (q0 + j < a.pieces) {
                        if (q0 + j == piece) xs = x;
                        if (!(fabsf(x - old[j]) <= PIECE_TOL * fmaxf(fabsf(x), fabsf(old[j])))) moved = true;
                        x = clip3(__builtin_fmaf(m[j].x, x, m[j].y), m[j].z, m[j].w);
                    }
                }
            }
        }
        const bool any = __syncthreads_or(moved);
        if (piece == 0 && tid == 0) a.settled[chain] = any ? 0 : 1;
        if (!any) return;
        if (tid < K) {
            dnext[tid] = xs;
            a.piece_start[cur + (bh * a.pieces + piece) * K + tid] = xs;
        }
        a.piece_map += cur;
    }
    float PA = 1.f, PB = 0.f, PL = -FLT_MAX, PH = FLT_MAX;    // thread c < K: the piece so far, as a map of coordinate c

    typedef Pack<float, CPT> Pr;
    typename Pk::Raw kreg[RUN];                  // this thread's k of the next chunk
    typename Pr::Raw rreg[RET_VEC ? RUN : 1];    // ... and its per-coordinate retention
    float betreg = 0.f, retreg = 1.f;            // next chunk: beta of token (run, u_own), retention of token `lane`
    // (rows past the end: reread; a row's address is the one before, a row further if there is one)
    const size_t u0 = (rows.batch + (size_t)(long long)rows.base) * a.H + h, chunk_rows = (size_t)C * a.H;
    const T *const kc = static_cast<const T *>(a.k) + u0 * K;
    const float *const bc = a.beta + u0, *const rc = HAS_RET ? a.retention + u0 * (RET_VEC ? K : 1) : nullptr;
#define OSDN_P1_LOAD(n_)                                                                         \
    {                                                                                            \
        const size_t off_ = (size_t)(n_) * chunk_rows;                                           \
        const int last_ = rows.count(n_) - 1, r0_ = RAG ? min(run * RUN, last_) : run * RUN;     \
        const int fl_ = fresh_lane(lane);                                                        \
        const int i_ = RAG ? min(run * RUN + u_own, last_) : run * RUN + u_own;                  \
        betreg = lane_elem(bc + off_, i_ * a.H);                                                 \
        if (RET == 1) retreg = lane_elem(rc + off_, (RAG ? min(lane, last_) : lane) * a.H);      \
        const T *kp_ = kc + (off_ * K + (uint32_t)r0_ * kstride);                                \
        const float *rp_ = RET_VEC ? rc + (off_ * K + (uint32_t)r0_ * kstride) : nullptr;        \
        _Pragma("unroll") for (int u = 0; u < RUN; ++u) {                                        \
            const size_t at_ = RAG ? 0 : (size_t)u * kstride;                                    \
            kreg[u] = row_elem(reinterpret_cast<const typename Pk::Raw *>(kp_ + at_), fl_);      \
            if (RET_VEC) rreg[u] = row_elem(reinterpret_cast<const typename Pr::Raw *>(rp_ + at_), fl_); \
            if (RAG) {                                                                           \
                const uint32_t st_ = u < last_ - r0_ ? kstride : 0u;                             \
                kp_ += st_;                                                                      \
                if (RET_VEC) rp_ += st_;                                                         \
            }                                                                                    \
        }                                                                                        \
    }
    if (RAG && TILES && rows.count(a.n1 - 1) < C) {      // the last chunk as a whole tile, for the backward pass
        const int there = rows.count(a.n1 - 1);
        const size_t off = (size_t)(a.n1 - 1) * chunk_rows, tl = (size_t)b * C * a.H + h;
        for (int u = 0; u < RUN; ++u) {
            const int i = run * RUN + u, from = min(i, there - 1);
            typedef typename Pk::Raw R;
            const R x = reinterpret_cast<const R *>(kc + (off + (size_t)from * a.H) * K)[lane];
            reinterpret_cast<R *>(static_cast<T *>(a.k_tail) + (tl + (size_t)i * a.H) * K)[lane] = i < there ? x : R{};
            if (RET_VEC)
                for (int e = 0; e < CPT; ++e) {
                    const float r = rc[(off + (size_t)from * a.H) * K + c0 + e];
                    a.ret_tail[(tl + (size_t)i * a.H) * K + c0 + e] = i < there ? r : 1.f;
                }
        }
        if (tid < C) {
            const size_t from = off + (size_t)min(tid, there - 1) * a.H, to = tl + (size_t)tid * a.H;
            a.beta_tail[to] = tid < there ? bc[from] : 0.f;
            if (HAS_RET && !RET_VEC) a.ret_tail[to] = tid < there ? rc[from] : 1.f;
        }
    }
    OSDN_P1_LOAD(a.n0)
    // (waited for here: loads that are pending when the loop is entered would make its head wait for the stores too)
    __builtin_amdgcn_s_waitcnt(0x0f70);         // vmcnt(0)
    __syncthreads();
    float dst[CPT];                             // d of this thread's coordinates at the start of the chunk
#pragma unroll
    for (int e = 0; e < CPT; ++e) dst[e] = dnext[c0 + e];
    bool boxed = !FAST;                         // this chunk is swept with the box
    int pub = 0, fl = 0;                        // map buffer and flag row of the next barrier
    for (int n = a.n0; n < a.n1; ++n) {
        const int t0 = n * C;
        const int nvalid = rows.count(n);
        // ---- this thread's k and s = k^2 (rows past the end of the sequence: no-op tokens) ----
        float kf[RUN][CPT], sv[RUN][CPT];
        if (nvalid < C) {
#pragma unroll
            for (int u = 0; u < RUN; ++u)
                if (run * RUN + u >= nvalid) kreg[u] = typename Pk::Raw{};
        }
#pragma unroll
        for (int u = 0; u < RUN; ++u) {
            Pk::unpack(kreg[u], kf[u]);
#pragma unroll
            for (int e = 0; e < CPT; ++e) {
                sv[u][e] = kf[u][e] * kf[u][e];
            }
        }
        const bool valid = run * RUN + u_own < nvalid;
        const float bet = betreg, ret = !RAG || lane < nvalid ? retreg : 1.f;
        // what the retention of the tokens before (run, u_own) leaves of d_0, unless that is nearly all of it, the lower face holds
        // it up, or eta is so large that the updates do (from this chunk's d and gates alone: where a call or a launch begins must
        // not show; K = 64, gates of 0.999, eta 1: 6.00 us a chunk with the fading guess, 5.40 without)
        float left = 1.f;
        if constexpr (RET == 1) {
            bool fades = a.eta <= 5e-4f * K && !__all(ret > 0.99995f);
            if (fades) {
                bool near = true;
#pragma unroll
                for (int e = 0; e < CPT; ++e) near = near && dst[e] <= 1.02f * lo;
                fades = !__all(near);
            }
            if (fades) {
                float x = ret;
#define OSDN_P1_SCAN(ctrl_, rows_) x *= __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0x3f800000, __builtin_bit_cast(int, x), ctrl_, rows_, 0xF, false));
                OSDN_P1_SCAN(0x111, 0xF) OSDN_P1_SCAN(0x112, 0xF) OSDN_P1_SCAN(0x114, 0xF) OSDN_P1_SCAN(0x118, 0xF)      // row_shr:1, 2, 4, 8
                OSDN_P1_SCAN(0x142, 0xA) OSDN_P1_SCAN(0x143, 0xC)                                                        // row_bcast:15, 31
#undef OSDN_P1_SCAN
                const int t = run * RUN + u_own;
                const float all = lane_bcast(x, 63);
                x = __builtin_bit_cast(float, __builtin_amdgcn_ds_bpermute((t - 1) * 4, __builtin_bit_cast(int, x)));
                bool faced = true;              // every coordinate comes to the lower face within this chunk
#pragma unroll
                for (int e = 0; e < CPT; ++e) faced = faced && dst[e] * all <= lo;
                left = t > 0 && !__all(faced) ? x : 1.f;
            }
        }
        // ---- the scalars of token (run, u_own): n_raw = sum s, first guess p = <d_0, s> times what retention leaves ----
        float nraw, cb, ca, p_cur, c_cur;
        {
            if (TILES) {                        // every wavefront an equal part
                const int c = run * (K / NRUN) + lane % (K / NRUN);
                a.d_ckpt[(bth * N + n) * K + c] = dnext[c];
            } else if (a.d_ckpt && run == 0) {
#pragma unroll
                for (int e = 0; e < CPT; ++e) a.d_ckpt[(bth * N + n) * K + c0 + e] = dst[e];
            }
            float vn[RUN], vp[RUN];
#pragma unroll
            for (int u = 0; u < RUN; ++u) {
                vn[u] = sv[u][0]; vp[u] = sv[u][0] * dst[0];
#pragma unroll
                for (int e = 1; e < CPT; ++e) { vn[u] = __builtin_fmaf(kf[u][e], kf[u][e], vn[u]); vp[u] = __builtin_fmaf(sv[u][e], dst[e], vp[u]); }
            }
            nraw = fold_tokens(vn);
            p_cur = fold_tokens(vp) * left;
            const float nn = fmaxf(nraw, a.eps);
            const float bp = a.beta_aware ? bet : 1.f;
            cb = valid ? a.eta * bp / nn : 0.f;
            ca = cb * bp;
            c_cur = cb - ca * p_cur;
        }
        float rv[RUN][RE];                      // retention of this thread's coordinates (no-op tokens: 1)
#pragma unroll
        for (int u = 0; u < RUN; ++u) {
            if (RET_VEC) {
                float r2[CPT];
                Pr::unpack(rreg[RET_VEC ? u : 0], r2);
#pragma unroll
                for (int e = 0; e < RE; ++e) rv[u][e] = run * RUN + u < nvalid ? r2[e] : 1.f;
            } else {
                rv[u][0] = HAS_RET ? __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, ret), run * RUN + u)) : 1.f;
            }
        }
        OSDN_P1_LOAD(min(n + 1, a.n1 - 1))       // (past the end: reloaded in vain)
        // ---- fixed-point sweeps ----
        // flags of a wavefront: 1: its p did not reproduce themselves, 2: the box matters (a sweep without it is void)
        if (FAST) {                             // (from d alone: where a call or a launch begins must not show)
            bool in = true;
#pragma unroll
            for (int e = 0; e < CPT; ++e) in = in && dst[e] > lo && dst[e] < hi;
            boxed = !__all(in);
        }
        int sweeps_used = 0;
        float dtr[RUN][CPT], dend[CPT];
        float c_acc = c_cur, p_acc = p_cur;     // what generated dtr and dend
        int verdict = 1;
        auto put_map = [&](int comp, const float (&v)[CPT]) {
            *reinterpret_cast<typename Pr::Raw *>(&maps[pub][comp][run * K + c0]) = Pr::pack(v);
        };
        auto get_map = [&](int comp, int j, float (&v)[CPT]) {
            Pr::unpack(*reinterpret_cast<const typename Pr::Raw *>(&maps[pub][comp][j * K + c0]), v);
        };
        for (int sweep = 0;; ++sweep) {
            float cv[RUN];
#pragma unroll
            for (int u = 0; u < RUN; ++u) cv[u] = lane_bcast(c_cur, fold_lane(u));
            // the map of this run, x -> clip3(A x + B, L, H), per coordinate
            if (FAST && !boxed) {
                float Bv[CPT];
#pragma unroll
                for (int e = 0; e < CPT; ++e) {
                    Bv[e] = cv[0] * sv[0][e];
#pragma unroll
                    for (int u = 1; u < RUN; ++u) Bv[e] = __builtin_fmaf(cv[u], sv[u][e], Bv[e]);
                }
                put_map(0, Bv);
            } else {
                float Av[CPT], Bv[CPT], Lv[CPT], Hv[CPT];
#pragma unroll
                for (int e = 0; e < CPT; ++e) {
                    float A = 1.f, B = 0.f, L = -FLT_MAX, H = FLT_MAX;
#pragma unroll
                    for (int u = 0; u < RUN; ++u) {
                        const float bs = cv[u] * sv[u][e];
                        if (HAS_RET) {
                            const float r = rv[u][RET_VEC ? e : 0];
                            A *= r;
                            B = __builtin_fmaf(r, B, bs);
                            L = clip3(__builtin_fmaf(r, L, bs), lo, hi);
                            H = clip3(__builtin_fmaf(r, H, bs), lo, hi);
                        } else {
                            B += bs;
                            L = clip3(L + bs, lo, hi);
                            H = clip3(H + bs, lo, hi);
                        }
                    }
                    Av[e] = A; Bv[e] = B; Lv[e] = L; Hv[e] = H;
                }
                put_map(0, Bv); put_map(1, Lv); put_map(2, Hv);
                if (RET_VEC) put_map(NCOMP - 1, Av);
                else if (HAS_RET && sweep == 0 && lane == 0) runA[n & 1][run] = Av[0];
            }
            // with the maps: the verdict on the sweep before, and d at the end of its last run
            if (sweep > 0) {
                if (run == NRUN - 1) {
#pragma unroll
                    for (int e = 0; e < CPT; ++e) dnext[c0 + e] = dend[e];
                }
                if (lane == 0) flags[fl][run] = verdict;
            }
            __syncthreads();
            if (sweep > 0) {
                int all = 0;
#pragma unroll
                for (int w = 0; w < NRUN; ++w) all |= flags[fl][w];
                fl ^= 1;
                if (FAST && (all & 2)) {        // once more, from where p has got to, with the box
                    boxed = true;
                    sweep = -1;
                    continue;
                }
                if (all == 0 || sweep >= P1_MAX_SWEEPS) break;
            }
            ++sweeps_used;
            float vp[RUN];
            bool within = true;
            if (FAST && !boxed) {
                // d at the start of this run: the runs to its left applied to d at the chunk start
                // (all runs are read, so that the reads go out together)
                float d[CPT], Bm[NRUN - 1][CPT];
#pragma unroll
                for (int j = 0; j < NRUN - 1; ++j) get_map(0, j, Bm[j]);
#pragma unroll
                for (int e = 0; e < CPT; ++e) {
                    d[e] = dst[e];
#pragma unroll
                    for (int j = 0; j < NRUN - 1; ++j) d[e] += j < run ? Bm[j][e] : 0.f;
                    within = within && d[e] >= lo;
#pragma unroll
                    for (int u = 0; u < RUN; ++u) {
                        dtr[u][e] = d[e];
                        vp[u] = e == 0 ? sv[u][e] * d[e] : __builtin_fmaf(sv[u][e], d[e], vp[u]);
                        d[e] = __builtin_fmaf(cv[u], sv[u][e], d[e]);
                    }
                    within = within && d[e] <= hi;
                    dend[e] = d[e];
                }
                within = within && (c_cur >= 0.f || !project);
            } else {
                float d[CPT], Av[CPT];
                float Bm[NRUN - 1][CPT], Lm[NRUN - 1][CPT], Hm[NRUN - 1][CPT];
#pragma unroll
                for (int j = 0; j < NRUN - 1; ++j) { get_map(0, j, Bm[j]); get_map(1, j, Lm[j]); get_map(2, j, Hm[j]); }
#pragma unroll
                for (int e = 0; e < CPT; ++e) d[e] = dst[e];
#pragma unroll
                for (int j = 0; j < NRUN - 1; ++j) {
                    if (RET_VEC) get_map(NCOMP - 1, j, Av);
#pragma unroll
                    for (int e = 0; e < CPT; ++e) {
                        if (!RET_VEC) Av[e] = HAS_RET ? runA[n & 1][j] : 1.f;
                        const float x = clip3(HAS_RET ? __builtin_fmaf(Av[e], d[e], Bm[j][e]) : d[e] + Bm[j][e], Lm[j][e], Hm[j][e]);
                        d[e] = j < run ? x : d[e];
                    }
                }
#pragma unroll
                for (int e = 0; e < CPT; ++e) {
                    // replay of the run's tokens (the same arithmetic as the reverse sweep's replay)
#pragma unroll
                    for (int u = 0; u < RUN; ++u) {
                        dtr[u][e] = d[e];
                        vp[u] = e == 0 ? sv[u][e] * d[e] : __builtin_fmaf(sv[u][e], d[e], vp[u]);
                        d[e] = clip3(d_bar<HAS_RET>(rv[u][RET_VEC ? e : 0], d[e], cv[u], sv[u][e]), lo, hi);
                    }
                    dend[e] = d[e];
                }
            }
            const float p_new = fold_tokens(vp);
            const bool ok = fabsf(p_new - p_cur) <= P1_TOL * fabsf(p_new);
            verdict = (__all(ok) ? 0 : 1) | (__all(within) ? 0 : 2);
            c_acc = c_cur; p_acc = p_cur;
            p_cur = p_new;
            c_cur = cb - ca * p_new;
            pub = pub + 1 == NBUF ? 0 : pub + 1;
        }
        // ---- accepted: (c_acc, p_acc) generated dtr and dend ----
        {
            T *ktp = static_cast<T *>(a.k_tilde) + (TILES ? (((size_t)bt * N + n) * a.H + h) * C : ((size_t)bt * a.T + t0) * a.H + h) * K;
            const uint32_t ktstride = TILES ? K : kstride;
            const int fl = fresh_lane(lane);
#pragma unroll
            for (int u = 0; u < RUN; ++u) {
                const int i = run * RUN + u;
                if (TILES || i < nvalid) {
                    float out[CPT];
#pragma unroll
                    for (int e = 0; e < CPT; ++e) out[e] = dtr[u][e] * kf[u][e];
                    row_elem(reinterpret_cast<typename Pk::Raw *>(ktp + (size_t)i * ktstride), fl) = Pk::pack(out);
                }
            }
        }
        // (RET == 0) off the box, by the margin at the upper face: d only rose, so that the last run's end counts (64 chains of
        // 64 chunks: 178.8 us, with every run looking 180.2; 177.7 where the sweeps themselves kept the margin, which swept a chain that stands within
        // it in vain)
        bool clear = true;
        if (RET == 0) {
            clear = FAST && !boxed;
            if (clear && run == NRUN - 1) {
                bool in = true;
#pragma unroll
                for (int e = 0; e < CPT; ++e) in = in && dend[e] <= mark_bound(lo, hi);
                clear = __all(in);
            }
        }
        if (TILES || (a.tok_scalars && valid)) {       // (eight lanes store the same)
            const size_t th = ((size_t)bt * a.T + t0) * a.H + h;
            lane_elem(reinterpret_cast<float4 *>(a.tok_scalars) + th, (run * RUN + u_own) * a.H) = make_float4(c_acc, p_acc, RET == 0 ? (clear ? -nraw : fabsf(nraw)) : nraw, (float)sweeps_used);
        }
        if (PIECES && tid < K) {                 // the accepted run maps, applied after the piece so far
            const int acc = pub == 0 ? NBUF - 1 : pub - 1;       // (the last published ones were dropped)
#pragma unroll
            for (int j = 0; j < NRUN; ++j) {
                const float A = RET_VEC ? maps[acc][NCOMP - 1][j * K + tid] : HAS_RET ? runA[n & 1][j] : 1.f;
                const float B = maps[acc][0][j * K + tid], L = maps[acc][1][j * K + tid], H = maps[acc][2][j * K + tid];
                PA *= A;
                PB = __builtin_fmaf(A, PB, B);
                PL = clip3(__builtin_fmaf(A, PL, B), L, H);
                PH = clip3(__builtin_fmaf(A, PH, B), L, H);
            }
        }
#pragma unroll
        for (int e = 0; e < CPT; ++e) dst[e] = dnext[c0 + e];
        pub = pub + 1 == NBUF ? 0 : pub + 1;
    }
    if (PIECES && tid < K) a.piece_map[(bh * a.pieces + piece) * K + tid] = make_float4(PA, PB, PL, PH);
    if (run == 0 && (!PIECES || piece == a.pieces - 1)) {
#pragma unroll
        for (int e = 0; e < CPT; ++e) a.d_out[bh * K + c0 + e] = dst[e];
    }
}

template <typename T, int RET, bool PIECES, bool TILES>
static int launch_precond_fwd_tp(const PrecondArgs &a, hipStream_t st) {
    dim3 grid((a.seq_chunks ? a.n_seqs : a.B) * a.H * (PIECES ? a.pieces : 1)), block(P1F);
    if (TILES && (a.T % C != 0 || !a.d_ckpt || !a.tok_scalars)) return -1;
    if (a.K == 64) with_rows(a.rows, [&](auto rag) { hipLaunchKernelGGL((precond_fwd_kernel<T, 64, RET, PIECES, TILES, decltype(rag)::value>), grid, block, 0, st, a); });
    else if (a.K == 128) with_rows(a.rows, [&](auto rag) { hipLaunchKernelGGL((precond_fwd_kernel<T, 128, RET, PIECES, TILES, decltype(rag)::value>), grid, block, 0, st, a); });
    else return -1;
    return 0;
}
template <typename T, int RET>
static int launch_precond_fwd_t(const PrecondArgs &a, hipStream_t st) {
    if (!a.kt_tiles) return a.pieces ? -1 : launch_precond_fwd_tp<T, RET, false, false>(a, st);
    return a.pieces ? launch_precond_fwd_tp<T, RET, true, true>(a, st) : launch_precond_fwd_tp<T, RET, false, true>(a, st);
}
int launch_precond_fwd(const PrecondArgs &a, bool bf16_io, hipStream_t st) {
    const int ret = a.retention ? (a.ret_vec ? 2 : 1) : 0;
    if (ret == 2) return bf16_io ? launch_precond_fwd_t<bf16, 2>(a, st) : launch_precond_fwd_t<float, 2>(a, st);
    if (ret == 1) return bf16_io ? launch_precond_fwd_t<bf16, 1>(a, st) : launch_precond_fwd_t<float, 1>(a, st);
    return bf16_io ? launch_precond_fwd_t<bf16, 0>(a, st) : launch_precond_fwd_t<float, 0>(a, st);
}

}  // namespace osdn
