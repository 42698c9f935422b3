// Recurrent (token-by-token) form of the OSDN update for short inputs: the decode step of
// Appendix K (gate, preconditioner update with the clip, rank-one write, read) for 1..64
// tokens in one launch, with the state slice of a workgroup held in registers throughout.
//
//   k~_t = d_t (.) k_t
//   S   <- alpha_t S ;  e = beta_t (v_t - S k_t) ;  S <- S + e k~_t^T ;  o_t = scale S q_t
//   (alpha_t a scalar, or one gate per key channel: S <- S Diag(alpha_t), the online-scaled
//   KDA recurrence in this library's V x K orientation of the state)
//   d_{t+1} = clip(r_t d_t + eta b'(1 - b' p)/n s),  s = k_t^2, n = max(sum s, eps), p = <d_t, s>
//
// step_kernel (one token; two or three of few chains): a workgroup of four wavefronts owns 16 rows of S of one (batch, head); a wavefront owns 4 of
// them, a lane K / 64 adjacent coordinates.  Every wavefront keeps its own copy of d (the
// update needs two sums over the coordinates, like the two inner products per row).
#include "osdn_precond.h"

namespace osdn {

constexpr int STEP_T = 256, STEP_RPW = 4, STEP_ROWS = (STEP_T / 64) * STEP_RPW;   // 16 rows per workgroup

// RET: 0 = no retention, 1 = one gate per (token, head), 2 = one per coordinate; GV: one state
// gate per key channel
template <typename T, int K, int RET, bool GV>
__global__ __launch_bounds__(STEP_T) void step_kernel(StepArgs a) {
    constexpr bool HAS_RET = RET != 0, RET_VEC = RET == 2;
    constexpr int CPT = K / 64;
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int nslice = a.V / STEP_ROWS;
    const int slice = blockIdx.x % nslice, chain = blockIdx.x / nslice;
    const int b = chain / a.H, h = chain % a.H;
    const size_t bh = (size_t)b * a.H + h;
    const int v0 = slice * STEP_ROWS + wave * STEP_RPW;
    const int c0 = lane * CPT;
    const bool project = a.d_min <= a.d_max;
    const float lo = project ? a.d_min : -INFINITY, hi = project ? a.d_max : INFINITY;

    float d[CPT], Sr[STEP_RPW][CPT];
#pragma unroll
    for (int e = 0; e < CPT; ++e) d[e] = a.d_in ? a.d_in[bh * K + c0 + e] : 1.f;
#pragma unroll
    for (int r = 0; r < STEP_RPW; ++r)
#pragma unroll
        for (int e = 0; e < CPT; ++e) Sr[r][e] = a.S_in ? a.S_in[(bh * a.V + v0 + r) * K + c0 + e] : 0.f;

    const T *qg = static_cast<const T *>(a.q), *kg = static_cast<const T *>(a.k), *vg = static_cast<const T *>(a.v);
    T *og = static_cast<T *>(a.o);
    for (int t = 0; t < a.T; ++t) {
        const size_t th = ((size_t)b * a.T + t) * a.H + h;
        float kf[CPT], qf[CPT], kt[CPT];
#pragma unroll
        for (int e = 0; e < CPT; ++e) {
            kf[e] = to_f32(kg[th * K + c0 + e]);
            qf[e] = to_f32(qg[th * K + c0 + e]);
            kt[e] = d[e] * kf[e];
        }
        const float bet = a.beta[th];
        float alpha[CPT];                           // one state gate per (token, head), or one per key channel
#pragma unroll
        for (int e = 0; e < CPT; ++e)
            alpha[e] = a.log_alpha ? __expf(GV ? a.log_alpha[th * K + c0 + e] : a.log_alpha[th]) : 1.f;
        float ret[CPT];                             // one gate per (token, head), or one per coordinate
#pragma unroll
        for (int e = 0; e < CPT; ++e)
            ret[e] = HAS_RET ? (RET_VEC ? a.retention[th * K + c0 + e] : a.retention[th]) : 1.f;
        float orow = 0.f;                           // lane r < 4 ends with the output of row v0 + r
#pragma unroll
        for (int r = 0; r < STEP_RPW; ++r) {
            float dot = 0.f;
#pragma unroll
            for (int e = 0; e < CPT; ++e) { Sr[r][e] *= alpha[e]; dot = __builtin_fmaf(Sr[r][e], kf[e], dot); }
            dot = wave_sum(dot);
            const float ev = bet * (to_f32(vg[th * a.V + v0 + r]) - dot);
            float od = 0.f;
#pragma unroll
            for (int e = 0; e < CPT; ++e) { Sr[r][e] = __builtin_fmaf(ev, kt[e], Sr[r][e]); od = __builtin_fmaf(Sr[r][e], qf[e], od); }
            od = wave_sum(od);
            if (lane == r) orow = od;
        }
        if (lane < STEP_RPW) og[th * a.V + v0 + lane] = from_f32<T>(a.scale * orow);
        // the preconditioner moves after the token has used it
        float sn = 0.f, sp = 0.f, sv[CPT];
#pragma unroll
        for (int e = 0; e < CPT; ++e) { sv[e] = kf[e] * kf[e]; sn += sv[e]; sp = __builtin_fmaf(sv[e], d[e], sp); }
        sn = wave_sum(sn);
        sp = wave_sum(sp);
        const float nn = fmaxf(sn, a.eps);
        const float bp = a.beta_aware ? bet : 1.f;
        const float cb = a.eta * bp / nn;
        const float step = cb - cb * bp * sp;
#pragma unroll
        for (int e = 0; e < CPT; ++e) d[e] = clip3(d_bar<HAS_RET>(ret[e], d[e], step, sv[e]), lo, hi);
    }
#pragma unroll
    for (int r = 0; r < STEP_RPW; ++r)
#pragma unroll
        for (int e = 0; e < CPT; ++e) a.S_out[(bh * a.V + v0 + r) * K + c0 + e] = Sr[r][e];
    if (slice == 0 && wave == 0) {
#pragma unroll
        for (int e = 0; e < CPT; ++e) a.d_out[bh * K + c0 + e] = d[e];
    }
}

// ---- several tokens a call -----------------------------------------------------------------
// Bound by vector instruction issue and by the chain token -> token, not by memory: the state is
// read and written once per call.  step_kernel repeats the update of d in each of the 32
// wavefronts of a chain, waits for a token's loads when it begins the token, and spends six lane
// moves on the sum of one row.  Here one wavefront of the workgroup (the producer) walks d and
// leaves k, k~, q, v and the gates of STEP_TB tokens in LDS, a block of tokens ahead of the
// others, with the loads of the block after that in flight; and 16 lanes own a row, so that a
// lane move serves four rows at once.  Every sum is formed in the order of step_kernel (adjacent
// pairs of coordinates, then a binary tree), so a call of T tokens equals T calls of one bit for
// bit.  128 chains of 128 x 128, 16 tokens: 29.6 -> 14.2 us (state in and out at copy speed: 3.3;
// its vector instructions, 70 per 4 rows and token, need about 7); 64 tokens 111 -> 42 us.
constexpr int STEP_TB = 4, STEP_CW = 4;                          // tokens of a block, wavefronts with rows of S

struct __attribute__((packed, aligned(4))) Quad { float v[4]; };   // the caller's state is aligned as floats are

// sums over 16 lanes, every lane with the result: a binary tree over adjacent lanes
__device__ __forceinline__ float row16_sum(float x) {
    x += dpp_f32<0xB1>(x);         // quad_perm [1,0,3,2]
    x += dpp_f32<0x4E>(x);         // quad_perm [2,3,0,1]
    x += dpp_f32<0x141>(x);        // row_half_mirror
    return x + dpp_f32<0x140>(x);  // row_mirror
}
// a lane's part of <a, b>, in the order of step_kernel
template <int CPL>
__device__ __forceinline__ float lane_dot(const float *a, const float *b) {
    float p[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        if constexpr (CPL == 8) p[i] = __builtin_fmaf(a[2 * i + 1], b[2 * i + 1], a[2 * i] * b[2 * i]);
        else p[i] = __builtin_fmaf(a[i], b[i], 0.f);      // (a rounded product: nothing to contract)
    }
    return (p[0] + p[1]) + (p[2] + p[3]);
}

// M rows of S per 16 lanes: 16 M rows per workgroup
template <typename T, int K, int RET, bool GV, int M>
__global__ __launch_bounds__(64 * (STEP_CW + 1)) void step_tokens_kernel(StepArgs a) {
    constexpr bool HAS_RET = RET != 0, RET_VEC = RET == 2;
    constexpr int CPT = K / 64, CPL = K / 16, HALF = K / CPL * 4, ROWS = STEP_CW * 4 * M;
    // coordinate c of a token sits at (c / 4 % (CPL / 4)) * HALF + c / CPL * 4 + c % 4: what the 16
    // lanes of a row read at one time is contiguous
    __shared__ __align__(16) float ks[2][STEP_TB][K], kts[2][STEP_TB][K], qs[2][STEP_TB][K];
    __shared__ __align__(16) float als[2][STEP_TB][GV ? K : 1];
    __shared__ float vs[2][STEP_TB][ROWS], bs[2][STEP_TB];
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int nslice = a.V / ROWS;
    const int slice = blockIdx.x % nslice, chain = blockIdx.x / nslice;
    const int b = chain / a.H, h = chain % a.H;
    const size_t bh = (size_t)b * a.H + h;
    const int v0 = slice * ROWS;
    const int nblk = (a.T + STEP_TB - 1) / STEP_TB;

    if (wave == STEP_CW) {                          // the producer
        const T *qg = static_cast<const T *>(a.q), *kg = static_cast<const T *>(a.k), *vg = static_cast<const T *>(a.v);
        const int c0 = lane * CPT;
        const int pos = c0 / 4 % (CPL / 4) * HALF + c0 / CPL * 4 + c0 % 4;
        const bool project = a.d_min <= a.d_max;
        const float lo = project ? a.d_min : -INFINITY, hi = project ? a.d_max : INFINITY;
        float d[CPT];
#pragma unroll
        for (int e = 0; e < CPT; ++e) d[e] = a.d_in ? a.d_in[bh * K + c0 + e] : 1.f;
        T kr[STEP_TB][CPT], qr[STEP_TB][CPT], vr[STEP_TB];
        float br[STEP_TB], gr[STEP_TB][GV ? CPT : 1], rr[STEP_TB][RET_VEC ? CPT : 1];
        auto request = [&](int blk) {               // tokens past the end: the last token again
#pragma unroll
            for (int i = 0; i < STEP_TB; ++i) {
                const int t = blk * STEP_TB + i < a.T ? blk * STEP_TB + i : a.T - 1;
                const size_t th = ((size_t)b * a.T + t) * a.H + h;
#pragma unroll
                for (int e = 0; e < CPT; ++e) { kr[i][e] = kg[th * K + c0 + e]; qr[i][e] = qg[th * K + c0 + e]; }
                vr[i] = vg[th * a.V + v0 + (lane & (ROWS - 1))];
                br[i] = a.beta[th];
                if constexpr (GV) {
#pragma unroll
                    for (int e = 0; e < CPT; ++e) gr[i][e] = a.log_alpha[th * K + c0 + e];
                } else {
                    gr[i][0] = a.log_alpha ? a.log_alpha[th] : 0.f;
                }
                if constexpr (RET_VEC) {
#pragma unroll
                    for (int e = 0; e < CPT; ++e) rr[i][e] = a.retention[th * K + c0 + e];
                } else {
                    rr[i][0] = HAS_RET ? a.retention[th] : 1.f;
                }
            }
        };
        request(0);
        for (int blk = 0; blk <= nblk; ++blk) {     // block blk is made while block blk - 1 is used
            if (blk < nblk) {
                const int buf = blk & 1, nt = a.T - blk * STEP_TB;
                T kc[STEP_TB][CPT];
                float sv[STEP_TB][CPT], cb[STEP_TB], bp[STEP_TB], rc[STEP_TB][RET_VEC ? CPT : 1];
#pragma unroll
                for (int i = 0; i < STEP_TB; ++i) {
                    float sn = 0.f;
#pragma unroll
                    for (int e = 0; e < CPT; ++e) {
                        kc[i][e] = kr[i][e];
                        const float kf = to_f32(kr[i][e]);
                        ks[buf][i][pos + e] = kf;
                        qs[buf][i][pos + e] = to_f32(qr[i][e]);
                        sv[i][e] = kf * kf;
                        sn += sv[i][e];
                    }
                    if (lane < ROWS) vs[buf][i][lane] = to_f32(vr[i]);
                    if constexpr (GV) {
#pragma unroll
                        for (int e = 0; e < CPT; ++e) als[buf][i][pos + e] = __expf(gr[i][e]);
                    }
                    else if (lane == 0) als[buf][i][0] = a.log_alpha ? __expf(gr[i][0]) : 1.f;
                    if (lane == 0) bs[buf][i] = br[i];
#pragma unroll
                    for (int e = 0; e < (RET_VEC ? CPT : 1); ++e) rc[i][e] = rr[i][e];
                    const float nn = fmaxf(wave_sum(sn), a.eps);
                    bp[i] = a.beta_aware ? br[i] : 1.f;
                    cb[i] = a.eta * bp[i] / nn;
                }
                if (blk + 1 < nblk) request(blk + 1);
#pragma unroll
                for (int i = 0; i < STEP_TB; ++i) {
                    if (i < nt) {
                        float sp = 0.f;
#pragma unroll
                        for (int e = 0; e < CPT; ++e) {
                            kts[buf][i][pos + e] = d[e] * to_f32(kc[i][e]);
                            sp = __builtin_fmaf(sv[i][e], d[e], sp);
                        }
                        sp = wave_sum(sp);
                        const float step = cb[i] - cb[i] * bp[i] * sp;
#pragma unroll
                        for (int e = 0; e < CPT; ++e)
                            d[e] = clip3(d_bar<HAS_RET>(rc[i][RET_VEC ? e : 0], d[e], step, sv[i][e]), lo, hi);
                    }
                }
            }
            __syncthreads();
        }
        if (slice == 0) {
#pragma unroll
            for (int e = 0; e < CPT; ++e) a.d_out[bh * K + c0 + e] = d[e];
        }
        return;
    }

    // rows r0 .. r0 + M - 1 of the slice, coordinates c0 .. c0 + CPL - 1
    const int l16 = lane & 15, r0 = wave * 4 * M + (lane >> 4) * M, c0 = l16 * CPL;
    float S[M][CPL];
#pragma unroll
    for (int m = 0; m < M; ++m)
#pragma unroll
        for (int j = 0; j < CPL / 4; ++j) {
            Quad x{};
            if (a.S_in) x = *reinterpret_cast<const Quad *>(a.S_in + (bh * a.V + v0 + r0 + m) * K + c0 + 4 * j);
#pragma unroll
            for (int e = 0; e < 4; ++e) S[m][4 * j + e] = x.v[e];
        }
    T *og = static_cast<T *>(a.o) + v0 + r0;
    auto read = [&](const float *row, float (&x)[CPL]) {
#pragma unroll
        for (int j = 0; j < CPL / 4; ++j) {
            const f32x4 w = *reinterpret_cast<const f32x4 *>(row + j * HALF + l16 * 4);
#pragma unroll
            for (int e = 0; e < 4; ++e) x[4 * j + e] = w[e];
        }
    };
    __syncthreads();                                // block 0 is there
    auto token = [&](int buf, int i) {           // lane m of a row's 16 returns the output of its row m
        float kf[CPL], kt[CPL], qf[CPL], al[CPL], od[M];
        read(ks[buf][i], kf);
        read(kts[buf][i], kt);
        read(qs[buf][i], qf);
        if constexpr (GV) read(als[buf][i], al);
        else {
#pragma unroll
            for (int e = 0; e < CPL; ++e) al[e] = als[buf][i][0];
        }
        const float bet = bs[buf][i];
#pragma unroll
        for (int m = 0; m < M; ++m) {
#pragma unroll
            for (int e = 0; e < CPL; ++e) S[m][e] *= al[e];
            const float ev = bet * (vs[buf][i][r0 + m] - row16_sum(lane_dot<CPL>(S[m], kf)));
#pragma unroll
            for (int e = 0; e < CPL; ++e) S[m][e] = __builtin_fmaf(ev, kt[e], S[m][e]);
            od[m] = row16_sum(lane_dot<CPL>(S[m], qf));
        }
        float out = od[0];
#pragma unroll
        for (int m = 1; m < M; ++m) out = l16 == m ? od[m] : out;
        return a.scale * out;
    };
    auto put = [&](int t, float out) { og[(((size_t)b * a.T + t) * a.H + h) * a.V + l16] = from_f32<T>(out); };
    for (int blk = 0; blk < nblk; ++blk) {
        const int buf = blk & 1, nt = a.T - blk * STEP_TB;
        if (nt >= STEP_TB) {                        // no branch between the tokens: reads of the next ones go ahead
            float out[STEP_TB];
#pragma unroll
            for (int i = 0; i < STEP_TB; ++i) out[i] = token(buf, i);
            if (l16 < M) {
#pragma unroll
                for (int i = 0; i < STEP_TB; ++i) put(blk * STEP_TB + i, out[i]);
            }
        } else {
            for (int i = 0; i < nt; ++i) {
                const float out = token(buf, i);
                if (l16 < M) put(blk * STEP_TB + i, out);
            }
        }
        __syncthreads();
    }
#pragma unroll
    for (int m = 0; m < M; ++m)
#pragma unroll
        for (int j = 0; j < CPL / 4; ++j) {
            Quad x;
#pragma unroll
            for (int e = 0; e < 4; ++e) x.v[e] = S[m][4 * j + e];
            *reinterpret_cast<Quad *>(a.S_out + (bh * a.V + v0 + r0 + m) * K + c0 + 4 * j) = x;
        }
}

template <typename T, int RET, bool GV, int M>
static void launch_step_tokens(const StepArgs &a, hipStream_t st) {
    const dim3 grid(a.B * a.H * (a.V / (4 * STEP_CW * M))), block(64 * (STEP_CW + 1));
    if (a.K == 64) hipLaunchKernelGGL((step_tokens_kernel<T, 64, RET, GV, M>), grid, block, 0, st, a);
    else hipLaunchKernelGGL((step_tokens_kernel<T, 128, RET, GV, M>), grid, block, 0, st, a);
}
// Which form.  `few`: workgroups of 16 rows are at most two a CU; then the dependent chain of a token
// counts, above that instruction issue does, and 32 rows per workgroup share one producer (4 chains of
// 64 tokens 28 against 33 us, 32 chains of 16: 9.5 against 10.8, 64 chains of 16: 10.9 against 11.2;
// 128 chains of 16 tokens level; 1024 chains of 8 tokens 49 against 42 us).  One token: step_kernel
// already moves the state at copy speed.  Two or three tokens of few chains: the producer's head
// start is not earned back (8 chains of 2 tokens 3.8 against 4.3 us; of many chains the wide form
// wins from two tokens on: 4096 chains 126 against 102 us).
template <typename T, int RET, bool GV>
static int launch_step_t(const StepArgs &a, hipStream_t st) {
    if (a.K != 64 && a.K != 128) return -1;
    const bool few = (long long)a.B * a.H * (a.V / 16) <= 512;
    if (a.T >= (few ? 4 : 2)) {
        if (few) launch_step_tokens<T, RET, GV, 1>(a, st);
        else launch_step_tokens<T, RET, GV, 2>(a, st);
        return 0;
    }
    const dim3 grid(a.B * a.H * (a.V / STEP_ROWS)), block(STEP_T);
    if (a.K == 64) hipLaunchKernelGGL((step_kernel<T, 64, RET, GV>), grid, block, 0, st, a);
    else hipLaunchKernelGGL((step_kernel<T, 128, RET, GV>), grid, block, 0, st, a);
    return 0;
}
template <typename T>
static int launch_step_io(const StepArgs &a, hipStream_t st) {
    const int ret = a.retention ? (a.ret_vec ? 2 : 1) : 0;
    const bool gv = a.log_alpha && a.gate_vec;
    if (ret == 2) return gv ? launch_step_t<T, 2, true>(a, st) : launch_step_t<T, 2, false>(a, st);
    if (ret == 1) return gv ? launch_step_t<T, 1, true>(a, st) : launch_step_t<T, 1, false>(a, st);
    return gv ? launch_step_t<T, 0, true>(a, st) : launch_step_t<T, 0, false>(a, st);
}
int launch_step(const StepArgs &a, bool bf16_io, hipStream_t st) {
    return bf16_io ? launch_step_io<bf16>(a, st) : launch_step_io<float>(a, st);
}

}  // namespace osdn
