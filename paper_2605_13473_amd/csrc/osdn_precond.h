// Shared pieces of the phase-1 kernels (preconditioner sweep and its reverse).
#pragma once
#include "osdn_kernels.h"

#include <cfloat>

namespace osdn {

constexpr int P1_MAX_SWEEPS = 66;       // 64 guarantee exactness
constexpr float P1_TOL = 1e-6f;         // relative agreement of the inner products between sweeps (forward)
constexpr float P1_TOL_BWD = 1e-7f;     // ... of sigma in the reverse sweep, whose errors add up in the adjoint of d
constexpr float PIECE_TOL = P1_TOL;     // ... of d at the start of a piece between sweeps over a sequence
constexpr float PIECE_TOL_BWD = 5e-7f;  // ... of its adjoint at the end of a piece (of the largest coordinate; such errors do not add up)
constexpr int PB = 8;                   // tokens per LDS prefetch block in the sequential loops

// projection onto [lo, hi] as one median-of-three (lo = -inf, hi = +inf when there is none)
__device__ __forceinline__ float clip3(float x, float lo, float hi) { return __builtin_amdgcn_fmed3f(x, lo, hi); }
// the affine step before projection, written once so that forward and replay round identically
template <bool HAS_RET>
__device__ __forceinline__ float d_bar(float r, float d, float step, float s) {
    return HAS_RET ? __builtin_fmaf(step, s, r * d) : __builtin_fmaf(step, s, d);
}
// Without retention the forward sweep marks a chunk, by the sign of its tokens' sum k^2, if a replay of the tokens one after the other
// (lands_inside, below) finds all of them inside the box: it was swept without the box, so that every c >= 0 and d rose, and d ends at or
// below this bound.  At the lower face, where d begins, rounding then does not matter; at the upper one the sums over runs and the
// replay may differ by the rounding of 64 sums each, 8e-6 of the largest |d|, which is at most that of the larger face.  (No lower
// face: -infinity, and nothing is marked.)
__device__ __forceinline__ float mark_bound(float lo, float hi) {
    return isinf(hi) ? FLT_MAX : hi - 2e-5f * fmaxf(fabsf(lo), fabsf(hi));
}
// Did the step land inside the box (the projection's gradient mask)?  Decided from the signs
// of (r d - face) + step s, each evaluated with a single rounding at its own scale, rather
// than by comparing the rounded sum with the face: a coordinate that sits on a face, or
// comes within an ulp of it, is then told apart from one pushed across it by less than an ulp.
template <bool HAS_RET>
__device__ __forceinline__ bool lands_inside(float r, float d, float step, float s, float lo, float hi) {
    const float above_lo = HAS_RET ? __builtin_fmaf(r, d, -lo) : d - lo;
    const float above_hi = HAS_RET ? __builtin_fmaf(r, d, -hi) : d - hi;
    return __builtin_fmaf(step, s, above_lo) >= 0.f && __builtin_fmaf(step, s, above_hi) <= 0.f;
}
__device__ __forceinline__ void store_vec(float *dst, const float (&v)[4]) {
    *reinterpret_cast<f32x4 *>(dst) = f32x4{v[0], v[1], v[2], v[3]};
}
__device__ __forceinline__ void store_vec(bf16 *dst, const float (&v)[8]) {
    bf16x8 o;
#pragma unroll
    for (int e = 0; e < 8; ++e) o[e] = (bf16)v[e];
    *reinterpret_cast<bf16x8 *>(dst) = o;
}
__device__ __forceinline__ void store_vec(bf16 *dst, const float (&v)[4]) {
    bf16x4 o;
#pragma unroll
    for (int e = 0; e < 4; ++e) o[e] = (bf16)v[e];
    *reinterpret_cast<bf16x4 *>(dst) = o;
}
__device__ __forceinline__ float wave_max(float x) {      // x >= 0
    x = fmaxf(x, dpp_f32<0xB1>(x));
    x = fmaxf(x, dpp_f32<0x4E>(x));
    x = fmaxf(x, dpp_f32<0x141>(x));
    x = fmaxf(x, dpp_f32<0x140>(x));
    x = fmaxf(x, dpp_f32<0x142, 0xA>(x));      // rows that are not written keep old = 0 <= x
    x = fmaxf(x, dpp_f32<0x143, 0xC>(x));
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, x), 63));
}
// One workgroup = 8 wavefronts, two per SIMD.
constexpr int P1T = 512, P1W = P1T / 64;

// partner lane ^ 4 inside a row of 16 lanes: two DPP moves (row_shl:4 into lanes 0-3 and 8-11 of
// every row, row_shr:4 into the others)
__device__ __forceinline__ float lane_xor4(float x) {
    const int xi = __builtin_bit_cast(int, x);
    int t = __builtin_amdgcn_update_dpp(0, xi, 0x104, 0xF, 0x5, false);
    t = __builtin_amdgcn_update_dpp(t, xi, 0x114, 0xF, 0xA, false);
    return __builtin_bit_cast(float, t);
}
// Every lane holds TS values v[0..TS); returns to lane l the sum of v[l % TS] over the group of
// TS lanes it belongs to (the 64 / TS partial sums per value are left to the caller).
template <int TS>
__device__ __forceinline__ float lane_fold(const float (&v)[TS], int lane) {
    static_assert(TS == 16 || TS == 8, "run length");
    // after the step with lane bit b, a lane keeps the values whose index has bit b equal to
    // its own and adds the partner lane's copy of them: the count halves, the group doubles
    float w[TS / 2], x[TS / 4], y[TS / 8];
    const bool b0 = lane & 1, b1 = lane & 2, b2 = lane & 4, b3 = lane & 8;
#pragma unroll
    for (int m = 0; m < TS / 2; ++m)
        w[m] = (b0 ? v[2 * m + 1] : v[2 * m]) + dpp_f32<0xB1>(b0 ? v[2 * m] : v[2 * m + 1]);     // lane ^ 1
#pragma unroll
    for (int m = 0; m < TS / 4; ++m)
        x[m] = (b1 ? w[2 * m + 1] : w[2 * m]) + dpp_f32<0x4E>(b1 ? w[2 * m] : w[2 * m + 1]);     // lane ^ 2
#pragma unroll
    for (int m = 0; m < TS / 8; ++m)
        y[m] = (b2 ? x[2 * m + 1] : x[2 * m]) + lane_xor4(b2 ? x[2 * m] : x[2 * m + 1]);         // lane ^ 4
    if (TS == 8) return y[0];                  // value lane % 8, summed over its 8 lanes
    return (b3 ? y[TS / 8 - 1] : y[0]) + dpp_f32<0x128>(b3 ? y[0] : y[TS / 8 - 1]);   // lane ^ 8 (row_ror:8)
}
// the same for 8 values, carried on to the sum over the whole wavefront: every lane gets the
// total of v[lane % 8] (fixed order of additions)
__device__ __forceinline__ float lane_fold8_all(const float (&v)[8], int lane) {
    float y = lane_fold<8>(v, lane);
    y += dpp_f32<0x128>(y);
    return add_xor32(add_xor16(y));
}
// Every lane holds the values v[0..8) of eight tokens; returns to every lane the sum over the wavefront
// of the token fold_token(lane).  The wide steps come first: a swap of halves (rows) between two
// values and one add leave a register with one value in either half (every other row), two
// instructions where selecting by lane bit takes three; then row rotations and mirrors into half of
// the banks.  17 instructions.
__device__ __forceinline__ int fold_token(int lane) {
    return 4 * (lane >> 3 & 1) + 2 * (lane >> 4 & 1) + (lane >> 5);
}
__device__ __forceinline__ constexpr int fold_lane(int token) {      // a lane that gets this token
    return (token >> 2) * 8 + (token >> 1 & 1) * 16 + (token & 1) * 32;
}
__device__ __forceinline__ float fold_tokens(const float (&v)[8]) {
    float w[4], y[2];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        float a = v[2 * i], b = v[2 * i + 1];
        asm("s_nop 1\n\tv_permlane32_swap_b32 %0, %1" : "+v"(a), "+v"(b));
        w[i] = a + b;
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        float a = w[2 * i], b = w[2 * i + 1];
        asm("s_nop 1\n\tv_permlane16_swap_b32 %0, %1" : "+v"(a), "+v"(b));
        y[i] = a + b;
    }
    float x = y[0] + dpp_f32<0x128>(y[0]);                                                                    // row_ror:8
    asm("s_nop 1\n\tv_add_f32_dpp %0, %1, %1 row_ror:8 row_mask:0xf bank_mask:0xc" : "+v"(x) : "v"(y[1]));
    x += dpp_f32<0x141>(x);                                                                                   // row_half_mirror
    x += dpp_f32<0xB1>(x);
    x += dpp_f32<0x4E>(x);
    return x;
}
__device__ __forceinline__ float lane_bcast(float x, int src_lane) {     // src_lane uniform
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, x), src_lane));
}
// ---- sweeps over a chunk in runs ------------------------------------------------------------
// The sequential kernels of both directions cut a chunk into 8 runs of 8 tokens, one wavefront per run,
// K / 64 adjacent coordinates per lane.
constexpr int RUN = 8;                           // tokens per run (fold_tokens takes eight); C / RUN runs = wavefronts
constexpr int P1F = C / RUN * 64;                // threads

// CPT adjacent elements of type T <-> floats, as one memory access
template <typename T, int CPT> struct Pack;
template <> struct Pack<bf16, 2> {
    typedef uint32_t Raw;
    static __device__ __forceinline__ void unpack(Raw w, float (&o)[2]) {
        o[0] = __builtin_bit_cast(float, w << 16);
        o[1] = __builtin_bit_cast(float, w & 0xffff0000u);
    }
    static __device__ __forceinline__ Raw pack(const float (&v)[2]) {
        const uint32_t lo = __builtin_bit_cast(unsigned short, (bf16)v[0]);
        const uint32_t hi = __builtin_bit_cast(unsigned short, (bf16)v[1]);
        return lo | (hi << 16);
    }
};
template <> struct Pack<bf16, 1> {
    typedef bf16 Raw;
    static __device__ __forceinline__ void unpack(Raw w, float (&o)[1]) { o[0] = (float)w; }
    static __device__ __forceinline__ Raw pack(const float (&v)[1]) { return (bf16)v[0]; }
};
template <> struct Pack<float, 2> {
    typedef float Raw __attribute__((ext_vector_type(2)));
    static __device__ __forceinline__ void unpack(Raw w, float (&o)[2]) { o[0] = w.x; o[1] = w.y; }
    static __device__ __forceinline__ Raw pack(const float (&v)[2]) { return Raw{v[0], v[1]}; }
};
template <> struct Pack<float, 1> {
    typedef float Raw;
    static __device__ __forceinline__ void unpack(Raw w, float (&o)[1]) { o[0] = w; }
    static __device__ __forceinline__ Raw pack(const float (&v)[1]) { return v[0]; }
};

// ---- a chunk of the recurrence in solved form ---------------------------------------------
// Where a chunk of 64 tokens has no retention and no coordinate meets the box, both sweeps are
// linear in the K-vector they carry (d forward, its adjoint backward) and couple the tokens only
// through 64 scalars (the inner products <d_t, s_t>, resp. sigma_t = <s_t, abar_t>), which solve a
// unit triangular 64 x 64 system built from the Gram matrix of the squared keys.  That system is
// inverted for all chunks side by side; what stays sequential per chunk is
//     x = S v + r0 ;  y = M x ;  w = w(y) ;  v' = v + t0 +- S^T w
// (S = the 64 x K tile of squared keys, v the carried vector): two matrix-vector products with
// S and one with the 64 x 64 inverse M.  Thread layouts of a 512-thread workgroup:
//   rows   : thread (i = tid / 8, part = tid % 8) owns coordinates [part * EPT, (part + 1) * EPT) of token i
//            (resp. columns [8 part, 8 part + 8) of row i of M); sums over the 8 lanes of a token
//   columns: thread (c = tid / NG, tg = tid % NG) owns tokens u * NG + tg of coordinate c; sums over NG lanes
template <int K> struct Lin {
    static constexpr int EPT = K / 8;
    static constexpr int NG = P1T / K;
    static constexpr int LD = K + (K == 128 ? 8 : 4);     // row stride of the s tile: column reads of a half-wave hit 32 banks
    static constexpr int VSTR = EPT + 4;                  // a thread's slice of a K-vector: slices start 16 bytes off a bank period
    static constexpr int XSTR = 12;                       // ... of a 64-vector (8 entries per slice)
    static __device__ __forceinline__ int vidx(int c) { return (c / EPT) * VSTR + c % EPT; }
    // Position of coordinate c inside a row of the s tile: the 16-byte groups of a 16-coordinate
    // slice are rotated by half the slice index, so that the 8 threads that write one group each
    // for 8 adjacent slices (128 bytes apart) cover all 32 banks; column reads stay conflict-free.
    static __device__ __forceinline__ int swz(int c) { return (c & ~12) | ((((c >> 2) + (c >> 5)) & 3) << 2); }
    static __device__ __forceinline__ int xidx(int i) { return (i >> 3) * XSTR + (i & 7); }
};
// sum over the 8 (4) adjacent lanes of an aligned group, returned to all of them
__device__ __forceinline__ float sum_lanes8(float x) {
    x += dpp_f32<0xB1>(x);
    x += dpp_f32<0x4E>(x);
    x += lane_xor4(x);
    return x;
}
__device__ __forceinline__ float sum_lanes4(float x) {
    x += dpp_f32<0xB1>(x);
    x += dpp_f32<0x4E>(x);
    return x;
}

// ---- where the backward kernels of phase 1 read ---------------------------------------------
// k, beta and retention of chunk n, head h: the caller's rows, or the tile of a ragged last chunk; tokens are H rows apart
template <typename T, int K, int RET, bool RAG> struct ChunkIn {
    const T *k;
    const float *beta, *ret;
    __device__ __forceinline__ ChunkIn(const PrecondBwdArgs &a, int b, int n, int h) {
        const int tile = a.rows.tail<RAG>(b, n);
        const size_t row = (tile < 0 ? a.rows.first<RAG>(b, n) : (size_t)tile * C) * a.H + h;
        k = static_cast<const T *>(tile < 0 ? a.k : a.k_tail) + row * K;
        beta = (tile < 0 ? a.beta : a.beta_tail) + row;
        ret = RET ? (tile < 0 ? a.retention : a.ret_tail) + row * (RET == 2 ? K : 1) : nullptr;
    }
};
// The same for a kernel that walks the chunks of one chain: base(n) as above, without a table.
template <typename T, int K, int RET, bool RAG> struct ChainIn {
    const T *k, *k_tail;
    const float *beta, *beta_tail, *ret, *ret_tail;
    size_t chunk_rows;
    int tail;                                    // the ragged chunk, or one that does not exist
    __device__ __forceinline__ ChainIn(const PrecondBwdArgs &a, int b, int n0, int h) {
        const ChainRows<RAG> rows(a.rows, a.seq_chunks, b, n0);
        const size_t u0 = (rows.batch + (size_t)(long long)rows.base) * a.H + h, t0 = (size_t)b * C * a.H + h;
        constexpr int RK = RET == 2 ? K : 1;
        chunk_rows = (size_t)C * a.H;
        tail = (rows.end - rows.base) % C ? (rows.end - rows.base) / C : -1;
        k = static_cast<const T *>(a.k) + u0 * K; k_tail = static_cast<const T *>(a.k_tail) + t0 * K;
        beta = a.beta + u0; beta_tail = a.beta_tail + t0;
        ret = RET ? a.retention + u0 * RK : nullptr; ret_tail = RET ? a.ret_tail + t0 * RK : nullptr;
    }
    __device__ __forceinline__ const T *k_of(int n) const { return RAG && n == tail ? k_tail : k + (size_t)n * chunk_rows * K; }
    __device__ __forceinline__ const float *beta_of(int n) const { return RAG && n == tail ? beta_tail : beta + (size_t)n * chunk_rows; }
    __device__ __forceinline__ const float *ret_of(int n) const { return RAG && n == tail ? ret_tail : ret + (size_t)n * chunk_rows * (RET == 2 ? K : 1); }
};

}  // namespace osdn
