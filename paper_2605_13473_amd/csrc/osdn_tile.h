// LDS operand tiles of the chain kernels, filled by direct global -> LDS loads (gfx950).
//
// A direct load moves 16 bytes per lane to consecutive LDS addresses (wave-uniform base + 16 *
// lane), so rows cannot be padded against bank conflicts.  Instead every row of a tile keeps its
// 16-byte groups in a permuted order: group c of row r sits at position c ^ f(r), and the lanes of
// a load fetch the groups in that order.  Measured LDS cycles per wavefront instruction, bf16 rows
// of 256 (128) bytes: fragment read along k 4.2 (4.2) against 32 (16) for unpadded rows and 8 (8)
// for 16 bytes of padding; transpose read 4.2 (4.1) against 16 (8); the best any layout reaches is
// 4.2 and 3.6.
//
// What the loads buy over a copy through registers: no staging registers, no LDS store
// instructions, and a queue that is as deep as the LDS ring.  They are issued and waited for by
// hand: the compiler does not know of them (its own count of outstanding accesses only ever waits
// for too much, never too little), and `wait_vm<N>` returns when all but the newest N vector memory
// accesses of the wavefront are complete (loads and stores retire in order).
#pragma once
#include "osdn_device.h"

namespace osdn {

// position of 16-byte group c of row r inside a tile with ROWB bytes per row
template <int ROWB> struct Swz {
    static_assert(ROWB == 32 || ROWB == 64 || ROWB == 128 || ROWB == 256 || ROWB == 512, "row length");
    static __device__ __forceinline__ uint32_t f(uint32_t r) {
        return ROWB >= 256 ? (r & 15u) : ROWB == 128 ? ((r >> 1) & 7u) : ROWB == 64 ? (((r >> 3) & 1u) << 1) : 0u;
    }
    static __device__ __forceinline__ uint32_t at(uint32_t r, uint32_t c) { return r * ROWB + ((c ^ f(r)) << 4); }
    // f(r + rows) ^ f(r), the same for every r that LdsLoad::init meets
    static __device__ __forceinline__ uint32_t step(uint32_t rows) { return ROWB >= 256 ? rows & 15u : 0u; }
};
// The same for a tile that is read transposed in runs of eight (RunFrag::tr): sixteen lanes take 8 bytes each of four rows and
// four groups next to each other, which lie in sixteen different groups of 256 bytes here.
template <int ROWB> struct SwzRun {
    static_assert(ROWB == 128 || ROWB == 256, "row length");
    static __device__ __forceinline__ uint32_t f(uint32_t r) {
        return ROWB == 256 ? ((r & 3u) << 2) | ((r >> 2) & 3u) : (((r >> 1) & 1u) << 2) | ((r >> 2) & 3u);
    }
    static __device__ __forceinline__ uint32_t at(uint32_t r, uint32_t c) { return r * ROWB + ((c ^ f(r)) << 4); }
    static __device__ __forceinline__ uint32_t step(uint32_t rows) { return ROWB == 256 ? (rows >> 2) & 3u : 0u; }
};

// MFMA fragments from a permuted tile.  kc: the contraction index runs along the row, tr: down the
// rows (bf16: LDS transpose read).  r0 is a multiple of 16; k0 of the MFMA step.
template <typename T, int ROWB> struct TileFrag;
// put stores a 16x16 accumulator tile transposed: its columns become rows r0.., its rows columns c0..
template <int ROWB> struct TileFrag<bf16, ROWB> {
    uint32_t kcl, trl, stl;                     // this lane's offsets for (row 0, k 0)
    __device__ __forceinline__ void init(int lane) {
        const uint32_t row = lane & 15, q = lane >> 4;
        kcl = row * ROWB + ((q ^ Swz<ROWB>::f(row)) << 4);
        stl = row * ROWB + (((q >> 1) ^ Swz<ROWB>::f(row)) << 4) + (q & 1) * 8;
        const uint32_t krow = q * 8 + (row >> 2);
        trl = krow * ROWB + ((((row & 3) >> 1) ^ Swz<ROWB>::f(krow)) << 4) + (row & 1) * 8;
    }
    __device__ __forceinline__ bf16x8 kc(const char *tile, int r0, int k0) const {
        return *reinterpret_cast<const bf16x8 *>(tile + r0 * ROWB + (kcl ^ (uint32_t)(k0 << 1)));
    }
    __device__ __forceinline__ bf16x8 tr(const char *tile, int k0, int r0) const {
        typedef short v4s __attribute__((ext_vector_type(4)));
        typedef __attribute__((address_space(3))) v4s *lds_v4s;
        // the second read is four rows further down, where f differs in one bit
        constexpr uint32_t FLIP = ROWB >= 256 ? 64u : ROWB == 128 ? 32u : 0u;
        const uint32_t o = trl ^ (uint32_t)(r0 << 1);
        const char *p = tile + k0 * ROWB;
        const v4s lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4s)(p + o));
        const v4s hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4s)(p + 4 * ROWB + (o ^ FLIP)));
        return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
    }
    __device__ __forceinline__ void put(char *tile, int r0, int c0, f32x4 acc) const {
        bf16x4 v;
#pragma unroll
        for (int r = 0; r < 4; ++r) v[r] = (bf16)acc[r];
        *reinterpret_cast<bf16x4 *>(tile + r0 * ROWB + (stl ^ (uint32_t)(c0 << 1))) = v;
    }
};
template <int ROWB> struct TileFrag<float, ROWB> {
    uint32_t row, q;
    __device__ __forceinline__ void init(int lane) { row = lane & 15; q = lane >> 4; }
    __device__ __forceinline__ float kc(const char *tile, int r0, int k0) const {
        return *reinterpret_cast<const float *>(tile + Swz<ROWB>::at(r0 + row, (uint32_t)k0 >> 2) + q * 4);
    }
    __device__ __forceinline__ float tr(const char *tile, int k0, int r0) const {
        return *reinterpret_cast<const float *>(tile + Swz<ROWB>::at(k0 + q, ((uint32_t)r0 + row) >> 2) + (row & 3) * 4);
    }
    __device__ __forceinline__ void put(char *tile, int r0, int c0, f32x4 acc) const {
        *reinterpret_cast<f32x4 *>(tile + Swz<ROWB>::at(r0 + row, ((uint32_t)c0 >> 2) + q)) = acc;
    }
};
// Fragments for products whose result is the next product's operand without leaving its registers.  Two accumulator tiles of
// 16 rows cover 32 rows (features, tokens) so that a lane's four rows of either are eight in a row: row m of the tile `half` is
// row 8 (m / 4) + 4 half + m % 4 of the 32.  Rounded, the eight values are the fragment (32 rows along the contraction, 16
// columns) of the next MFMA, and 16 bytes in a row for memory.
template <int ROWB> struct RunFrag {
    uint32_t rowl[2], trl;
    __device__ __forceinline__ void init(int lane) {
        const uint32_t m = lane & 15, q = lane >> 4;
#pragma unroll
        for (int half = 0; half < 2; ++half) rowl[half] = Swz<ROWB>::at((m >> 2) * 8 + half * 4 + (m & 3), q);
        trl = SwzRun<ROWB>::at(q * 8 + (m >> 2), m & 3);
    }
    // rows of `half` of the 32 from r0 on, contraction index from k0 on along the row
    __device__ __forceinline__ bf16x8 rows(const char *tile, int r0, int half, int k0) const {
        return *reinterpret_cast<const bf16x8 *>(tile + r0 * ROWB + (rowl[half] ^ (uint32_t)(k0 << 1)));
    }
    // columns of `half` of the 32 from r0 on, contraction index from k0 on down the rows (a tile permuted by SwzRun)
    __device__ __forceinline__ bf16x8 tr(const char *tile, int k0, int r0, int half) const {
        typedef short v4s __attribute__((ext_vector_type(4)));
        typedef __attribute__((address_space(3))) v4s *lds_v4s;
        const uint32_t o = trl ^ (uint32_t)(r0 << 1);
        const char *p = tile + k0 * ROWB + half * 8;
        const v4s lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4s)(p + o));
        const v4s hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4s)(p + 4 * ROWB + (o ^ 16u)));
        return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
    }
    static __device__ __forceinline__ bf16x8 pack(f32x4 a, f32x4 b) {
        bf16x8 o;
#pragma unroll
        for (int e = 0; e < 4; ++e) { o[e] = (bf16)a[e]; o[4 + e] = (bf16)b[e]; }
        return o;
    }
};
// a whole permuted tile to memory (rows gstride bytes apart), 16 bytes per thread and step
template <int ROWB, int ROWS>
__device__ __forceinline__ void tile_to_global(char *g, uint32_t gstride, const char *tile, int tid, int nthreads) {
    for (int i = tid; i < ROWS * (ROWB / 16); i += nthreads) {
        const uint32_t r = i / (ROWB / 16), c = i % (ROWB / 16);
        *reinterpret_cast<u32x4 *>(g + r * gstride + (c << 4)) = *reinterpret_cast<const u32x4 *>(tile + Swz<ROWB>::at(r, c));
    }
}

// ------------------------------------------------------------ direct loads ----
__device__ __forceinline__ uint32_t lds_offset(const void *p) {      // LDS byte address of a __shared__ object
    return (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const char *)p;
}
// 16 (4) bytes per lane from base + voff (base wave-uniform) to LDS address lds + 16 (4) * lane
__device__ __forceinline__ void load_lds16(const void *base, uint32_t voff, uint32_t lds) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                 :: "s"(lds), "v"(voff), "s"(base) : "m0", "memory");
}
__device__ __forceinline__ void load_lds4(const void *base, uint32_t voff, uint32_t lds) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, %2"
                 :: "s"(lds), "v"(voff), "s"(base) : "m0", "memory");
}
// A line per lane on its way into the L2: 4 bytes of it go to LDS address lds + 4 * lane, where nothing reads them
constexpr int LINE = 128;
__device__ __forceinline__ void touch(const char *p, uint32_t lds) {
    const uintptr_t at = reinterpret_cast<uintptr_t>(p) & ~(uintptr_t)3;
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, off" :: "s"(lds), "v"(at) : "m0", "memory");
}
// all but the newest N vector memory accesses of this wavefront are complete
template <int N> __device__ __forceinline__ void wait_vm() {
    asm volatile("s_waitcnt vmcnt(%0)" :: "n"(N) : "memory");
}

// A [ROWS x ROWB bytes] tile shared by the NW wavefronts of a workgroup; every load covers 1 KB.
template <int ROWB, int ROWS, int NW, typename SW = Swz<ROWB>> struct LdsLoad {
    static constexpr int NI = ROWB * ROWS / 1024;          // loads of the whole tile
    static constexpr int MIN = NI / NW;                    // every wavefront issues at least this many
    static constexpr int RPI = 1024 / ROWB;                // rows per load
    static_assert(NI >= 1 && (NI % NW == 0 || NI < NW), "loads must split evenly over the wavefronts, or be fewer");
    // f(r) repeats every 16 rows: one lane offset serves all loads of a wavefront if they are a multiple of
    // 16 rows apart; with fewer, r + m STEP = r ^ (m STEP) modulo 16 (rows of at least 256 bytes)
    static constexpr int STEP = NW * RPI;
    static_assert(NI <= NW || STEP % 16 == 0 || (ROWB >= 256 && (STEP & (STEP - 1)) == 0), "row permutation");
    uint32_t voff;
    __device__ __forceinline__ void init(uint32_t gstride, int wave, int lane) {     // gstride: bytes between rows in memory
        const uint32_t r = wave * RPI + lane / (ROWB / 16), ph = lane % (ROWB / 16);
        voff = r * gstride + ((ph ^ SW::f(r)) << 4);
    }
    // wide: the source is 16-byte aligned (only a caller's tensor may not be: then the tile goes
    // through registers, which is slower and does the same)
    // rot: the wavefront starts with its rot-th load.  Workgroups that read the same tile at the same time
    // start in different places, so that together they have more of it in flight and find the rest in the
    // L2 (8 workgroups per tile, 40 KB a step from HBM beside stores of 8 KB: 1.05 -> 0.83 us per step).
    __device__ __forceinline__ void issue(char *tile, const char *g, uint32_t gstride, int wave, int lane, int rot = 0, bool wide = true, int last = ROWS - 1) const {
        const uint32_t lds = lds_offset(tile);
        constexpr int M = (NI + NW - 1) / NW;
        static_assert((M & (M - 1)) == 0, "loads per wavefront");
#pragma unroll
        for (int j = 0; j < M; ++j) {
            const int m = (j + rot) & (M - 1), i = wave + m * NW;
            if (NI % NW == 0 || i < NI) {
                const char *gm = g + (size_t)m * NW * RPI * gstride;
                uint32_t vo = voff ^ (SW::step(m * STEP) << 4);
                if (last < ROWS - 1) {              // (uniform) rows behind the last one that exists repeat it
                    const uint32_t r = i * RPI + lane / (ROWB / 16), ph = lane % (ROWB / 16);
                    gm = g;
                    vo = min(r, (uint32_t)last) * gstride + ((ph ^ SW::f(r)) << 4);
                }
                if (wide) load_lds16(gm, vo, lds + i * 1024);
                else *reinterpret_cast<u32x4 *>(tile + i * 1024 + lane * 16) = *reinterpret_cast<const u32x4 *>(gm + vo);
            }
        }
    }
};

}  // namespace osdn
