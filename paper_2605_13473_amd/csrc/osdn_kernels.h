// Argument blocks and launchers of the OSDN kernels (internal to the library).
#pragma once
#include "osdn_device.h"

namespace osdn {

// Every kernel works on the chunks [n0, n1) of the sequence (all of them in one launch, or a
// segment when the two phases are pipelined against each other); what a sequential kernel
// carries across a segment boundary (d, S, dS, the adjoint of d) goes through the same
// buffers that hold it at the ends of the sequence.
//
// Packed sequences (seq_chunks != null): the token axis holds n_seqs sequences one after the
// other, each starting on a chunk boundary; sequence s owns the chunks
// [seq_chunks[s], seq_chunks[s+1]).  The token tensors and per-chunk buffers then have one
// batch entry, the carried tensors (d, S and their adjoints) one entry per sequence, and the
// sequential kernels run one chain per (sequence, head).  A chain takes its start value from
// the *_first / *_last pointer when its sequence begins (ends, in the backward pass) inside
// [n0, n1), and from the carry buffer otherwise.
// The caller's rows of the token tensors.  Sequences need not be whole chunks: the kernels read and write the caller's
// tensors where they are, clamp the row of a token that does not exist to the last one that does, and give
// such tokens the values that change nothing (k = dO = 0, beta = 0, log alpha = 0, retention = 1).  The workspace is
// laid out for whole chunks.  The many kernels of phase 1's backward pass take k, beta and retention of a sequence's
// ragged last chunk from a whole tile that the forward sweep leaves (`tail`): clamped rows cost the chain 8 %.
// 65536 packed tokens, 16 heads of 128 x 128 in bf16, forward and backward: 3737 us with padded copies of
// the inputs, 3371 without; one prompt of 1531 tokens 121 and 108.
struct Rows {
    int T;                                // tokens per batch entry of the caller's tensors
    // packed ragged sequences, else null: per chunk, its first row; its tokens - 1, and (from bit 6) its sequence
    const int *chunk_row, *chunk_seq;
    bool ragged() const { return chunk_row || T % C != 0; }
    // first row of chunk n of batch entry b, and how many of its tokens exist (at least 1); RAG: some chunk is not whole
    // (a template parameter of every kernel: the code for the others costs calls of whole chunks up to 4 %)
    template <bool RAG> __device__ __forceinline__ size_t first(int b, int n) const { return RAG && chunk_row ? (size_t)chunk_row[n] : (size_t)b * T + (size_t)n * C; }
    template <bool RAG> __device__ __forceinline__ int count(int n) const { return !RAG ? C : chunk_row ? (chunk_seq[n] & 63) + 1 : (T - n * C < C ? T - n * C : C); }
    // the tile that holds the chunk if it is not whole, else -1
    template <bool RAG> __device__ __forceinline__ int tail(int b, int n) const {
        if (!RAG) return -1;
        const int s = chunk_row ? chunk_seq[n] : 0;
        return chunk_row ? ((s & 63) == 63 ? -1 : s >> 6) : T - n * C < C ? b : -1;
    }
};
// launches with the kernel instance for whole or ragged chunks: f(std::true_type or std::false_type).  Both are to give the
// same bits (a call padded by its caller against a ragged one): sums of two products are written as the fma they are
template <typename F> inline void with_rows(const Rows &r, F &&f) {
    if (r.ragged()) f(std::true_type{});
    else f(std::false_type{});
}
// The same for a kernel that walks the chunks of one chain (b: batch entry, or packed sequence; n0: a chunk of it).
template <bool RAG> struct ChainRows {
    int base, end;                        // row of (the sequence's) chunk 0; one past its last row
    __device__ __forceinline__ ChainRows(const Rows &r, const int *seq_chunks, int b, int n0) {
        if (RAG && r.chunk_row) {
            const int last = seq_chunks[b + 1] - 1;
            base = r.chunk_row[n0] - n0 * C;
            end = r.chunk_row[last] + (r.chunk_seq[last] & 63) + 1;
        } else {
            base = 0;
            end = r.T;
            batch = seq_chunks ? 0 : (size_t)b * r.T;
        }
    }
    // (in 64 bits throughout: from a 32-bit sum the compiler forms a loader's addresses anew for every chunk, eight products; one
    // chain of 1024 chunks, state_fwd: 618 us, so 599)
    __device__ __forceinline__ size_t first(int n) const { return batch + (size_t)(long long)base + (size_t)n * C; }
    __device__ __forceinline__ int count(int n) const { const int c = end - (base + n * C); return RAG && c < C ? c : C; }
    size_t batch = 0;
};

struct PrecondArgs {
    int B, T, H, K;
    int n0, n1;
    int n_seqs;               // 0: plain batch
    const int *seq_chunks;    // [n_seqs + 1] or null; behind them the sequences, longest first [n_seqs]
    const float *d_first;     // packed sequences: d before the first token, [n_seqs,H,K] or null
    float eta, d_min, d_max, eps;
    int beta_aware;
    Rows rows;                // of k, beta, retention
    const void *k;            // [B,T,H,K] io
    const float *beta;        // [B,T,H]
    const float *retention;   // [B,T,H] ([B,T,H,K] with ret_vec) or null
    int ret_vec;              // one retention per coordinate
    const float *d_in;        // [B,H,K] or null
    void *k_tilde;            // [B,T,H,K] io, or ...
    int kt_tiles;             // ... [B,T/64,H,64,K]: one contiguous tile per chunk and head
    float *d_out;             // [B,H,K]
    float *d_ckpt;            // [B,H,T/64,K] or null
    float *tok_scalars;       // [B,T,H,4] or null: per token (step, <d,k^2>, sum k^2, unused), kept for the backward; without
                              // retention the sum's sign is a mark: the last token's is flipped in a chunk that stays well off the box (mark_bound)
    void *k_tail;             // [sequences,64,H,K] io: k of ragged last chunks, whole, kept for the backward
    float *beta_tail, *ret_tail;      // [sequences,64,H], as retention
    // Sweeps over the whole sequence (pieces > 0, plain batches only): a chain is cut into
    // pieces of piece_chunks chunks, one workgroup per piece.  Sweep number `sweep` reads the
    // start values and piece maps x -> clip3(A x + B, L, H) that sweep - 1 left (two buffers
    // each, used in turn) and returns at once for a chain whose start values no longer move.
    int pieces, piece_chunks, sweep;
    float *piece_start;       // [2][B*H*pieces, K]
    float4 *piece_map;        // [2][B*H*pieces, K]  (A, B, L, H)
    int *settled;             // [B*H] or null: a chain whose entry is set is left alone
};

struct PrecondBwdArgs {
    int B, T, H, K;
    int n0, n1;
    int n_seqs;
    const int *seq_chunks;
    const float *dd_last;     // packed sequences: adjoint of the final d, [n_seqs,H,K] or null
    float eta, d_min, d_max, eps;
    int beta_aware;
    Rows rows;                // of k, beta, retention and their gradients
    const void *k;
    const float *beta, *retention;
    const void *k_tail;       // ragged last chunks, from the forward sweep
    const float *beta_tail, *ret_tail;
    const float *d_ckpt;     // retention [B,T,H], or [B,T,H,K] with ret_vec
    int ret_vec;
    float *tok_scalars;       // [B,T,H,4] from the forward sweep: (step, <d,k^2>, +-sum k^2, -); the chain
                              // kernel puts sigma_t into the fourth slot for the post kernel
    uint2 *masks;             // [B,H,T/64,K]: bit i = token i of the chunk stayed inside the box
    float *a_ckpt;            // [B,H,T/64,K]: adjoint of d at the right end of every chunk
    const void *dkt;          // [B,N,H,64,K] io: dL/dk~ from phase 2
    const void *dk_read;      // [B,N,H,64,K] io: read-side dL/dk from phase 2
    const float *dd_out;      // [B,H,K] or null
    void *dk;                 // [B,T,H,K] io
    float *dbeta;             // [B,T,H] in/out
    float *dretention;        // [B,T,H] ([B,T,H,K] with ret_vec) or null
    float *dd_in;             // [B,H,K]
    // chunks in solved form (no retention; null: never): per chunk, whether it qualifies (no
    // coordinate met the box), the inverse (I + U)^-1, rho0 and the chunk's sum of lambda
    int *lin_clean;           // [B,H,T/64]
    void *lin_M;              // [B,H,T/64,64,64] io
    float *lin_r0;            // [B,H,T/64,64]
    float *lin_t0;            // [B,H,T/64,K]
    // Sweeps over the whole sequence (pieces > 0, plain batches only), as in the forward pass: one workgroup per piece of
    // piece_chunks chunks; sweep number `sweep` reads the records (x, y, P, g) that sweep - 1 left (two buffers in turn)
    int pieces, piece_chunks, sweep;
    float4 *piece_map;        // [2][B*H*pieces, K]
    int *settled;             // [B*H] or null: a chain whose entry is set is left alone
    unsigned char *lin_aux;   // [B,H,T/64,2048]: with a retention gate, the indicators and retention products of the chunk
};

// The recurrent step (decode): state in registers, 1..64 tokens per launch.
struct StepArgs {
    int B, T, H, K, V;
    float scale, eta, d_min, d_max, eps;
    int beta_aware;
    const void *q, *k, *v;            // [B,T,H,*] io
    const float *beta, *log_alpha, *retention;   // [B,T,H]; log_alpha, retention may be null;
    int ret_vec;                      // retention is [B,T,H,K]: one value per coordinate
    int gate_vec;                     // log_alpha is [B,T,H,K]: one state gate per key channel
    const float *d_in, *S_in;         // [B,H,K], [B,H,V,K]; may be null (ones / zeros)
    void *o;                          // [B,T,H,V] io
    float *S_out, *d_out;             // S_out may be S_in (a workgroup reads its rows before it writes them)
};

// Everything the chunkwise (phase 2) kernels need.  Per-chunk tiles live in the workspace in
// [B,N,H,rows,cols] order, one contiguous tile per chunk and head: what the workgroups of a launch
// (numbered head first) or the chains of a chain kernel (in step) touch at one time is then
// contiguous in memory and spreads over all its channels.
struct ChunkArgs {
    SliceMap map;             // chain kernels: the slices of the launch (the launchers say; first, with the sizes: one line of arguments)
    int B, T, H, K, V, N;
    int n0, n1;
    int n_seqs;
    const int *seq_chunks;
    const float *S_first;             // packed sequences: [n_seqs,H,V,K] or null
    const float *dS_last;             // packed sequences: adjoint of the final S, or null
    float scale;
    Rows rows;                        // of q, k, v, beta, log_alpha, o, dO and the gradients
    // caller tensors
    const void *q, *k, *v;            // [B,T,H,*] io
    const float *beta, *log_alpha;    // [B,T,H]; log_alpha may be null
    const float *S_in;                // [B,H,V,K] or null
    void *o;                          // [B,T,H,V] io
    float *S_out;                     // [B,H,V,K]
    // workspace (forward)
    void *kt;                         // [B,N,H,64,K] io   k~
    void *Tm;                         // [B,N,H,64,64] io  (I + A)^-1
    void *Wn;                         // [B,N,H,64,K] io   -W
    void *Tu;                         // [B,N,H,64,64] io  (I + A)^-1 diag(beta)
    float *gates;                     // [B,N,H,3,64] f32  cumulative log-decay G inside the chunk, gamma = e^G, rho = e^(G_C - G)
    void *Et;                         // [B,N,H,V,64] io   E transposed
    void *S_ckpt;                     // [B,N,H,V,K] io    state at the start of each chunk (null: not kept)
    void *Pm;                         // [B,N,H,64,64] io  P = tril(Gamma . Q K~^T), from output_fwd for the backward
                                      //                   chain (null: not kept; Tm may be null likewise)
    int narrow_slices;                // chain kernels: 16 rows of the state per workgroup instead of 32 (bwd_chain with fp32 at K = 128: always 16)
    int asks_ahead;                   // state_fwd with bf16 I/O and slices of 16: the lines of its operands ahead of the tiles
    // one state gate per key channel (gate_vec: log_alpha is [B,T,H,K]; forward only): chunk_prep
    // folds the cumulative channel decays Gamma into the operands and leaves
    int gate_vec;
    void *Qg;                         // [B,N,H,64,K] io   Gamma . Q   (taking the place of q, k, kt in the kernels that follow)
    void *Kg;                         // [B,N,H,64,K] io   Gamma . K
    void *Kd;                         // [B,N,H,64,K] io   K~ / Gamma
    void *Kw;                         // [B,N,H,64,K] io   K~ . gamC / Gamma, what the chain kernels multiply: it stays below
                                      //                   K~, where K~ / Gamma times a state or its adjoint leaves the range
                                      //                   of the type (e^79 at the strongest decay a chunk may have)
    float *gamC;                      // [B,N,H,K] f32     decay of every channel over the whole chunk
    float *dgamC;                     // [B,N,H,K] f32     backward: gamC . dL/dgamC
    // backward
    const void *dO;                   // [B,T,H,V] io
    const float *dS_out;              // [B,H,V,K] or null
    void *dEt;                        // [B,N,H,V,64] io   dE transposed (complete)
    void *dS_ckpt;                    // [B,N,H,V,K] io    adjoint of the state at the END of each chunk
    float *dS_in;                     // [B,H,V,K]
    void *dq, *dv;                    // io
    void *dk_read, *dkt;              // [B,N,H,64,K] io: the two parts of dL/dk that phase 1 combines
    float *dbeta, *dlog_alpha;        // [B,T,H]; dlog_alpha may be null
};

int launch_precond_fwd(const PrecondArgs &a, bool bf16_io, hipStream_t st);
int launch_step(const StepArgs &a, bool bf16_io, hipStream_t st);
int launch_seq_tables(const int *cu, const int *seq_chunks, const int *order, int n_seqs, int N, int *tables, hipStream_t st);
int launch_precond_mask(const PrecondBwdArgs &a, bool bf16_io, hipStream_t st);
// solved form with a retention gate per (token, head): which = 0 masks, inverse and indicators (forward
// data only), 1 rho0 and t0 (needs dL/dk~), 2 the chain; chunks [n0, n1)
int launch_precond_gen(const PrecondBwdArgs &a, bool bf16_io, int which, hipStream_t st);
int launch_precond_lin_bwd(const PrecondBwdArgs &a, bool bf16_io, bool m_part, hipStream_t st);
int launch_precond_chain(const PrecondBwdArgs &a, bool bf16_io, hipStream_t st);
int launch_precond_post(const PrecondBwdArgs &a, bool bf16_io, hipStream_t st);
int launch_chunk_prep(const ChunkArgs &a, bool bf16_io, hipStream_t st);
int launch_state_fwd(const ChunkArgs &a, bool bf16_io, hipStream_t st);
int launch_output_fwd(const ChunkArgs &a, bool bf16_io, hipStream_t st);
int launch_bwd_chain(const ChunkArgs &a, bool bf16_io, hipStream_t st);
int launch_bwd_post(const ChunkArgs &a, bool bf16_io, hipStream_t st);

// Backward with one state gate per key channel: phase 2 runs on the folded operands
// (Gamma . Q, Gamma . K, K~ / Gamma) and leaves the gradients with respect to those; this
// kernel turns them, in place, into the gradients with respect to q, k (read side) and k~,
// and collects dL/dlog_alpha.
struct UnfoldArgs {
    int B, T, H, K, N;
    int n0, n1;
    Rows rows;                        // of log_alpha, q, k, dq and dlog_alpha
    const float *log_alpha;           // [B,T,H,K]
    const void *q, *k, *kt;           // io: the unfolded operands (q, k: [B,T,H,K]; kt: [B,N,H,64,K])
    void *dq, *dk_read, *dkt;         // io, dq [B,T,H,K], the others [B,N,H,64,K]: in: w.r.t. the folded operands; out: w.r.t. q, k, k~
    const float *dgamC;               // [B,N,H,K]
    float *dlog_alpha;                // [B,T,H,K]
};
int launch_unfold(const UnfoldArgs &a, bool bf16_io, hipStream_t st);

}  // namespace osdn
