// Index tables of packed sequences.  Sequences that are not whole chunks are worked on where the caller
// put them (Rows in osdn_kernels.h); two small tables, one entry per chunk, say where: chunk_row[c] = packed row
// of the chunk's first token, chunk_seq[c] = its tokens - 1 and, from bit 6 on, its sequence.
#include "osdn_kernels.h"

namespace osdn {

// The host's offsets reach the device as kernel arguments (nothing to keep alive, no copy engine), 255
// sequences a launch; a workgroup writes the entries of one sequence.  65536 packed tokens in 67 sequences: one launch of
// 4.5 us, where the tables themselves took five.
constexpr int TABLE_SEQS = 255;
struct SeqBlock { int row[TABLE_SEQS + 1], chunk[TABLE_SEQS + 1], order[TABLE_SEQS]; };
__global__ __launch_bounds__(64) void seq_tables_kernel(SeqBlock blk, int *seq_chunks, int *order, int *chunk_row, int *chunk_seq, int first_seq) {
    const int s = blockIdx.x, c0 = blk.chunk[s], c1 = blk.chunk[s + 1], row = blk.row[s], end = blk.row[s + 1];
    if (threadIdx.x == 0) order[s] = blk.order[s];
    if (threadIdx.x < 2) seq_chunks[s + threadIdx.x] = threadIdx.x ? c1 : c0;        // (the next sequence's too: the last has none)
    for (int c = c0 + (int)threadIdx.x; c < c1; c += 64) {
        const int r = row + (c - c0) * C;
        chunk_row[c] = r;
        chunk_seq[c] = (end - r < C ? end - r : C) - 1 + (first_seq + s) * 64;
    }
}

// tables: seq_chunks [n_seqs + 1], order [n_seqs], chunk_row [N], chunk_seq [N]; cu and seq_chunks (n_seqs + 1 entries) and order on the host
int launch_seq_tables(const int *cu, const int *seq_chunks, const int *order, int n_seqs, int N, int *tables, hipStream_t st) {
    for (int at = 0; at < n_seqs; at += TABLE_SEQS) {
        SeqBlock blk;
        const int n = n_seqs - at < TABLE_SEQS ? n_seqs - at : TABLE_SEQS;
        for (int i = 0; i <= TABLE_SEQS; ++i) {
            blk.row[i] = i <= n ? cu[at + i] : 0;
            blk.chunk[i] = i <= n ? seq_chunks[at + i] : 0;
            if (i < TABLE_SEQS) blk.order[i] = i < n ? order[at + i] : 0;
        }
        hipLaunchKernelGGL(seq_tables_kernel, dim3(n), dim3(64), 0, st, blk, tables + at, tables + n_seqs + 1 + at,
                           tables + 2 * n_seqs + 1, tables + 2 * n_seqs + 1 + N, at);
    }
    return 0;
}

}  // namespace osdn
