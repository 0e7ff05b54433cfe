// Host-side rules of the launches: operand ranges, launch limits, choice of kernels.  Plain C++ without HIP, so that the
// rules can be compiled and checked without a GPU.
#pragma once
#include <stddef.h>

// Elements from the first to the last one of a matrix stored as `outer` rows of `inner` elements, ld apart: the range of
// the buffer descriptor that its loads go through.  An empty matrix has none; without that case K = 0 with padded rows
// gives a negative number, which as an unsigned range covers the offset that stands for "out of range".
constexpr long ms_matrix_extent(long outer, long inner, long ld) {
    return outer > 0 && inner > 0 ? (outer - 1) * ld + inner : 0;
}
// Whether a kernel may load the matrix through a descriptor with 32-bit byte offsets (rows that go backwards may not)
constexpr long kBufferBytes = (1L << 32) - (1L << 20);
constexpr bool ms_buffer_range_ok(long outer, long inner, long ld, int es) {
    return (outer <= 1 || ld >= 0) && ms_matrix_extent(outer, inner, ld) * es < kBufferBytes;
}

// HIP refuses a launch of 2^32 threads or more along one dimension
constexpr long kLaunchThreads = 0xffffffffL;
constexpr bool ms_launch_fits(long workgroups, int threads) { return workgroups <= kLaunchThreads / threads; }
// The same number of workgroups (or a few more) in one row where that may be launched, else in rows of 2^20
struct MsGrid { unsigned x, y; };
constexpr MsGrid ms_fold_grid(long workgroups, int threads) {
    return ms_launch_fits(workgroups, threads) ? MsGrid{(unsigned)workgroups, 1u} : MsGrid{1u << 20, (unsigned)((workgroups + (1L << 20) - 1) >> 20)};
}

// fp32 attention on 16-row tiles: whether the batch can be addressed and launched (max_seqlen is an upper bound; heads =
// workgroups along y).  The scalar kernels, one workgroup per token, take the rest: a batch of very many short sequences
// under a large bound among them.
constexpr int kF32AttnTile = 16;
constexpr bool ms_f32_attention_tiles(int hd, long n, long n_seqs, long max_seqlen, int nq, int nkv, int heads) {
    return (hd == 64 || hd == 80 || hd == 128) && n * (nq + 2 * nkv) * hd * 4 < kBufferBytes && max_seqlen > 0 && heads <= 65535 &&
           ms_launch_fits(n_seqs * ((max_seqlen + kF32AttnTile - 1) / kF32AttnTile), 256);
}
