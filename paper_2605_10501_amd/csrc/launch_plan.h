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
