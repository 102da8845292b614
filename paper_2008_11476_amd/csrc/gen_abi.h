// Arguments shared by the host and the kernels generated at run time beyond
// the interpreter's own (hvx_desc.h): plain data, no pointers to host memory.
#pragma once
#include "hvx_desc.h"

namespace hvx {

// One image of a batch run by one generated kernel: its I/O table, its size,
// the first work-group of the launch that works on it and the rows of its bands.
struct GenBatchImage {
  IOTable io;
  int32_t w, h;
  int32_t block0;
  int32_t rows;  // rows of a band (streamed kernels)
};

// Rows per loop iteration of a streamed kernel; the next four rows are loaded
// while four are computed.
constexpr int kStreamUnroll = 4;

// How a streamed kernel's items divide an image of h rows, where an output row
// reads up to `ext` rows above and below.
//
// whole: the image's last `tail` rows (ext, up to a multiple of kStreamUnroll)
// are a band of their own; the rows before them, up to a multiple of
// kStreamUnroll by `shift`, are dealt out in bands of `rows`.  All bands but
// the first start `shift` rows early, so each holds whole iterations; the
// first still starts at row 0 and computes the `shift` rows it shares with the
// second again.  Only the first band reads rows above the image, only the last
// below it.
//
// Otherwise every band goes row by row, each border rule decided as it goes:
// images under eight columns, images too low for two such bands, `rows` that
// are no whole iterations or below ext + shift, and a single band before the
// tail that is not whole iterations, as it can neither start early nor run on
// into the tail's rows, which are not all loaded.  A wave takes 0.4 to 1 us
// for a row so, and 2 ext rows before its first: 7x4096 Unsharp 1502 us as one
// item, 6.9 in bands (tiles 7.4), the F32 corner response 2513 and 13.1
// (15.4), four Gaussian5x5 4003 and 24.9 (20.9); 640x19, three Gaussian5x5
// 20.2 and 12.1 (13.6).
//
// Every wave starts with this, so what depends on `whole` is decided once, not
// per band (Gaussian3x3 -> Histogram + MeanStdDev of 3840x2160, whose waves
// take several bands, 14.9 -> 14.6 us), and a band is found without their number
// n, a division that only the host and the reducing kernels make.
struct StreamBands {
  int32_t rows, n;
  int32_t end, shift, tail;  // the first row after those dealt out; shift and tail: 0 unless whole
  bool whole;
};
__host__ __device__ inline int stream_tail(int ext) {
  return (ext + kStreamUnroll - 1) / kStreamUnroll * kStreamUnroll;
}
__host__ __device__ inline StreamBands stream_bands(int w, int h, int rows, int ext) {
  const int tail = stream_tail(ext), shift = (tail - h) & (kStreamUnroll - 1);
  const bool whole = w >= 8 && h >= tail + 2 * kStreamUnroll && rows % kStreamUnroll == 0 && rows >= ext + shift &&
                     (shift == 0 || h - tail + shift > rows);
  const int t = whole ? tail : 0, s = whole ? shift : 0;
  return {rows, (int)((unsigned)(h - t + s + rows - 1) / (unsigned)rows) + (t > 0 ? 1 : 0), h - t, s, t, whole};
}
// Band `band`: output rows [y0, y1) (`last`: the image's last rows follow), of
// which those from `own` on are the next band's to count.
struct StreamBand {
  int32_t y0, y1, own;
  bool last;
};
__host__ __device__ inline StreamBand stream_band(const StreamBands& b, int band) {
  const int start = band > 0 ? band * b.rows - b.shift : 0;
  const bool last = b.tail > 0 && start >= b.end;
  const int y0 = last ? b.end : start;
  const int y1 = last ? y0 : start + b.rows < b.end ? start + b.rows : b.end, next = (band + 1) * b.rows - b.shift;
  return {y0, y1, next < y1 ? next : y1, last};
}

// Partial results of one work-group of a generated kernel that reduces
// global operators: for each of its reduce operators in program order, a
// block of 32-bit words (even-sized, so 64-bit values stay aligned):
// HISTOGRAM / EQHIST the p0 counts, MINMAX {min, max}, MMCOUNT the two
// (value, count) keys of the extremes, SUMS the 64-bit sums of v and v^2.
__host__ __device__ inline int red_block_words(int kind, int p0) {
  switch (kind) {
    case OP_HISTOGRAM:
    case OP_EQHIST: return (p0 + 1) & ~1;
    case OP_MINMAX: return 2;
    default: return 4;  // MMCOUNT, SUMS
  }
}

__host__ __device__ inline int red_slot_words(const GProg& P) {
  int w = 0;
  for (int i = 0; i < P.nops; ++i)
    if (is_reduce_op(P.ops[i].kind)) w += red_block_words(P.ops[i].kind, P.ops[i].p0);
  return w;
}

}  // namespace hvx
