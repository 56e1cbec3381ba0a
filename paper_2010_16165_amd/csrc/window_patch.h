// Internal: the run of input pixels that a tile of output pixels needs (conv_window.hip).  The
// planner reserves LDS by it and the kernel fills LDS by it, from the same functions.  And which
// tile a workgroup takes.
#pragma once
#include <cstdint>

namespace fupr {

// The pixels of a batch, rows and images one behind the other, are numbered as one row.  Tap (r, s)
// of the output pixel at (n, pp, qq) reads number window_origin + r * W + s (where it is inside the image).
constexpr int window_origin(int n, int pp, int qq, int H, int W, int stride, int pad) {
  return (n * H + pp * stride - pad) * W + qq * stride - pad;
}

// From a window's origin to its last tap.
constexpr int window_reach(int R, int S, int W) { return (R - 1) * W + S - 1; }

// A tile's run goes from the origin of its first output pixel to the last tap of its last one.  That
// holds every tap inside an image only while windows follow each other in it: with a padding beyond
// half a window the first window of a row (or image) can begin before the last one of the row
// (image) above, and with one beyond the window a run can begin behind the pixels it is for.
constexpr bool window_runs_are_whole(int R, int S, int pad) { return 2 * pad <= (R < S ? R : S); }

// The most pixels a run of BM output pixels takes, the pixel of zeros before it included.  Needs
// window_runs_are_whole: no term is negative then, since stride * (Q - 1) <= W + 2 pad - S <= W and
// likewise for the rows.
constexpr int64_t most_run_pixels(int BM, int R, int S, int stride, int H, int W, int P, int Q) {
  const int64_t rows = (BM - 1 + Q - 1) / Q;                              // row ends crossed, at most
  const int64_t images = (BM - 1 + (int64_t)P * Q - 1) / ((int64_t)P * Q);   // image ends crossed, at most
  const int64_t row_end = (int64_t)stride * W - (int64_t)stride * (Q - 1);
  const int64_t image_end = (H - (int64_t)stride * (P - 1)) * W;
  return 1 + (int64_t)(BM - 1) * stride + rows * row_end + images * image_end + window_reach(R, S, W) + 1;
}

// Workgroups are given to the eight XCDs in turn, and an XCD takes per_xcd tiles that follow each other: the tile
// of a workgroup, or -1 where it has none.  A grid may be larger than total tiles need (the other convolution's of a
// launch of two): a workgroup beyond its XCD's share must not go on into the next XCD's.
constexpr int kXcds = 8;
constexpr int tiles_per_xcd(int total) { return (total + kXcds - 1) / kXcds; }
constexpr int tile_of_workgroup(uint32_t block, int per_xcd, int total) {
  const int in_xcd = (int)(block / kXcds), tile = (int)(block % kXcds) * per_xcd + in_xcd;
  return in_xcd < per_xcd && tile < total ? tile : -1;
}

}  // namespace fupr
