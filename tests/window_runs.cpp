// Walks every tile of many geometries as conv_window.hip does: the pixels the kernel fills must not
// exceed those the planner reserves, and every tap inside an image must lie in the filled run.
// Prints the number of tiles walked; exit status 1 with the first geometry that fails.
#include <algorithm>
#include <cstdio>

#include "window_patch.h"

using namespace fupr;

int main() {
  const int tiles[] = {16, 32, 64, 112};
  long walked = 0;
  for (int R = 1; R <= 5; ++R)
    for (int S = 1; S <= 5; ++S)
      for (int pad = 0; pad <= std::max(R, S); ++pad) {
        if (!window_runs_are_whole(R, S, pad)) continue;
        for (int stride = 1; stride <= 6; ++stride)
          for (int H : {1, 2, 3, 5, 7, 14})
            for (int W : {1, 2, 3, 4, 7, 13, 17, 33, 120}) {
              if (H + 2 * pad < R || W + 2 * pad < S) continue;
              const int P = (H + 2 * pad - R) / stride + 1, Q = (W + 2 * pad - S) / stride + 1;
              const int N = P * Q < 64 ? 70 / (P * Q) + 2 : 2, M = N * P * Q;
              for (int BM : tiles)
                for (int m0 = 0; m0 < M; m0 += BM) {
                  const int end = std::min(m0 + BM, M);
                  auto origin = [&](int m) {
                    return window_origin(m / (P * Q), m % (P * Q) / Q, m % Q, H, W, stride, pad);
                  };
                  const int first = origin(m0), last = origin(end - 1) + window_reach(R, S, W);
                  bool ok = 1 + last - first + 1 <= most_run_pixels(BM, R, S, stride, H, W, P, Q);
                  for (int m = m0; m < end && ok; ++m) {
                    const int ih = m % (P * Q) / Q * stride - pad, iw = m % Q * stride - pad;
                    for (int r = 0; r < R; ++r)
                      for (int s = 0; s < S; ++s)
                        if (ih + r >= 0 && ih + r < H && iw + s >= 0 && iw + s < W) {
                          const int at = origin(m) + r * W + s;
                          ok = ok && at >= first && at <= last;
                        }
                  }
                  if (!ok) {
                    std::printf("%d x %d pad %d stride %d on %d x %d x %d, tile %d at %d\n", R, S, pad, stride, N, H,
                                W, BM, m0);
                    return 1;
                  }
                  ++walked;
                }
            }
      }
  std::printf("%ld\n", walked);
  return 0;
}
