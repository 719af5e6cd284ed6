// Host check of the index arithmetic that places a lane's samples at the end
// of a view (last_read_col / read_shift of common.h), over rows up to the
// widest accepted: for every lane near a limit, the vector that it reads lies
// inside the view, and after the shift each sample of the row is its own and
// each place past the view's end holds zero.
#include <cstdint>
#include <cstdio>

#include "common.h"

using namespace dwtfrag;

static long checked = 0, failures = 0;

static void lane(int64_t n_valid, int64_t at, int w, int span, int64_t c) {
  if (c < 0 || c > 0x7FFFFFFF - span) return;
  const int c0 = int(c / span) * span;
  const int last = last_read_col(n_valid, at, span);
  const int64_t from = at + (c0 < last ? c0 : last);
  const int sh = last < w ? read_shift(c0, last, span) : 0;
  ++checked;
  if (c0 >= w) return;  // (such lanes hold nothing of the row; what they read is inside all the same)
  bool ok = from >= 0 && from + span <= n_valid;
  for (int t = 0; t < span; ++t) {
    if (c0 + t >= w) break;
    const bool inside = at + c0 + t < n_valid;
    const int64_t got = t + sh < span ? from + t + sh : -1;  // -1: a zero shifted in
    ok &= got == (inside ? at + c0 + t : -1);
  }
  if (!ok && ++failures < 20)
    std::printf("n_valid %lld row at %lld width %d span %d: lane at column %d reads from %lld, shift %d\n",
                (long long)n_valid, (long long)at, w, span, c0, (long long)(from - at), sh);
}

int main() {
  const int64_t widths[] = {1, 7, 8, 9, 300, 4096, (1 << 28) - 9, (1 << 28) - 1, 1 << 28, (1 << 28) + 9,
                            (1 << 28) + 1003, 300000001, (1 << 29) + 16, (int64_t(1) << 30) + 1, 0x7FFF0000 - 1,
                            0x7FFF0000};
  for (int64_t w : widths)
    for (int span : {8, 16})
      for (int64_t rows : {1, 2, 3, 40})
        for (int64_t rest : {int64_t(1), int64_t(3), w / 2, w - span, w - 1, w}) {
          if (rest < 1 || rest > w) continue;
          const int64_t n_valid = (rows - 1) * w + rest;
          if (n_valid < span) continue;
          for (int64_t r = 0; r < rows; ++r) {
            const int64_t near[] = {0, 64, w / 2, rest, w, int64_t(1) << 28, int64_t(1) << 30};
            for (int64_t x : near)
              for (int64_t d = -3 * span; d <= 3 * span; d += span) lane(n_valid, r * w, int(w), span, x + d);
          }
        }
  std::printf("%ld lanes, %ld failures\n", checked, failures);
  return failures != 0;
}
