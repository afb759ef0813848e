// Host check of the rolling blocks' fit rule: for every shape that roll_fits accepts,
// every block after a lane's first is taken up before the step of its first cell in the
// band, and off column 0.  (The step that takes a block up starts it with minus
// infinity, so the cell left of and above that first one, which may lie in the band,
// has to come after.)  Prints the number of shapes that fit, or the first fault.
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <random>

#include "internal.h"

static bool sound(int M, int N, int w, int R, int LG) {
  auto centre = [&](int64_t i) { return i * N / M; };
  const int nblocks = (M + R - 1) / R;
  for (int b = LG; b < nblocks; ++b) {
    const int before = b - LG; // of the same lane
    const int last = (int)std::min<int64_t>(N, centre((int64_t)before * R + R) + w) + before;
    const int take = (alnk::roll_leave(last, R) + 7) / 8 * 8; // looked at every 8 steps
    const int64_t lo = centre((int64_t)b * R + 1) - w;
    if (lo < 1 || take >= lo + b) {
      std::printf("FAIL M %d N %d w %d rows %d lanes %d block %d: taken up at step %d, first cell at %d\n",
                  M, N, w, R, LG, b, take, (int)lo + b);
      return false;
    }
  }
  return true;
}

int main(int argc, char **argv) {
  std::mt19937 rng(argc > 1 ? std::atoi(argv[1]) : 1);
  static const int shapes[4][2] = {{2, 16}, {4, 16}, {2, 64}, {4, 64}};
  long fit = 0;
  auto check = [&](int M, int N, int w) {
    for (const auto &s : shapes)
      if (alnk::roll_fits(M, N, w, s[0], s[1])) {
        ++fit;
        if (!sound(M, N, w, s[0], s[1])) return false;
      }
    return true;
  };
  // about square at every width, where the rule's line lies
  for (int w = 0; w <= 200; ++w)
    for (int M = 300; M <= 1500; M += 97)
      for (int N = M - 60; N <= M + 20; ++N)
        if (!check(M, N, w)) return 1;
  for (int k = 0; k < 200000; ++k) {
    const int M = 1 + (int)(rng() % 2500), w = (int)(rng() % 300);
    const int N = std::max(1, (int)(M * (0.2 + 3e-3 * (rng() % 1000))));
    if (!check(M, N, w)) return 1;
  }
  std::printf("%ld\n", fit);
  return 0;
}
