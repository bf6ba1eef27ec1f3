// Host build of the FP32 count estimates (fastdraw.hpp) on cells of windows, their weights
// formed as the tile kernel forms them (the erf polynomial, rounded to FP32), for comparison
// with the counts that det_erf's weights define.  A cell's axes are given by the arguments of
// the erf at its edges, a0 < a1 and b0 < b1 (C99 hex floats).
// Usage: fastdraw_window_check binom   stdin lines "N a0 a1 b0 b1 u" -> "sure count" per line
//        fastdraw_window_check normal  stdin lines "N a0 a1 b0 b1 w0 w1 w2" -> "sure count" per
//                                      line (the tick pair's even cell)
#include <cstdio>
#include <cstdlib>
#include <cstring>

#include "erfpoly.hpp"
#include "fastdraw.hpp"

using namespace wct;

static float weight(const char* lo, const char* hi) {
  return (float)(0.5 * (erf_poly(std::strtod(hi, nullptr)) - erf_poly(std::strtod(lo, nullptr))));
}

int main(int argc, char** argv) {
  if (argc < 2) return 2;
  char t[5][64];
  const bool normal = std::strcmp(argv[1], "normal") == 0;
  if (!normal && std::strcmp(argv[1], "binom") != 0) return 2;
  double q;
  while (std::scanf("%lf %63s %63s %63s %63s", &q, t[0], t[1], t[2], t[3]) == 5) {
    const float N = (float)q, mu = weight(t[0], t[1]) * N * weight(t[2], t[3]), p = mu * (1.0f / N);
    int k = 0;
    bool sure = true;
    if (normal) {
      unsigned w0, w1, w2;
      if (std::scanf("%u %u %u", &w0, &w1, &w2) != 3) return 2;
      float ze, zo;
      const bool ok = fast_normal_pair(w0, w1, w2, &ze, &zo);
      sure = fast_normal_count(N, mu, p, ze, &k) && ok;
    } else {
      if (std::scanf("%63s", t[4]) != 1) return 2;
      const uint32_t w = (uint32_t)(std::strtod(t[4], nullptr) * 0x1p32);  // the upper word of u
      const uint32_t x = entry_x(p, 37), y = entry_y(w, 4321);             // as it waits for its batch
      if (!(fmaf((float)w, 0x1p-32f, mu) < fast_zero_limit(N)))
        sure = mu >= (float)kMuSwitch ? fast_chopdown(N, entry_p(x), entry_u(y), &k)
                                      : fast_inversion(N, entry_p(x), entry_u(y), &k);
    }
    std::printf("%d %d\n", (int)sure, k);
  }
  return 0;
}
