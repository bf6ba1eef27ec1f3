// Host build of the FP32 count estimates (fastdraw.hpp), for comparison with the counts
// that define them.
// Usage: fastdraw_host_check binom   stdin lines "N p u" (p, u as C99 hex floats)
//                                    -> "sure count" per line, p and u rounded as waiting
//                                    cells hold them and the cell routed as the tile kernel does; each search
//                                    continues for (3 x line number mod 700) passes after its
//                                    own end, as a lane does beside slower lanes of its wave
//        fastdraw_host_check normal  stdin lines "w0 w1 w2 w3 N p_even p_odd"
//                                    -> "sure count sure count"
#include <cstdio>
#include <cstdlib>
#include <cstring>

#include "fastdraw.hpp"

using namespace wct;

int main(int argc, char** argv) {
  if (argc < 2) return 2;
  char b0[64], b1[64];
  if (std::strcmp(argv[1], "normal") == 0) {
    unsigned w0, w1, w2, w3;
    int N;
    while (std::scanf("%u %u %u %u %d %63s %63s", &w0, &w1, &w2, &w3, &N, b0, b1) == 7) {
      const float nf = (float)N, pe = (float)std::strtod(b0, nullptr), po = (float)std::strtod(b1, nullptr);
      float ze, zo;
      int ke, ko;
      const bool ok = fast_normal_pair(w0, w1, w2, &ze, &zo);
      const bool se = fast_normal_count(nf, nf * pe, pe, ze, &ke) && ok;
      const bool so = fast_normal_count(nf, nf * po, po, zo, &ko) && ok;
      std::printf("%d %d %d %d\n", (int)se, ke, (int)so, ko);
    }
    return 0;
  }
  if (std::strcmp(argv[1], "binom") != 0) return 2;
  long long N;
  long line = 0;
  while (std::scanf("%lld %63s %63s", &N, b0, b1) == 3) {
    const float nf = (float)N, p = (float)std::strtod(b0, nullptr), u = (float)std::strtod(b1, nullptr);
    const uint32_t w = (uint32_t)(std::strtod(b1, nullptr) * 0x1p32);  // the upper word of u
    const uint32_t x = entry_x(p, 37), y = entry_y(w, 4321);  // as it waits for its batch
    if ((x & kEntryRow) != 37 || (y & kEntryDst) != 4321) return 3;
    const float mu = nf * p;
    int k = 0;
    bool sure = true;
    wct_host_extra_passes = (int)(3 * line++ % 700);
    if (!(u + mu < fast_zero_limit(nf)))
      sure = mu >= (float)kMuSwitch ? fast_chopdown(nf, entry_p(x), entry_u(y), &k) : fast_inversion(nf, entry_p(x), entry_u(y), &k);
    std::printf("%d %d\n", (int)sure, k);
  }
  return 0;
}
