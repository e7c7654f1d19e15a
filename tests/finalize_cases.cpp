// The slices of the wide finalisation, for every box: each partial in one
// slice, no more slices than the work space holds, and none long where more
// could share the work.
#include <cstdio>

#include "../paper_1601_03815_amd/csrc/runtime.hpp"

int main() {
  for (long long n = 4; n <= 1024; ++n) {
    const int blocks = (int)((n * n * n + 255) / 256);
    const int per = dhit::finalize_per(blocks), g = (blocks + per - 1) / per;
    const bool covers = (long long)g * per >= blocks && (long long)(g - 1) * per < blocks;
    const bool shared = blocks <= 4096 ? g == 1 : (g >= 2 && g <= dhit::kFinalizeLevels && (per == 4096 || g == 64));
    if (!covers || !shared) {
      std::printf("n = %lld: %d partials, %d slices of %d\n", n, blocks, g, per);
      return 1;
    }
  }
  return 0;
}
