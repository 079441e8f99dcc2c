// Scratch of the forward transform (host code of dwt.hip): every approximation that a
// launch leaves for another launch of many blocks fits the part it goes to, the two
// parts alternate, a part is never larger than n^2 / 4 (the fixed scratch of the entry
// that does not allocate), and 32 images of a launch together take no more than 8
// images at n^2 / 2 each.  Built and run by tests/test_native_dwt.py.
#include "../../paper_1512_08401_amd/csrc/dwt.hip"
#include "../../paper_1512_08401_amd/csrc/filters.cpp"

#include <stdexcept>

namespace wdb {
[[noreturn]] void fail(wdb_status, const char* fmt, ...) { throw std::runtime_error(fmt); }
void set_last_error(const std::string&) {}
void clear_last_error() {}
}  // namespace wdb

int main() {
  using namespace wdb;
  int plans = 0;
  for (int n = 2; n <= 1 << 14; n *= 2)
    for (int levels = 1; (n >> levels) >= 1; ++levels) {
      const DwtScratch need = dwt_scratch(n, levels);
      const size_t N = static_cast<size_t>(n) * n;
      // the launches of dwt_forward_many
      int M = n, left = levels, turn = 0;
      while (left > 0 && M > kTailSide) {
        const int nl = launch_levels(M, left);
        const bool on = left > nl && (M >> nl) > kTailSide;
        M >>= nl;
        left -= nl;
        if (on && static_cast<size_t>(M) * M > (turn ? need.b : need.a)) return 1;
        turn ^= 1;
      }
      if (need.a > N / 4 || need.b > N / 4) return 2;
      if (n < 2048 && need.a + need.b) return 3;
      if (kBatch * (need.a + need.b) > 8 * 2 * (N / 4)) return 4;
      plans += need.a > 0;
    }
  if (!plans) return 5;
  std::puts("all checks passed");
  return 0;
}
