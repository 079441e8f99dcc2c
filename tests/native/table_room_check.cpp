// The memory a build's table of PSF weights takes and may take (psf.hpp): never more
// than an eighth of what is free beside the kept entries, and half of all offsets.
// Built and run by tests/test_native_build.py.
#include "../../paper_1512_08401_amd/csrc/common.hpp"
#include "../../paper_1512_08401_amd/csrc/psf.hpp"

int main() {
  const size_t GB = size_t{1} << 30;
  for (size_t free : {size_t{0}, size_t{1}, GB, 7 * GB, 64 * GB, 288 * GB})
    for (size_t kept : {size_t{0}, size_t{1}, GB, 8 * GB, 300 * GB}) {
      const size_t room = wdb::weight_table_room(free, kept);
      if (free <= kept ? room != 0 : room > (free - kept) / 8) return 1;
    }
  // every offset at most twice: 2 (R + 1) (2 R + 1) >= (2 R + 1)^2 of them
  for (int64_t n : {2, 64, 1024, 16384})
    for (int64_t R : {int64_t{0}, int64_t{1}, int64_t{18}, n / 2 - 1}) {
      const size_t all = static_cast<size_t>((2 * R + 1) * (2 * R + 1) * n * n) * sizeof(double);
      const size_t bytes = wdb::weight_table_bytes(n, R);
      if (2 * bytes < all || 2 * bytes > all + static_cast<size_t>((2 * R + 1) * n * n) * sizeof(double)) return 2;
    }
  // the largest builds that took a quarter of an empty card with all offsets still have it
  for (int64_t R : {9, 18, 30})
    if (wdb::weight_table_bytes(1024, R) > wdb::weight_table_room(280 * GB, GB)) return 3;
  std::puts("all checks passed");
  return 0;
}
