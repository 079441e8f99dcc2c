// try_alloc (common.hpp) answers false for a failed device allocation and for
// nothing else.  Built and run by tests/test_native_build.py.
#include "../../paper_1512_08401_amd/csrc/common.hpp"

int main() {
  int runs = 0;
  if (!wdb::try_alloc([&] { ++runs; })) return 1;
  if (wdb::try_alloc([&] { ++runs; throw wdb::Error{WDB_ERR_OOM, "no memory"}; })) return 2;
  for (wdb_status other : {WDB_ERR_HIP, WDB_ERR_ARG, WDB_ERR_DIVERGED}) {
    try {
      (void)wdb::try_alloc([&] { ++runs; throw wdb::Error{other, "a fault that came up here"}; });
      return 3;
    } catch (const wdb::Error& e) {
      if (e.code != other) return 4;
    }
  }
  try {
    (void)wdb::try_alloc([&] { ++runs; throw 7; });
    return 5;
  } catch (int) {
  }
  if (runs != 6) return 6;
  std::puts("all checks passed");
  return 0;
}
