// Prints, for seeded random symmetric tridiagonal matrices (a, b), couplings bm
// and kept counts l, the basis change and the reduced matrix of the library's
// restart_basis (tridiag.hpp).  Checked with numpy by tests/test_native_restart.py.
#include "../../paper_1512_08401_amd/csrc/tridiag.hpp"

#include <cstdio>
#include <random>

int main() {
  std::mt19937_64 rng(4321);
  std::uniform_real_distribution<double> U(-1.0, 1.0);
  const int sizes[][2] = {{2, 1}, {3, 2}, {5, 1}, {7, 6}, {48, 20}, {48, 47}};
  for (int kind = 0; kind < 3; ++kind) {   // random; nearly decoupled; clustered, as near convergence
    for (const auto& s : sizes) {
      const int m = s[0], l = s[1];
      std::vector<double> a(m), b(m - 1);
      for (double& x : a) x = kind == 2 ? 1.0 + 1e-9 * U(rng) : U(rng);
      for (double& x : b) x = kind == 1 ? 1e-9 * U(rng) : U(rng);
      const double bm = kind == 2 ? 1e-7 : 0.3;
      wdb::Restart r = wdb::restart_basis(a, b, bm, l);
      std::printf("%d %d %.17g", m, l, bm);
      for (auto* v : {&a, &b, &r.C, &r.a, &r.b})
        for (double x : *v) std::printf(" %.17g", x);
      std::printf("\n");
    }
  }
  return 0;
}
