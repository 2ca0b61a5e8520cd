// The twiddle tables: made once and shared by every thread that asks, and each
// stage's entry within the bound that the key transform's error rests on.
#include <quadmath.h>
#include <stdio.h>

#include <thread>
#include <vector>

#include "internal.h"

using namespace vlp;

int main() {
  const FftTables* seen[8];
  std::vector<std::thread> ts;
  for (int i = 0; i < 8; ++i) ts.emplace_back([&seen, i] { seen[i] = &fft_tables(); });
  for (auto& t : ts) t.join();
  for (int i = 0; i < 8; ++i)
    if (seen[i] != seen[0]) return printf("tables made twice\n"), 1;
  __float128 worst = 0;
  for (int k = 0; k < 9; ++k)
    for (int b = 0; b < (1 << k); ++b) {
      int rev = 0;
      for (int x = 0; x < k; ++x) rev |= ((b >> x) & 1) << (k - 1 - x);
      const __float128 ang = 8 * atanq(1) * (ldexpq(1, -(k + 3)) + ldexpq(rev, -(k + 1)));
      const double* d = seen[0]->dd[(1 << k) + b];
      const __float128 er = (__float128)d[0] + d[1] - cosq(ang), ei = (__float128)d[2] + d[3] - sinq(ang);
      const __float128 e = sqrtq(er * er + ei * ei);
      if (e > worst) worst = e;
    }
  printf("largest twiddle error 2^%.2f\n", (double)log2q(worst));
  if (log2q(worst) > -61.06) return printf("twiddles not exact enough\n"), 1;
  printf("tables OK\n");
  return 0;
}
