// Host twiddle tables of the double-precision negacyclic transform (fft.h).
#include <math.h>

#include "internal.h"

namespace vlp {

namespace {

// s of stage k, block b: exp(2 pi I (2^-(k+3) + brv_k(b) / 2^(k+1))), to long double.
void stage_twiddle(int k, int b, long double* c, long double* s) {
  int rev = 0;
  for (int t = 0; t < k; ++t) rev |= ((b >> t) & 1) << (k - 1 - t);
  const long double turns = ldexpl(1.0L, -(k + 3)) + ldexpl((long double)rev, -(k + 1));
  const long double ang = 2.0L * acosl(-1.0L) * turns;
  *c = cosl(ang);
  *s = sinl(ang);
}

}  // namespace

void make_fft_tables(FftTables* t) {
  // Every stage's twiddles once (511 sines and cosines); the lanes' are copies.
  for (int e = 0; e < 4; ++e) t->dd[0][e] = 0;
  for (int k = 0; k < 9; ++k)
    for (int b = 0; b < (1 << k); ++b) {
      long double c, s;
      stage_twiddle(k, b, &c, &s);
      double* d = t->dd[(1 << k) + b];
      d[0] = (double)c;
      d[1] = (double)(c - (long double)d[0]);
      d[2] = (double)s;
      d[3] = (double)(s - (long double)d[2]);
    }
  auto put = [t](double (&to)[2], int k, int b) {
    to[0] = t->dd[(1 << k) + b][0];
    to[1] = t->dd[(1 << k) + b][2];
  };
  for (int L = 0; L < 64; ++L) {
    const int rho = L & 15, i4 = L >> 5, i3 = (L >> 4) & 1;
    const int i8 = L >> 5;  // of layout 4
    const int k_of[11] = {4, 5, 6, 6, 7, 8, 8, 3, 3, 2, 1};
    const int tail = (rho << 3) | (i4 << 2) | (i3 << 1);  // block of stage 7 with i2 = 0
    const int b_of[11] = {rho,          rho << 1, rho << 2,       (rho << 2) | 2, tail, tail << 1, (tail << 1) | 2,
                          i8 << 2, (i8 << 2) | 2, i8 << 1, i8};
    for (int e = 0; e < 11; ++e) put(t->lane[e][L], k_of[e], b_of[e]);
  }
  // Half-size inverse (i8 = hf): stages 8, 7 in lane (i3 i2 | i4 | i7 i6 i5),
  // 6, 5 in lane (i1 i0 | i4 | i7 i6 i5), 4, 3 in lane (i7 i6 | i3..i0), 2, 1 uniform.
  for (int hf = 0; hf < 2; ++hf)
    for (int L = 0; L < 64; ++L) {
      const int i3 = L >> 5, i2 = (L >> 4) & 1, i4 = (L >> 3) & 1, top = (hf << 3) | (L & 7);  // i8 i7 i6 i5
      const int b7 = (((top << 1) | i4) << 2) | (i3 << 1) | i2;                                // i8..i2
      const int mid = (hf << 2) | (L >> 4);                                                    // i8 i7 i6
      const int k_of[8] = {8, 7, 6, 5, 4, 3, 2, 1};
      const int b_of[8] = {b7 << 1, b7, ((top << 1) | i4) << 1, (top << 1) | i4, mid << 1, mid, hf << 1, hf};
      for (int e = 0; e < 8; ++e) put(t->half[hf][e][L], k_of[e], b_of[e]);
    }
}

const FftTables& fft_tables() {
  static const FftTables tables = [] {
    FftTables t;
    make_fft_tables(&t);
    return t;
  }();
  return tables;
}

}  // namespace vlp
