// The transforms of csrc/fft.h on the CPU, one value at a time: the butterflies,
// the key's double-double transform and the rounding are the header's own or, where
// they stand inside a kernel, in the same order.  Prints the largest distance of a
// product's coefficient from its integer, alone and in units of u S, and the
// error of the key's transform; exits non-zero where a bound of the header or a
// word is wrong.
#include <quadmath.h>
#include <stdint.h>

// The header's cross-lane moves are not used here.
struct NoLanes {
  uint32_t operator[](int) const { return 0; }
};
static inline NoLanes no_lanes(uint32_t, uint32_t) { return NoLanes(); }
#define __builtin_amdgcn_permlane16_swap(a, b, c, d) no_lanes(a, b)
#define __builtin_amdgcn_permlane32_swap(a, b, c, d) no_lanes(a, b)
#define __builtin_amdgcn_fence(a, b) (void)0
#define __builtin_amdgcn_wave_barrier() (void)0

#include "internal.h"
#include "fft.h"

#include <math.h>
#include <stdio.h>
#include <stdlib.h>

#include <algorithm>
#include <vector>

using namespace vlp;
typedef std::vector<Cplx> Poly;  // 512 complex points
typedef __float128 Q;

static FftTables T;
static uint64_t rng_state = 0x9E3779B97F4A7C15ull;
static uint32_t rnd() {  // xorshift64*
  rng_state ^= rng_state >> 12;
  rng_state ^= rng_state << 25;
  rng_state ^= rng_state >> 27;
  return (uint32_t)((rng_state * 0x2545F4914F6CDD1Dull) >> 32);
}

// Twiddle of stage k, block b, and whether the butterfly is its I-times form:
// block 2b + 1 uses block 2b's, except in stage 4, whose blocks are the lanes'.
static bool twiddle(int k, int b, double* c, double* s) {
  const bool rot = k != 4 && k > 0 && (b & 1);
  if (k < 4) {
    *c = W_RE[w_index(k, b)];
    *s = W_IM[w_index(k, b)];
  } else {
    const double* d = T.dd[(1 << k) + (rot ? b - 1 : b)];
    *c = d[0];
    *s = d[2];
  }
  return rot;
}

static void stage(Poly& z, int k, bool inverse) {
  const int half = FFT_N >> (k + 1);
  for (int t = 0; t < FFT_N / 2; ++t) {
    const int b = t / half, u = b * 2 * half + t % half, v = u + half;
    double c, s;
    const bool rot = twiddle(k, b, &c, &s);
    if (inverse) rot ? bf_inv<true>(z[u], z[v], c, s) : bf_inv<false>(z[u], z[v], c, s);
    else rot ? bf_fwd<true>(z[u], z[v], c, s) : bf_fwd<false>(z[u], z[v], c, s);
  }
}

// Transformed key channel, scaled by 1/512; its errors (relative in the 2-norm, in
// units of u) before and after the rounding where `errors` is given.
static Poly key_transform(int ch, const uint32_t* a, const uint32_t* b, double* errors) {
  std::vector<DD> re(FFT_N), im(FFT_N);
  std::vector<Q> qr(FFT_N), qi(FFT_N);
  for (int i = 0; i < FFT_N; ++i) {
    re[i] = {key_value(ch, a, b, i), 0.0};
    im[i] = {key_value(ch, a, b, i + FFT_N), 0.0};
    qr[i] = re[i].h;
    qi[i] = im[i].h;
  }
  for (int k = 0; k < 9; ++k)
    for (int t = 0; t < FFT_N / 2; ++t) {
      const int half = FFT_N >> (k + 1), b_ = t / half, u = b_ * 2 * half + t % half, v = u + half;
      const double* w = T.dd[(1 << k) + b_];
      dd_bf(re[u], im[u], re[v], im[v], DD{w[0], w[1]}, DD{w[2], w[3]});
      if (!errors) continue;
      int rev = 0;
      for (int x = 0; x < k; ++x) rev |= ((b_ >> x) & 1) << (k - 1 - x);
      const Q ang = 8 * atanq(1) * (ldexpq(1, -(k + 3)) + ldexpq(rev, -(k + 1))), c = cosq(ang), s = sinq(ang);
      const Q tr = c * qr[v] - s * qi[v], ti = c * qi[v] + s * qr[v];
      qr[v] = qr[u] - tr;
      qi[v] = qi[u] - ti;
      qr[u] += tr;
      qi[u] += ti;
    }
  Poly z(FFT_N);
  Q norm = 0, before = 0, after = 0;
  for (int i = 0; i < FFT_N; ++i) {
    z[i] = {(re[i].h + re[i].l) * (1.0 / FFT_N), (im[i].h + im[i].l) * (1.0 / FFT_N)};
    if (!errors) continue;
    const Q br = (Q)re[i].h + re[i].l - qr[i], bi = (Q)im[i].h + im[i].l - qi[i];
    const Q ar = (Q)z[i].r * FFT_N - qr[i], ai = (Q)z[i].i * FFT_N - qi[i];
    norm += qr[i] * qr[i] + qi[i] * qi[i];
    before += br * br + bi * bi;
    after += ar * ar + ai * ai;
  }
  if (errors) {
    errors[0] = std::max(errors[0], (double)sqrtq(before / norm) / UNIT_ROUNDOFF);
    errors[1] = std::max(errors[1], (double)sqrtq(after / norm) / UNIT_ROUNDOFF);
  }
  return z;
}

static int64_t exact(const std::vector<int32_t>* d, const std::vector<double>* key, int k) {
  int64_t sum = 0;
  for (int r = 0; r < 2 * ELL; ++r)
    for (int i = 0; i < RING_N; ++i) {
      const int64_t p = (int64_t)d[r][i] * (int64_t)key[r][(k - i) & (RING_N - 1)];
      sum += i <= k ? p : -p;
    }
  return sum;
}
static double norm2(const std::vector<int32_t>& x) {
  double s = 0;
  for (int32_t v : x) s += (double)v * v;
  return sqrt(s);
}
static double norm2(const std::vector<double>& x) {
  double s = 0;
  for (double v : x) s += v * v;
  return sqrt(s);
}
static int32_t low_field(uint64_t x) { return (int32_t)((uint32_t)x << (32 - LO_SHIFT)) >> (32 - LO_SHIFT); }
static uint64_t bits(double x) { return __builtin_bit_cast(uint64_t, x); }

static const char* const DIGITS[] = {"all -64", "all 63", "one wave", "signs", "uniform"};
static const char* const KEYS[] = {"lows down", "lows up", "A up B down", "one wave", "another wave", "uniform"};

int main() {
  make_fft_tables(&T);
  const uint32_t E = 1u << (KEY_SHIFT - 1);
  const uint32_t pos_low = 0x7FFFFFFFu / (2 * E) * (2 * E) + E, pos_high = pos_low - 1, neg_high = 0x80000000u + E - 1,
                 neg_low = 0x80000000u + E;
  double worst[2] = {0, 0}, worst_units[2] = {0, 0}, key_error[2] = {0, 0};
  int64_t worst_low = 0;
  long wrong = 0;
  const int freqs[] = {0, 1, 301, 511};
  for (int f : freqs)
    for (int dk = 0; dk < 5; ++dk)
      for (int kk = 0; kk < 6; ++kk) {
        if (f != 0 && dk != 2 && kk != 3 && kk != 4) continue;  // no frequency in the case
        auto wave = [&](int fr, int i) { return cos(M_PI * (2 * fr + 1) * i / RING_N) >= 0; };
        std::vector<int32_t> d[2 * ELL];
        std::vector<uint32_t> key[2 * ELL];  // words of A, then of B
        std::vector<double> kv[2 * ELL];
        for (int r = 0; r < 2 * ELL; ++r) {
          d[r].resize(RING_N);
          key[r].resize(2 * RING_N);
          for (int i = 0; i < RING_N; ++i) {
            const uint32_t x = rnd();
            d[r][i] = dk == 0 ? -64 : dk == 1 ? 63 : dk == 2 ? (wave(f, i) ? 63 : -64) : dk == 3 ? ((x & 1) ? 63 : -64)
                                                                                                : (int)(x & 127) - 64;
            uint32_t a, b;
            switch (kk) {
              case 0: a = b = pos_low; break;
              case 1: a = b = neg_high; break;
              case 2: a = neg_high; b = pos_low; break;
              case 3: a = wave(f, i) ? pos_high : neg_low; b = 0u - a; break;
              case 4: a = b = wave((f + 37) & 511, i) ? pos_low : neg_high; break;
              default: a = rnd(); b = rnd(); break;
            }
            key[r][i] = a;
            key[r][RING_N + i] = b;
          }
        }
        Poly fd[2 * ELL];
        for (int r = 0; r < 2 * ELL; ++r) {
          fd[r].resize(FFT_N);
          for (int i = 0; i < FFT_N; ++i) fd[r][i] = {(double)d[r][i], (double)d[r][i + FFT_N]};
          for (int k = 0; k < 9; ++k) stage(fd[r], k, false);
        }
        std::vector<uint32_t> word[2] = {std::vector<uint32_t>(RING_N), std::vector<uint32_t>(RING_N)};
        for (int ch = 0; ch < FFT_CHANNELS; ++ch) {
          Poly s(FFT_N);
          double S = 0;
          for (int r = 0; r < 2 * ELL; ++r) {
            const uint32_t *a = key[r].data(), *b = a + RING_N;
            const Poly k = key_transform(ch, a, b, r == 0 ? key_error : nullptr);
            kv[r].resize(RING_N);
            for (int j = 0; j < RING_N; ++j) kv[r][j] = key_value(ch, a, b, j);
            S += norm2(d[r]) * norm2(kv[r]);
            for (int i = 0; i < FFT_N; ++i) {
              const Cplx x = fd[r][i], v = k[i];
              s[i].r = r ? __builtin_fma(x.r, v.r, s[i].r) : x.r * v.r;
              s[i].i = r ? __builtin_fma(x.r, v.i, s[i].i) : x.r * v.i;
              s[i].r = __builtin_fma(-x.i, v.i, s[i].r);
              s[i].i = __builtin_fma(x.i, v.r, s[i].i);
            }
          }
          for (int k = 8; k >= 0; --k) stage(s, k, true);
          const double magic = 6755399441055744.0;
          for (int j = 0; j < RING_N; ++j) {
            const double x = j < FFT_N ? s[j].r : s[j - FFT_N].i;
            const int64_t e = exact(d, kv, j);
            const double err = fabs(x - (double)e);
            worst[ch == 2] = std::max(worst[ch == 2], err);
            worst_units[ch == 2] = std::max(worst_units[ch == 2], err / (UNIT_ROUNDOFF * S));
            if (ch < 2) {
              word[ch][j] = (uint32_t)bits(x + magic) << KEY_SHIFT;
            } else {
              const int32_t la = low_field(bits(x + magic));
              const int32_t lb = low_field(bits(x + (magic + (double)(1 << (LO_SHIFT - 1)))) >> LO_SHIFT);
              worst_low = std::max<int64_t>(worst_low, std::max(abs(la), abs(lb)));
              word[0][j] += (uint32_t)la;
              word[1][j] += (uint32_t)lb;
            }
          }
        }
        long bad = 0;
        for (int c = 0; c < 2; ++c)
          for (int j = 0; j < RING_N; ++j) {
            uint32_t w = 0;
            for (int r = 0; r < 2 * ELL; ++r)
              for (int i = 0; i < RING_N; ++i) {
                const uint32_t p = (uint32_t)d[r][i] * key[r][c * RING_N + ((j - i) & (RING_N - 1))];
                w += i <= j ? p : 0u - p;
              }
            bad += w != word[c][j];
          }
        if (bad) printf("%ld wrong words: digits %s, key %s, frequency %d\n", bad, DIGITS[dk], KEYS[kk], f);
        wrong += bad;
      }
  printf("distance from the integer: hi %.4f (%.2f u S), packed %.4f (%.2f u S); largest low sum %lld\n", worst[0],
         worst_units[0], worst[1], worst_units[1], (long long)worst_low);
  printf("key transform: %.3g u before its rounding, %.3f u after\n", key_error[0], key_error[1]);
  const double bound[2] = {ERROR_UNITS * UNIT_ROUNDOFF * ROW_NORMS * MAX_HI, ERROR_UNITS * UNIT_ROUNDOFF * ROW_NORMS * MAX_LO};
  const bool ok = wrong == 0 && worst[0] <= bound[0] && worst[1] <= bound[1] && worst_units[0] <= ERROR_UNITS &&
                  worst_units[1] <= ERROR_UNITS && worst_low == 6 * 1024 * 64 * (int64_t)MAX_LO_WORD &&
                  key_error[0] <= 0.034 && key_error[1] <= 1.034;
  printf(ok ? "exactness OK\n" : "exactness FAILED\n");
  return ok ? 0 : 1;
}
