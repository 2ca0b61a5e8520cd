// Negacyclic transforms of length 1024 in double precision, in registers of
// one wavefront, and the exactness argument they carry.
//
// A real polynomial p of degree < 1024 modulo X^1024 + 1 is the complex
// polynomial z_i = p_i + I p_(i+512) modulo X^512 - I (the other factor is its
// conjugate).  Stage k splits each of the 2^k factors X^m - w into
// X^(m/2) - s and X^(m/2) + s with s = sqrt(w), the butterfly
// (u, v) -> (u + s v, u - s v); nine stages leave the 512 values.  Block b of
// stage k has s = exp(2 pi I (2^-(k+3) + brv_k(b) / 2^(k+1))), so block 2b + 1
// of a stage uses I times block 2b's.  No separate twist is needed, and the
// forward butterfly is six FMAs: x = u + s v (4), y = 2 u - x (2).
//
// Why the results are exact integers.  A CMux adds, per output word, the
// negacyclic products of six digit polynomials (|d| <= 64) with key
// polynomials.  Each key word k (taken signed, |k| <= 2^31) is split as
// k = 16 hi + lo, lo in [-8, 7]; three real products per coefficient are
// computed: hi of output A, hi of output B, and lo of both outputs packed as
// lo_A + 2^23 lo_B (|sum over lo| <= 6*1024*64*8 < 2^22, so the two parts
// separate).  Largest key values: |hi| <= 2^27, packed < 2^26.01.  With
// u = 2^-53 and S = sum over the six rows of ||d||_2 ||k||_2
// <= 6 * (32*64) * (32 max|k|) = 2^18.585 max|k|, the worst-case error of a
// coefficient is at most S times the sum of the relative errors along the way:
//   forward   9 stages x 3.72 u: x carries two roundings (<= u (|t| + |x|), t
//             the partial sum), y those and one more, the twiddle sqrt(2)/2 u;
//             in the 2-norm of an output pair at most (3.01 + 0.71) u;
//   key       1.04 u: one rounding after a transform in double-double, whose
//             twiddles are exact to 64 bits (below);
//   products  9.9 u: 12 FMAs per component, each u times a partial sum;
//   inverse   9 stages x 3.71 u: the difference (1), its product with the
//             twiddle (2), the twiddle (0.71).  An error made by stage k
//             reaches a coefficient through that stage's elements, which
//             cover disjoint groups of the 512 values: (1/512) sum |value|
//             <= S bounds it for every stage.
// Together 77.9 u S: 0.457 for hi and 0.23 for the packed part, below the 1/2
// that rounding to the nearest integer allows, for every key and input.  (With
// one channel per output, unsplit, the bound is 7.3: not exact for every
// input.)  Measured on extreme and random digits and keys: 0.04 and 0.02, at
// most 7.3 u S.
#pragma once
#include <stdint.h>

#include <hip/hip_runtime.h>

namespace vlp {

constexpr int FFT_N = 512;         // complex points
constexpr int KEY_SHIFT = 4;       // k = 16 hi + lo
constexpr int LO_SHIFT = 23;       // lo_A + 2^23 lo_B
constexpr int FFT_CHANNELS = 3;    // hi_A, hi_B, packed lo

// The bounds above: 77.9 u S below 1/2 for both kinds of channel, and the two
// packed sums apart.
constexpr double ERROR_UNITS = 77.9;
constexpr double MAX_LO_WORD = 1 << (KEY_SHIFT - 1);
constexpr double MAX_HI = (2147483648.0 + MAX_LO_WORD) / (1 << KEY_SHIFT);
constexpr double MAX_LO = MAX_LO_WORD * (1.0 + (double)(1 << LO_SHIFT));
constexpr double ROW_NORMS = 6.0 * (32 * 64) * 32;  // S / max|k|
constexpr double UNIT_ROUNDOFF = 1.0 / 9007199254740992.0;
static_assert(ERROR_UNITS * UNIT_ROUNDOFF * ROW_NORMS * MAX_HI < 0.46 &&
                  ERROR_UNITS * UNIT_ROUNDOFF * ROW_NORMS * MAX_LO < 0.46,
              "rounding to the nearest integer is exact");
static_assert(6 * 1024 * 64 * MAX_LO_WORD < (1 << (LO_SHIFT - 1)), "the packed sums separate");

// Word j of the key polynomials a (output A) and b (output B) in channel ch.
__host__ __device__ __forceinline__ double split_word(uint32_t word, double* hi) {  // lo; *hi
  const int32_t k = (int32_t)word, lo = (int32_t)(word << (32 - KEY_SHIFT)) >> (32 - KEY_SHIFT);
  *hi = (double)(((int64_t)k - lo) >> KEY_SHIFT);
  return (double)lo;
}
__host__ __device__ __forceinline__ double key_value(uint32_t ch, const uint32_t* a, const uint32_t* b, uint32_t j) {
  double hi;
  if (ch == 0) return split_word(a[j], &hi), hi;
  if (ch == 1) return split_word(b[j], &hi), hi;
  return split_word(a[j], &hi) + (double)(1 << LO_SHIFT) * split_word(b[j], &hi);
}

// Double-double arithmetic of the key's transform: an unevaluated sum h + l, l a
// few ulp of h.  The sums are never normalised on the way (l stays small over
// nine stages), which takes a third of the operations away.  The transform's
// error, relative in the 2-norm, is that of its twiddles: their angles are
// products of two long doubles (64 bits, below pi), each twiddle is within
// 2^-61.06, so nine stages stay below 0.034 u before the one rounding (2.2e-3 u
// measured against 128-bit arithmetic, 0.73 u after the rounding).
struct DD {
  double h, l;
};
__host__ __device__ __forceinline__ DD dd_add(DD a, DD b) {
#pragma clang fp contract(off)
  const double s = a.h + b.h, bb = s - a.h;
  return {s, ((a.h - (s - bb)) + (b.h - bb)) + (a.l + b.l)};
}
__host__ __device__ __forceinline__ DD dd_neg(DD a) { return {-a.h, -a.l}; }
__host__ __device__ __forceinline__ DD dd_dot(DD w, DD v, DD x, DD y) {  // w v + x y
#pragma clang fp contract(off)
  const double p = w.h * v.h, e = __builtin_fma(w.h, v.h, -p), q = x.h * y.h, f = __builtin_fma(x.h, y.h, -q);
  const double s = p + q, bb = s - p;
  const double lo = __builtin_fma(w.h, v.l, __builtin_fma(w.l, v.h, __builtin_fma(x.h, y.l, x.l * y.h)));
  return {s, ((p - (s - bb)) + (q - bb)) + ((e + f) + lo)};
}
// One butterfly of a stage with twiddle (wr, wi).
__host__ __device__ __forceinline__ void dd_bf(DD& ur, DD& ui, DD& vr, DD& vi, DD wr, DD wi) {
  const DD tr = dd_dot(wr, vr, dd_neg(wi), vi), ti = dd_dot(wr, vi, wi, vr);
  vr = dd_add(ur, dd_neg(tr));
  vi = dd_add(ui, dd_neg(ti));
  ur = dd_add(ur, tr);
  ui = dd_add(ui, ti);
}

struct Cplx {
  double r, i;
};

// Stage twiddles that depend on the register index only (stages 0-3, layout
// 1): entry (1 << k) / 2 + (b >> 1) of stage k, block b; block 2b + 1 is I
// times block 2b.
constexpr double W_RE[8] = {0.7071067811865476, 0.9238795325112867, 0.9807852804032304, 0.5555702330196022,
                            0.9951847266721969, 0.6343932841636455, 0.881921264348355,  0.2902846772544624};
constexpr double W_IM[8] = {0.7071067811865476,  0.3826834323650898, 0.19509032201612828, 0.8314696123025452,
                            0.0980171403295606, 0.773010453362737,  0.47139673682599764, 0.9569403357322088};
constexpr int w_index(int k, int b) { return (1 << k) / 2 + (b >> 1); }

// Forward butterfly with twiddle s (ROT: I s).
template <bool ROT>
__device__ __forceinline__ void bf_fwd(Cplx& u, Cplx& v, double sr, double si) {
  double xr, xi;
  if constexpr (!ROT) {
    xr = __builtin_fma(sr, v.r, __builtin_fma(-si, v.i, u.r));
    xi = __builtin_fma(sr, v.i, __builtin_fma(si, v.r, u.i));
  } else {
    xr = __builtin_fma(-sr, v.i, __builtin_fma(-si, v.r, u.r));
    xi = __builtin_fma(sr, v.r, __builtin_fma(-si, v.i, u.i));
  }
  v.r = __builtin_fma(2.0, u.r, -xr);
  v.i = __builtin_fma(2.0, u.i, -xi);
  u.r = xr;
  u.i = xi;
}

// Inverse butterfly (twice the inverse of the forward one): (x + y, conj(s) (x - y)).
template <bool ROT>
__device__ __forceinline__ void bf_inv(Cplx& x, Cplx& y, double sr, double si) {
  const double dr = x.r - y.r, di = x.i - y.i;
  x.r += y.r;
  x.i += y.i;
  const double vr = __builtin_fma(sr, dr, si * di), vi = __builtin_fma(sr, di, -(si * dr));
  y.r = ROT ? vi : vr;   // conj(I s) d = -I conj(s) d
  y.i = ROT ? -vr : vi;
}

// Layout 1: position i = 32 q + l, register q = 0..15, l = lane & 31; the two
// half-wavefronts hold two polynomials.  Stages 0-3 (register bits 3-0).
template <int K>
__device__ __forceinline__ void fwd_stage1(Cplx (&z)[16]) {
#pragma unroll
  for (int p = 0; p < 8; ++p) {
    constexpr int B = 8 >> K;  // register stride
    const int q = ((p / B) * 2 * B) + (p % B);
    const int b = q >> (4 - K);
    if (b & 1) bf_fwd<true>(z[q], z[q + B], W_RE[w_index(K, b)], W_IM[w_index(K, b)]);
    else bf_fwd<false>(z[q], z[q + B], W_RE[w_index(K, b)], W_IM[w_index(K, b)]);
  }
}
template <int K>
__device__ __forceinline__ void inv_stage1(Cplx (&z)[16]) {
#pragma unroll
  for (int p = 0; p < 8; ++p) {
    constexpr int B = 8 >> K;
    const int q = ((p / B) * 2 * B) + (p % B);
    const int b = q >> (4 - K);
    if (b & 1) bf_inv<true>(z[q], z[q + B], W_RE[w_index(K, b)], W_IM[w_index(K, b)]);
    else bf_inv<false>(z[q], z[q + B], W_RE[w_index(K, b)], W_IM[w_index(K, b)]);
  }
}

// Layouts 2 and 3: eight registers per lane, one polynomial over 64 lanes.
//   2: register (i4 i3 i2), lane (i1 i0 | i8 i7 i6 i5): stages 4, 5, 6
//   3: register (i1 i0 i2), lane (i4 i3 | i8 i7 i6 i5): stages 7, 8; the order
//      in which the key is stored
// Their stages' twiddles depend on the lane; per lane, seven complex values:
// stage 4, stage 5, stage 6 (i4 = 0, 1), stage 7, stage 8 (i2 = 0, 1).  Layout
// 4 (below) has four more.
constexpr int LANE_TW = 11;

__device__ __forceinline__ void swap_lane(double& a, double& b, bool rows16) {
  const uint64_t x = __builtin_bit_cast(uint64_t, a), y = __builtin_bit_cast(uint64_t, b);
  uint32_t xl = (uint32_t)x, xh = (uint32_t)(x >> 32), yl = (uint32_t)y, yh = (uint32_t)(y >> 32);
  if (rows16) {
    const auto l = __builtin_amdgcn_permlane16_swap(xl, yl, false, false);
    const auto h = __builtin_amdgcn_permlane16_swap(xh, yh, false, false);
    a = __builtin_bit_cast(double, ((uint64_t)h[0] << 32) | l[0]);
    b = __builtin_bit_cast(double, ((uint64_t)h[1] << 32) | l[1]);
  } else {
    const auto l = __builtin_amdgcn_permlane32_swap(xl, yl, false, false);
    const auto h = __builtin_amdgcn_permlane32_swap(xh, yh, false, false);
    a = __builtin_bit_cast(double, ((uint64_t)h[0] << 32) | l[0]);
    b = __builtin_bit_cast(double, ((uint64_t)h[1] << 32) | l[1]);
  }
}
// Layout 2 <-> 3 (its own inverse): register bit 2 <-> lane bit 5, register bit 1 <-> lane bit 4.
__device__ __forceinline__ void swap_23(Cplx (&z)[8]) {
#pragma unroll
  for (int m = 0; m < 4; ++m) {
    swap_lane(z[m].r, z[m + 4].r, false);
    swap_lane(z[m].i, z[m + 4].i, false);
  }
#pragma unroll
  for (int h = 0; h < 8; h += 4)
#pragma unroll
    for (int m = h; m < h + 2; ++m) {
      swap_lane(z[m].r, z[m + 2].r, true);
      swap_lane(z[m].i, z[m + 2].i, true);
    }
}

// tw: this lane's entry of an LDS table [LANE_TW][64].  TwA: stages 4-6, TwB: 7, 8.
struct TwA {
  double2 t0, t1, t2, t3;
};
struct TwB {
  double2 t4, t5, t6;
};
__device__ __forceinline__ TwA load_twa(const double2* tw) { return {tw[0], tw[64], tw[128], tw[192]}; }
__device__ __forceinline__ TwB load_twb(const double2* tw) { return {tw[256], tw[320], tw[384]}; }

__device__ __forceinline__ void fwd_stages456(Cplx (&z)[8], const TwA& t) {
#pragma unroll
  for (int m = 0; m < 4; ++m) bf_fwd<false>(z[m], z[m + 4], t.t0.x, t.t0.y);  // stage 4
#pragma unroll
  for (int m = 0; m < 2; ++m) {  // stage 5
    bf_fwd<false>(z[m], z[m + 2], t.t1.x, t.t1.y);
    bf_fwd<true>(z[m + 4], z[m + 6], t.t1.x, t.t1.y);
  }
  bf_fwd<false>(z[0], z[1], t.t2.x, t.t2.y);  // stage 6
  bf_fwd<true>(z[2], z[3], t.t2.x, t.t2.y);
  bf_fwd<false>(z[4], z[5], t.t3.x, t.t3.y);
  bf_fwd<true>(z[6], z[7], t.t3.x, t.t3.y);
}
__device__ __forceinline__ void fwd_stages78(Cplx (&z)[8], const TwB& t) {
#pragma unroll
  for (int m = 0; m < 4; m += 2) {  // stage 7 (i2 = m & 1)
    bf_fwd<false>(z[m], z[m + 4], t.t4.x, t.t4.y);
    bf_fwd<true>(z[m + 1], z[m + 5], t.t4.x, t.t4.y);
  }
  bf_fwd<false>(z[0], z[2], t.t5.x, t.t5.y);  // stage 8: i1 = m >> 2, i2 = m & 1
  bf_fwd<true>(z[4], z[6], t.t5.x, t.t5.y);
  bf_fwd<false>(z[1], z[3], t.t6.x, t.t6.y);
  bf_fwd<true>(z[5], z[7], t.t6.x, t.t6.y);
}
__device__ __forceinline__ void inv_stages87(Cplx (&z)[8], const TwB& t) {
  bf_inv<false>(z[0], z[2], t.t5.x, t.t5.y);
  bf_inv<true>(z[4], z[6], t.t5.x, t.t5.y);
  bf_inv<false>(z[1], z[3], t.t6.x, t.t6.y);
  bf_inv<true>(z[5], z[7], t.t6.x, t.t6.y);
#pragma unroll
  for (int m = 0; m < 4; m += 2) {
    bf_inv<false>(z[m], z[m + 4], t.t4.x, t.t4.y);
    bf_inv<true>(z[m + 1], z[m + 5], t.t4.x, t.t4.y);
  }
}
__device__ __forceinline__ void inv_stages654(Cplx (&z)[8], const TwA& t) {
  bf_inv<false>(z[0], z[1], t.t2.x, t.t2.y);
  bf_inv<true>(z[2], z[3], t.t2.x, t.t2.y);
  bf_inv<false>(z[4], z[5], t.t3.x, t.t3.y);
  bf_inv<true>(z[6], z[7], t.t3.x, t.t3.y);
#pragma unroll
  for (int m = 0; m < 2; ++m) {
    bf_inv<false>(z[m], z[m + 2], t.t1.x, t.t1.y);
    bf_inv<true>(z[m + 4], z[m + 6], t.t1.x, t.t1.y);
  }
#pragma unroll
  for (int m = 0; m < 4; ++m) bf_inv<false>(z[m], z[m + 4], t.t0.x, t.t0.y);
}

// Layout 4, one polynomial over 64 lanes on its way back: register (i7 i6 i5),
// lane (i8 | i4..i0), stages 3, 2, 1; then register bit 2 and lane bit 5 change
// places, register (i8 i6 i5), lane (i7 | i4..i0), stage 0.  tw: four complex
// values per lane: stage 3 (i7 = 0, 1), stage 2, stage 1.
struct TwC {
  double2 t7, t8, t9, t10;
};
__device__ __forceinline__ TwC load_twc(const double2* tw) { return {tw[448], tw[512], tw[576], tw[640]}; }
__device__ __forceinline__ void inv_stages3210(Cplx (&z)[8], const TwC& t) {
  bf_inv<false>(z[0], z[1], t.t7.x, t.t7.y);
  bf_inv<true>(z[2], z[3], t.t7.x, t.t7.y);
  bf_inv<false>(z[4], z[5], t.t8.x, t.t8.y);
  bf_inv<true>(z[6], z[7], t.t8.x, t.t8.y);
#pragma unroll
  for (int m = 0; m < 2; ++m) {
    bf_inv<false>(z[m], z[m + 2], t.t9.x, t.t9.y);
    bf_inv<true>(z[m + 4], z[m + 6], t.t9.x, t.t9.y);
  }
#pragma unroll
  for (int m = 0; m < 4; ++m) bf_inv<false>(z[m], z[m + 4], t.t10.x, t.t10.y);
#pragma unroll
  for (int m = 0; m < 4; ++m) {
    swap_lane(z[m].r, z[m + 4].r, false);
    swap_lane(z[m].i, z[m + 4].i, false);
  }
#pragma unroll
  for (int m = 0; m < 4; ++m) bf_inv<false>(z[m], z[m + 4], W_RE[0], W_IM[0]);
}

// Forward stages 1, 2, 3 in register (i7 i6 i5), lane (i8 | i4..i0).
__device__ __forceinline__ void fwd_stages123(Cplx (&z)[8], const TwC& t) {
#pragma unroll
  for (int m = 0; m < 4; ++m) bf_fwd<false>(z[m], z[m + 4], t.t10.x, t.t10.y);
#pragma unroll
  for (int m = 0; m < 2; ++m) {
    bf_fwd<false>(z[m], z[m + 2], t.t9.x, t.t9.y);
    bf_fwd<true>(z[m + 4], z[m + 6], t.t9.x, t.t9.y);
  }
  bf_fwd<false>(z[0], z[1], t.t7.x, t.t7.y);
  bf_fwd<true>(z[2], z[3], t.t7.x, t.t7.y);
  bf_fwd<false>(z[4], z[5], t.t8.x, t.t8.y);
  bf_fwd<true>(z[6], z[7], t.t8.x, t.t8.y);
}

// Exchange between layouts 1 and 2 through LDS, one component at a time:
// element i of a polynomial is double 33 (i >> 5) + (i & 31): 64-bit accesses
// are served 16 lanes at a time by 32 banks, so 16 consecutive doubles (layout
// 1) and 16 rows of one column (layout 2) each touch every bank once.  One wavefront's
// LDS operations complete in issue order: no wait between the passes.
constexpr int XROW = 33, XPOLY = 16 * XROW;  // doubles
__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

}  // namespace vlp
