// Device kernels of libvlp: key preparation, batched blind rotation with
// sample extraction, batched key switching, and small helpers.
#include <hip/hip_runtime.h>

#include <cmath>
#include <type_traits>

#include "internal.h"
#include "fft.h"

namespace vlp {

// Global-address-space views: loads through them are global (not flat)
// loads, so they are not counted by the LDS wait of the transposes.
typedef const uint32_t __attribute__((address_space(1))) g_u32;

__device__ __forceinline__ KsItem ks_item(const KsSource& src, uint32_t t) {
  if (src.items) return src.items[t];
  KsItem it = src.first;
  it.u1 += (size_t)t * CT_N;
  if (it.u2) it.u2 += (size_t)t * CT_N;
  it.out += (size_t)t * CT_n;
  return it;
}

// ---------------------------------------------------------------------------
// Key preparation
// ---------------------------------------------------------------------------

// One workgroup of 256 threads per key polynomial and channel: splits the
// words (fft.h), transforms in LDS (a butterfly per thread and stage), scales
// by 1/512 and stores in layout 3, [8 registers][64 lanes].  Bound: double-
// precision issue (VALU 66% busy), 89 us per keyset (116 us with every sum and
// product normalised).
__global__ __launch_bounds__(256) void bk_transform_kernel(const uint32_t* __restrict__ bk_coeff,
                                                           double2* __restrict__ bk_fft,
                                                           const double4* __restrict__ dd_tw) {
  __shared__ DD s_re[FFT_N], s_im[FFT_N];
  const uint32_t row = blockIdx.x / FFT_CHANNELS, ch = blockIdx.x % FFT_CHANNELS;  // row = i * 6 + r
  const uint32_t* a = bk_coeff + (size_t)row * 2 * RING_N;
  for (uint32_t i = threadIdx.x; i < FFT_N; i += 256) {
    s_re[i] = {key_value(ch, a, a + RING_N, i), 0.0};
    s_im[i] = {key_value(ch, a, a + RING_N, i + FFT_N), 0.0};
  }
  const uint32_t t = threadIdx.x;
  for (int k = 0; k < 9; ++k) {
    __syncthreads();
    const uint32_t half = FFT_N >> (k + 1), b = t / half, u = b * 2 * half + t % half, v = u + half;
    const double4 w = dd_tw[(1 << k) + b];
    DD vr = s_re[v], vi = s_im[v], ur = s_re[u], ui = s_im[u];
    dd_bf(ur, ui, vr, vi, DD{w.x, w.y}, DD{w.z, w.w});
    s_re[u] = ur;
    s_im[u] = ui;
    s_re[v] = vr;
    s_im[v] = vi;
  }
  __syncthreads();
  // Rows in the order a step reads them: digit 0 of A, digit 0 of B, digit 1 of A, ...
  const uint32_t i_row = row / (2 * ELL), r = row % (2 * ELL);
  double2* out = bk_fft + ((size_t)(i_row * 2 * ELL + (r % ELL) * 2 + r / ELL) * FFT_CHANNELS + ch) * FFT_N;
  for (uint32_t i = t; i < FFT_N; i += 256) {
    const uint32_t lane = (i >> 5) | ((i & 8) << 1) | ((i & 16) << 1), m = ((i & 3) << 1) | ((i >> 2) & 1);
    out[m * 64 + lane] = make_double2((s_re[i].h + s_re[i].l) * (1.0 / FFT_N), (s_im[i].h + s_im[i].l) * (1.0 / FFT_N));
  }
}

// The key-switching key [1024][8][4][631] in the layout of KSK_WORDS
// (internal.h).  One thread per (group, tile, lane): it reads that output
// word's entries of 4 coefficients and 4 levels and writes their bytes as 12
// words of 16 bytes, a run of 1 KiB per wavefront each.
__global__ __launch_bounds__(256) void ksk_relayout_kernel(const uint32_t* __restrict__ in, uint4* __restrict__ out) {
  const uint32_t lane = threadIdx.x & 63, tile = blockIdx.x, q = blockIdx.y * 4 + (threadIdx.x >> 6);
  const uint32_t w = 32 * tile + (lane & 31), h = lane >> 5;
  uint32_t b[3][4][4] = {};  // [block][plane][word]
#pragma unroll
  for (uint32_t c = 0; c < 4; ++c)
#pragma unroll
    for (uint32_t t = 0; t < 4; ++t) {
      uint32_t f[3] = {0, 0, 0};
      if (w < (uint32_t)CT_n) {
        const uint32_t* k = in + (size_t)((4 * q + c) * KS_T + 4 * h + t) * 4 * CT_n + w;
        f[0] = k[CT_n];
        f[1] = k[2 * CT_n];
        f[2] = k[3 * CT_n] - f[0] - f[1];
      }
#pragma unroll
      for (uint32_t n = 0; n < 3; ++n) {
        const uint32_t d = 3 * t + n;
        uint32_t v = f[n];
#pragma unroll
        for (uint32_t p = 0; p < 4; ++p) {
          const int32_t s = (int8_t)(v & 0xFFu);
          b[d >> 2][p][d & 3] |= (uint32_t)(uint8_t)s << (8 * c);
          v = (v - (uint32_t)s) >> 8;
        }
      }
    }
  uint4* o = out + (size_t)(q * KS_TILES + tile) * (3 * 4 * 64) + lane;
#pragma unroll
  for (int k = 0; k < 3; ++k)
#pragma unroll
    for (int p = 0; p < 4; ++p) o[(k * 4 + p) * 64] = make_uint4(b[k][p][0], b[k][p][1], b[k][p][2], b[k][p][3]);
}

// ---------------------------------------------------------------------------
// Blind rotation + sample extraction, one wavefront per rotation
// (br1_kernel): the whole CMux in one wavefront, so its steps need no
// workgroup barrier.  Bound: double-precision FMA issue.  Per step and
// wavefront about 3,600 VALU instructions (320 of them lane swaps that take
// two issue slots): 6 forward and 3 inverse 512-point transforms (216 and 288
// FMAs or adds per lane), 576 product FMAs, 370 for rotation and digits, 180
// for rounding and recombination.  256 VGPRs, two wavefronts per SIMD, 8
// rotations per CU.
// The VALU issues for 15.7k of the 22.5k clocks of a step and wavefront at 8
// rotations per CU (counters: 70% busy).  Beside it the step moves 147 KB of
// key through the vector L1 (64 B/clk; a build without these loads takes 10.7
// instead of 12.0 ms for 2,048) and exchanges its transforms through LDS; both
// are kept in flight behind arithmetic (eight key loads always outstanding, the
// exchange's real parts under way while the imaginary ones are computed).
// Measured (rotations only): 2,048 in 12.0 ms (171k/s; the two-prime NTT
// kernel it replaces: 21.7 ms, 94k/s; 12.0 to 12.5 ms on
// different cards), 1,024 at 4 per CU in 7.1 ms (10.9 ms;
// 7.6 with at most 256 registers per wavefront, which 8 per CU need and which
// spill 20).
// ---------------------------------------------------------------------------
// The wavefronts of a workgroup read the same key: a barrier every few steps
// keeps them close enough to share it in the L1 and L2.  With 8 per CU every
// step is best (2,048 rotations back to back: 11.99 ms; every 8 steps 12.14,
// every 16 12.22); with 4, one per SIMD, the stalls of a barrier are not
// filled by another wavefront (1,024: 7.45 ms; every 8 7.16, every 16 7.12).
constexpr int steps_per_barrier(int rot) { return rot == 8 ? 1 : 16; }

// Rounding and the halves of the two lower digits: the top digit of a
// difference plus this offset is its top field read as a signed number, and
// the lower ones their fields minus 64, i.e. with bit 6 flipped, likewise.
constexpr uint32_t DEC_OFFSET = (1u << 24) + (1u << 17) + (1u << 10);

// Accumulator polynomial in LDS: rows of 32 coefficients behind one row that
// holds the negated last row, so that coefficient j - ab of a lane that falls
// off the front of row 0 is read there: the lanes of a row then share one sign.
constexpr int ACC_WORDS = 33 * 32;

// Gate pre-combination of word w and its modulus switch.
__device__ __forceinline__ uint32_t abar_of(const BrItem& I, uint32_t w) {
  uint32_t x = (uint32_t)I.ca * ((const g_u32*)I.a)[w];
  if (I.b) x += (uint32_t)I.cb * ((const g_u32*)I.b)[w];
  for (uint32_t t = 0; t < I.n_more; ++t) x += (uint32_t)I.cm * ((const g_u32*)I.more[t])[w];
  if (w == (uint32_t)LWE_n) x += I.cst;
  return (x + (1u << 20)) >> 21;
}

// The key is one stream of batches of 8 values per lane (one transformed
// digit polynomial's products with one channel), read in order; v holds the
// batch that comes next.  Each value is replaced by the one of the batch after
// as soon as it is used, so eight loads are always in flight, also while the
// next digit is transformed.
typedef int v4i __attribute__((ext_vector_type(4)));
__device__ __forceinline__ void key_load(double2 (&v)[8], __amdgpu_buffer_rsrc_t key, int lane16, int off, int m) {
  const v4i w = __builtin_amdgcn_raw_buffer_load_b128(key, lane16 + (m & 3) * 1024, off + (m >> 2) * 4096, 0);
  v[m] = __builtin_bit_cast(double2, w);
}
// Key rows are touched PREFETCH_STEPS ahead of their use, so that the loads of
// the wavefronts find them in L2: each XCD has its own L2, and its workgroups
// (blockIdx mod 8) share the step's 18 batches among their wavefronts (`batch`
// counts an XCD's wavefronts, those past 18 touch nothing), one 128-byte line
// per lane.  1,024 rotations with the key in HBM: 8.00 -> 7.07 ms (in the
// last-level cache 7.00 -> 7.06); 2,048: 12.35 -> 11.96 ms (11.96 either way).
// The other kernels hold the loads of a whole step or of its longest wait and gain
// nothing (br6_kernel, 256: 3.05 -> 2.93 ms, but 2.77 -> 2.93 from the cache).
constexpr int PREFETCH_STEPS = 4, NUM_XCD = 8, STEP_BATCHES = 2 * ELL * FFT_CHANNELS;
__device__ __forceinline__ uint32_t key_touch(__amdgpu_buffer_rsrc_t key, int lane, int i, int batch) {
  const int step = i + PREFETCH_STEPS;
  const bool use = batch < STEP_BATCHES && step < LWE_n;  // else: offsets out of the buffer's range load nothing
  return __builtin_amdgcn_raw_buffer_load_b32(key, lane * 128 + (use ? 0 : (int)BK_FFT_BYTES),
                                              use ? (step * STEP_BATCHES + batch) * 8192 : 0, 0);
}

// Brings the keys of a round's first and last rotation from HBM into the
// memory-side cache (256 MiB, two keys), one load per 128-byte line: workgroup
// part of parts, WARM_THREADS threads.  A rotation by itself waits for HBM in each
// of its steps when its key has not been used lately, as it keeps only a step's
// loads in flight; a workgroup on a CU that a small round leaves idle, which
// touches lines only, runs well ahead of it.  One rotation with a key from HBM:
// 3.23 -> 2.79 ms, 300: 4.82 -> 4.42 ms.  With the key there already: 2.77 -> 2.78
// and 4.39 -> 4.41 ms.  More such workgroups (4, 8, 32 or all idle CUs) gain
// nothing further.  Loading into the L2 just ahead of use would gain at most 4%
// more for one rotation and nothing for 37.
// A launch ends no earlier than its helpers, so a thread keeps WARM_LOADS loads
// in flight: a helper by itself with two keys then waits less often than the
// rotations have steps.  With one load at a time it waited 3,780 times: 510
// rotations with two keys took 4.71 ms (4.53 on another card; now 4.39) where
// 512, without a helper, take 4.44, and 255 took 2.96 (now 2.88).  The lines of
// two keys are taken in turn; those of further keys between them are not read.
constexpr uint32_t WARM_BLOCKS = 2, WARM_THREADS = 384, WARM_LOADS = 8;
constexpr uint32_t KEY_LINES = BK_FFT_BYTES / 128;
static_assert(2 * ((KEY_LINES + WARM_THREADS * WARM_LOADS - 1) / (WARM_THREADS * WARM_LOADS)) < LWE_n,
              "a helper by itself ends before the rotations");
__device__ __forceinline__ void key_warm(const BrItem* __restrict__ items, uint32_t count, uint32_t part,
                                         uint32_t parts) {
  const void *const first = items[0].bk, *const last = items[count - 1].bk;
  const uint32_t stride = parts * WARM_THREADS;
  auto touch = [&](const void* bk, uint32_t e) {  // line KEY_LINES is out of the buffer's range: nothing is read
    const __amdgpu_buffer_rsrc_t key = __builtin_amdgcn_make_buffer_rsrc((void*)bk, 0, (int)BK_FFT_BYTES, 0x00027000);
    uint32_t x[WARM_LOADS];
#pragma unroll
    for (uint32_t u = 0; u < WARM_LOADS; ++u)
      x[u] = __builtin_amdgcn_raw_buffer_load_b32(key, (int)(min(e + u * stride, KEY_LINES) * 128), 0, 0);
    asm volatile("" ::"v"(x[0]), "v"(x[1]), "v"(x[2]), "v"(x[3]), "v"(x[4]), "v"(x[5]), "v"(x[6]), "v"(x[7]));
  };
  for (uint32_t e = part * WARM_THREADS + threadIdx.x; e < KEY_LINES; e += WARM_LOADS * stride) {
    touch(first, e);
    if (last != first) touch(last, e);
  }
}

// Products of one transformed digit polynomial with one of its key channels:
// s += a * v (FIRST: s = a * v); NEXT: replaces v by the batch at offset off.
template <bool FIRST, bool NEXT>
__device__ __forceinline__ void key_products(Cplx (&s)[8], const Cplx (&a)[8], double2 (&v)[8],
                                             __amdgpu_buffer_rsrc_t key, int lane16, int off) {
#pragma unroll
  for (int m = 0; m < 8; ++m) {
    s[m].r = FIRST ? a[m].r * v[m].x : __builtin_fma(a[m].r, v[m].x, s[m].r);
    s[m].i = FIRST ? a[m].r * v[m].y : __builtin_fma(a[m].r, v[m].y, s[m].i);
    s[m].r = __builtin_fma(-a[m].i, v[m].y, s[m].r);
    s[m].i = __builtin_fma(a[m].i, v[m].x, s[m].i);
    if (NEXT) key_load(v, key, lane16, off, m);
    __builtin_amdgcn_sched_barrier(0);
  }
}

template <int ROT>
__global__ __launch_bounds__(64 * ROT) __attribute__((amdgpu_waves_per_eu(ROT > 4 ? 2 : 1))) void br1_kernel(
    const BrItem* __restrict__ items, uint32_t count, const double2* __restrict__ lane_tw) {
  __shared__ uint32_t s_acc[ROT][2 * ACC_WORDS];
  __shared__ double s_x[ROT][2 * XPOLY];
  __shared__ double2 s_tw[LANE_TW][64];
  for (int e = threadIdx.x; e < LANE_TW * 64; e += 64 * ROT) s_tw[0][e] = lane_tw[e];
  __syncthreads();
  const int lane = threadIdx.x & 63, c = lane >> 5, l = lane & 31, rho = lane & 15;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t idx = blockIdx.x * ROT + wave;
  if (idx >= count) {  // no rotation: only meets the others at their barriers
    for (int i = 0; i < LWE_n; i += steps_per_barrier(ROT)) __builtin_amdgcn_s_barrier();
    return;
  }
  const BrItem I = items[idx];
  uint32_t* acc = s_acc[wave] + c * ACC_WORDS + 32 + l;  // this lane's column of its polynomial
  const double2* tw = &s_tw[0][lane];
  double* xw = s_x[wave] + c * XPOLY + l;                 // layout 1 side of the exchange
  double* xr = s_x[wave] + XROW * rho + ((lane >> 5) << 1) + ((lane >> 4) & 1);  // layout 2 side
  // acc = (0, X^(-bbar) * mu * (1 + X + ... + X^1023)).
  {
    const uint32_t bbar = __builtin_amdgcn_readfirstlane(abar_of(I, LWE_n));
    const uint32_t rot = (2048u - bbar) & 2047u;
#pragma unroll
    for (int R = 0; R < 32; ++R) {
      const uint32_t j = 32 * R + l;
      const bool neg = (j < (rot & 1023u)) != (rot >= 1024u);
      const uint32_t v = c == 0 ? 0u : (neg ? (0u - I.mu) : I.mu);
      acc[32 * R] = v;
      if (R == 31) acc[-32] = 0u - v;
    }
  }
  const double magic = 6755399441055744.0;  // 1.5 * 2^52: the sum's low words are the nearest integer
  const int unit = wave * (int)((gridDim.x + NUM_XCD - 1) / NUM_XCD) + (int)(blockIdx.x / NUM_XCD);
  uint32_t own[32];  // this lane's accumulator coefficients
#pragma unroll
  for (int R = 0; R < 32; ++R) own[R] = acc[32 * R];
  uint32_t abars = 0;
  const __amdgpu_buffer_rsrc_t key =
      __builtin_amdgcn_make_buffer_rsrc((void*)I.bk, 0, (int)BK_FFT_BYTES, 0x00027000);
  const int lane16 = lane * 16;
  int off = 0;
  double2 v[8];
#pragma unroll
  for (int m = 0; m < 8; ++m) key_load(v, key, lane16, off, m);
  for (int i = 0; i < LWE_n; ++i) {
    if (i % steps_per_barrier(ROT) == 0) __builtin_amdgcn_s_barrier();
    if ((i & 63) == 0) abars = i + lane < LWE_n ? abar_of(I, i + lane) : 0u;
    const uint32_t ab = __builtin_amdgcn_readlane(abars, i & 63);
    const int abh = (int)(ab >> 5), abl = (int)(ab & 31);
    uint32_t D[32];
    wave_lds_sync();  // the accumulator updates of the last step
    {
      const uint32_t* src = acc - abl;
      uint32_t w[32];
#pragma unroll
      for (int R = 0; R < 32; ++R) w[R] = src[((R - abh) & 31) * 32];
#pragma unroll
      for (int R = 0; R < 32; ++R) {
        const uint32_t mask = 0u - (uint32_t)(((R - abh) >> 5) & 1);
        D[R] = (w[R] ^ mask) + ((DEC_OFFSET - mask) - own[R]);
      }
    }
    Cplx s[FFT_CHANNELS][8];
    // The second and third digits of two coefficients share a word, which
    // halves the registers they occupy while the first is worked on.
    uint32_t P[16];
    auto digit = [&](auto first_t, unsigned shift) {
      constexpr bool first = decltype(first_t)::value;
      Cplx z[16];
#pragma unroll
      for (int q = 0; q < 16; ++q) {
        if constexpr (first) {
          z[q].r = (double)((int)D[q] >> 25);
          z[q].i = (double)((int)D[16 + q] >> 25);
          P[q] = (((D[q] >> 9) & 0xFFFFu) | ((D[16 + q] << 7) & 0xFFFF0000u)) ^ 0x81008100u;
        } else {
          z[q].r = (double)(int)__builtin_amdgcn_sbfe(P[q], shift, (unsigned)BG_BIT);
          z[q].i = (double)(int)__builtin_amdgcn_sbfe(P[q], shift + 16, (unsigned)BG_BIT);
        }
      }
      fwd_stage1<0>(z);
      fwd_stage1<1>(z);
      fwd_stage1<2>(z);
      // Stage 3 and the exchange of its outputs, real parts first: they are on
      // their way while the imaginary parts are computed.
      Cplx a[8], b[8];
      wave_lds_sync();
#pragma unroll
      for (int q = 0; q < 16; q += 2) {
        const double wr = W_RE[w_index(3, q >> 1)], wi = W_IM[w_index(3, q >> 1)];
        const Cplx &u = z[q], &w = z[q + 1];
        const double x = (q >> 1) & 1 ? __builtin_fma(-wr, w.i, __builtin_fma(-wi, w.r, u.r))
                                      : __builtin_fma(wr, w.r, __builtin_fma(-wi, w.i, u.r));
        xw[XROW * q] = x;
        xw[XROW * (q + 1)] = __builtin_fma(2.0, u.r, -x);
      }
      wave_lds_sync();
#pragma unroll
      for (int m = 0; m < 8; ++m) a[m].r = xr[4 * m];
#pragma unroll
      for (int m = 0; m < 8; ++m) b[m].r = xr[XPOLY + 4 * m];
      wave_lds_sync();
#pragma unroll
      for (int q = 0; q < 16; q += 2) {
        const double wr = W_RE[w_index(3, q >> 1)], wi = W_IM[w_index(3, q >> 1)];
        const Cplx &u = z[q], &w = z[q + 1];
        const double x = (q >> 1) & 1 ? __builtin_fma(wr, w.r, __builtin_fma(-wi, w.i, u.i))
                                      : __builtin_fma(wr, w.i, __builtin_fma(wi, w.r, u.i));
        xw[XROW * q] = x;
        xw[XROW * (q + 1)] = __builtin_fma(2.0, u.i, -x);
      }
      wave_lds_sync();
      // A wavefront's LDS reads return in issue order: the twiddles first.
      const TwA ta = load_twa(tw);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int m = 0; m < 8; ++m) a[m].i = xr[4 * m];
      const TwB tb = load_twb(tw);
#pragma unroll
      for (int m = 0; m < 8; ++m) b[m].i = xr[XPOLY + 4 * m];
      __builtin_amdgcn_sched_barrier(0);
      fwd_stages456(a, ta);
      swap_23(a);
      fwd_stages78(a, tb);
      __builtin_amdgcn_sched_barrier(0);
      key_products<first, true>(s[0], a, v, key, lane16, off + 1 * 8192);
      fwd_stages456(b, ta);
      __builtin_amdgcn_sched_barrier(0);
      key_products<first, true>(s[1], a, v, key, lane16, off + 2 * 8192);
      swap_23(b);
      __builtin_amdgcn_sched_barrier(0);
      key_products<first, true>(s[2], a, v, key, lane16, off + 3 * 8192);
      double2 w[8];
#pragma unroll
      for (int m = 0; m < 8; ++m) key_load(w, key, lane16, off + 4 * 8192, m);
      __builtin_amdgcn_sched_barrier(0);
      fwd_stages78(b, tb);
      __builtin_amdgcn_sched_barrier(0);
      key_products<false, true>(s[0], b, v, key, lane16, off + 5 * 8192);
      key_products<false, false>(s[1], b, w, key, lane16, 0);
      off += 6 * 8192;
      key_products<false, true>(s[2], b, v, key, lane16, off);
    };
    digit(std::true_type(), 0);
#pragma unroll 1
    for (int shift = 9; shift > 0; shift -= 7) digit(std::false_type(), (unsigned)shift);
    const uint32_t touched = key_touch(key, lane, i, unit);
    __builtin_amdgcn_sched_barrier(0);
    // Inverse transforms; each exchange's reads are in flight while the other
    // channels are worked on.
    TwB tb = load_twb(tw);
    __builtin_amdgcn_sched_barrier(0);
    TwA ta = load_twa(tw);
    __builtin_amdgcn_sched_barrier(0);
    inv_stages87(s[0], tb);
    inv_stages87(s[1], tb);
    __builtin_amdgcn_sched_barrier(0);
    swap_23(s[0]);
    swap_23(s[1]);
    __builtin_amdgcn_sched_barrier(0);
    inv_stages654(s[0], ta);
    inv_stages654(s[1], ta);
    __builtin_amdgcn_sched_barrier(0);
    Cplx h[16];
    wave_lds_sync();
#pragma unroll
    for (int m = 0; m < 8; ++m) xr[4 * m] = s[0][m].r;
#pragma unroll
    for (int m = 0; m < 8; ++m) xr[XPOLY + 4 * m] = s[1][m].r;
    wave_lds_sync();
#pragma unroll
    for (int q = 0; q < 16; ++q) h[q].r = xw[XROW * q];
    wave_lds_sync();
#pragma unroll
    for (int m = 0; m < 8; ++m) xr[4 * m] = s[0][m].i;
#pragma unroll
    for (int m = 0; m < 8; ++m) xr[XPOLY + 4 * m] = s[1][m].i;
    wave_lds_sync();
#pragma unroll
    for (int q = 0; q < 16; ++q) h[q].i = xw[XROW * q];
    __builtin_amdgcn_sched_barrier(0);
    inv_stages87(s[2], tb);
    swap_23(s[2]);
    inv_stages654(s[2], ta);
    __builtin_amdgcn_sched_barrier(0);
    // The packed channel over all 64 lanes (layout 4).
    double* pw = xr;
    const double* pr = s_x[wave] + XROW * 8 * c + l;
    Cplx z[8];
    wave_lds_sync();
#pragma unroll
    for (int m = 0; m < 8; ++m) {
      pw[4 * m] = s[2][m].r;
      pw[XPOLY + 4 * m] = s[2][m].i;
    }
    wave_lds_sync();
    const TwC tc = load_twc(tw);
#pragma unroll
    for (int m = 0; m < 8; ++m) {
      z[m].r = pr[XROW * m];
      z[m].i = pr[XPOLY + XROW * m];
    }
#pragma unroll
    for (int R = 0; R < 32; ++R) own[R] = acc[32 * R];
    __builtin_amdgcn_sched_barrier(0);
    inv_stage1<3>(h);
    inv_stage1<2>(h);
    inv_stage1<1>(h);
    inv_stage1<0>(h);
    uint32_t hi[32];
#pragma unroll
    for (int q = 0; q < 16; ++q) {
      hi[q] = (uint32_t)__builtin_bit_cast(uint64_t, h[q].r + magic);
      hi[16 + q] = (uint32_t)__builtin_bit_cast(uint64_t, h[q].i + magic);
    }
    __builtin_amdgcn_sched_barrier(0);
    inv_stages3210(z, tc);
    // Register m = (i8 i6 i5), lane (i7 | l): the integers of both outputs for
    // rows R (i7 = 0) and R + 4 (i7 = 1); a lane swap turns lane bit 5 from i7
    // into the output, as in hi.
#pragma unroll
    for (int t = 0; t < 16; ++t) {
      const int m = t & 7, R = 8 * (m >> 2) + 2 * ((m >> 1) & 1) + (m & 1) + 16 * (t >> 3);
      const double x = t < 8 ? z[m].r : z[m].i;
      const uint32_t la = __builtin_amdgcn_sbfe((uint32_t)__builtin_bit_cast(uint64_t, x + magic), 0u, (unsigned)LO_SHIFT);
      const uint64_t wb = __builtin_bit_cast(uint64_t, x + (magic + (double)(1 << (LO_SHIFT - 1))));
      const uint32_t lb = __builtin_amdgcn_sbfe(
          __builtin_amdgcn_alignbit((uint32_t)(wb >> 32), (uint32_t)wb, LO_SHIFT), 0u, (unsigned)LO_SHIFT);
      const auto lo = __builtin_amdgcn_permlane32_swap(la, lb, false, false);
      own[R] += (hi[R] << KEY_SHIFT) + lo[0];
      own[R + 4] += (hi[R + 4] << KEY_SHIFT) + lo[1];
      acc[32 * R] = own[R];
      acc[32 * (R + 4)] = own[R + 4];
    }
    acc[-32] = 0u - own[31];
    asm volatile("" ::"v"(touched));
  }
  wave_lds_sync();
  // SampleExtract: a'_0 = A_0, a'_j = -A_(N-j), b' = B_0.
  const uint32_t* A = s_acc[wave] + 32;
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int j = 64 * r + lane;
    const uint32_t a = A[j];
    if (j == 0) I.out[0] = a;
    else I.out[RING_N - j] = 0u - a;
  }
  if (lane == 0) I.out[RING_N] = A[ACC_WORDS];
}

// ---------------------------------------------------------------------------
// Blind rotation, three wavefronts per rotation and two rotations per
// workgroup (br3_kernel), for rounds of one to two rotations per CU: wavefront
// j transforms digit j of both accumulator halves, multiplies with its two key
// rows, hands the other wavefronts their channels' partial sums through LDS
// and transforms channel j (hi_A, hi_B, packed lo) back; the packed channel's
// integers go to the other two through LDS.  Three barriers per step.  Bound:
// the latency of that chain (about 1,300 VALU instructions, LDS round trips
// and barriers), which the two rotations fill for each other: 512 rotations in
// 4.4 ms (6.3 ms before, with four wavefronts and two-prime transforms), one
// per workgroup 3.1 ms for 256.
// ---------------------------------------------------------------------------
constexpr int BR3_ROT = 2;
__global__ __launch_bounds__(192 * BR3_ROT) __attribute__((amdgpu_waves_per_eu(2))) void br3_kernel(
    const BrItem* __restrict__ items, uint32_t count, const double2* __restrict__ lane_tw) {
  constexpr int REGION = 2 * XPOLY;  // doubles: one polynomial's values (1,024 doubles), padded for the exchange
  constexpr int REGIONS = 6;
  static_assert(192 * BR3_ROT == WARM_THREADS, "key_warm's workgroup");
  const uint32_t blocks = (count + BR3_ROT - 1) / BR3_ROT;
  if (blockIdx.x >= blocks) {
    key_warm(items, count, blockIdx.x - blocks, gridDim.x - blocks);
    return;
  }
  // No CU is idle: every workgroup reads its part first (512 rotations: 4.82 ->
  // 4.40 ms with a key from HBM, 4.38 and 4.36 ms otherwise).
  if (gridDim.x == blocks) key_warm(items, count, blockIdx.x, blocks);
  __shared__ double s_x[BR3_ROT][REGIONS][REGION];
  __shared__ double2 s_tw[LANE_TW][64];
  __shared__ uint32_t s_acc[BR3_ROT][2][3 * RING_N];
  for (int e = threadIdx.x; e < LANE_TW * 64; e += 192 * BR3_ROT) s_tw[0][e] = lane_tw[e];
  const int lane = threadIdx.x & 63, c = lane >> 5, l = lane & 31, rho = lane & 15;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int rot_i = wave / 3, j = wave % 3;
  const uint32_t idx = blockIdx.x * BR3_ROT + rot_i;
  const bool active = idx < count;
  const BrItem I = items[active ? idx : count - 1];  // an idle rotation repeats the last one and writes nothing
  const int j1 = j == 2 ? 0 : j + 1, j2 = j == 0 ? 2 : j - 1;  // (j + 1) mod 3, (j + 2) mod 3
  double(*X)[REGION] = s_x[rot_i];
  // Regions: wavefront j's first and second outgoing partial sums;
  // the region that only this wavefront reads last is its inverse exchange.
  double* mine = X[j];
  double* mine2 = X[3 + j];
  const double* in1 = X[j2];
  const double* in2 = X[3 + j1];
  double* inv = X[3 + j1];
  double* lo_words = X[3];  // wavefront 2's inverse region
  // Each accumulator polynomial p is held as the window p, -p, p: coefficient
  // t of X^ab p is word (-ab mod 2048) + t.
  const uint32_t* acc = s_acc[rot_i][c] + l;  // this lane's column of its half's polynomial
  const double2* tw = &s_tw[0][lane];
  double* xw = mine + c * XPOLY + l;
  double* xr = mine + XROW * rho + ((lane >> 5) << 1) + ((lane >> 4) & 1);
  if (j < 2) {
    const uint32_t bbar = __builtin_amdgcn_readfirstlane(abar_of(I, LWE_n));
    const uint32_t rot = (2048u - bbar) & 2047u;
#pragma unroll
    for (int R = 0; R < 16; ++R) {  // wavefront j: polynomial j
      const uint32_t jj = 64 * R + lane;
      const bool neg = (jj < (rot & 1023u)) != (rot >= 1024u);
      const uint32_t v = j == 0 ? 0u : (neg ? (0u - I.mu) : I.mu);
      uint32_t* p = s_acc[rot_i][j] + jj;
      p[0] = p[2 * RING_N] = v;
      p[RING_N] = 0u - v;
    }
  }
  // Offset of digit j: rounding and the halves of the digits below it; the
  // digit itself is then a signed 7-bit field.
  const unsigned shift = 32 - BG_BIT * (j + 1);
  const uint32_t offset = (1u << 10) + (j < 2 ? 1u << 17 : 0u) + (j < 1 ? 1u << 24 : 0u);
  const double magic = 6755399441055744.0;  // 1.5 * 2^52: the sum's low words are the nearest integer
  uint32_t abars = 0;
  const __amdgpu_buffer_rsrc_t key =
      __builtin_amdgcn_make_buffer_rsrc((void*)I.bk, 0, (int)BK_FFT_BYTES, 0x00027000);
  const int lane16 = lane * 16;
  int off = j * 6 * 8192;  // key batches of step i: ((3 i + j) * 2 + c) * 3 + channel
  // The step's six batches in the order they are used; v holds the next one.
  const int order[6] = {j1 * 8192, (3 + j1) * 8192, j2 * 8192, (3 + j2) * 8192, j * 8192, (3 + j) * 8192};
  double2 v[8];
#pragma unroll
  for (int m = 0; m < 8; ++m) key_load(v, key, lane16, off + order[0], m);
  __syncthreads();
  for (int i = 0; i < LWE_n; ++i, off += 18 * 8192) {
    if ((i & 63) == 0) abars = i + lane < LWE_n ? abar_of(I, i + lane) : 0u;
    const uint32_t ab = __builtin_amdgcn_readlane(abars, i & 63);
    Cplx z[16];
    {
      const uint32_t* src = acc + ((0u - ab) & (2 * RING_N - 1));
      uint32_t w[32], own[32];
#pragma unroll
      for (int R = 0; R < 32; ++R) w[R] = src[32 * R];
#pragma unroll
      for (int R = 0; R < 32; ++R) own[R] = acc[32 * R];
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int R = 0; R < 32; ++R) {
        const uint32_t D = (w[R] - own[R]) + offset;
        const double d = (double)(int)__builtin_amdgcn_sbfe(D, shift, (unsigned)BG_BIT);
        (R < 16 ? z[R & 15].r : z[R & 15].i) = d;
      }
    }
    fwd_stage1<0>(z);
    fwd_stage1<1>(z);
    fwd_stage1<2>(z);
    fwd_stage1<3>(z);
    Cplx a[8], b[8];
    wave_lds_sync();
#pragma unroll
    for (int q = 0; q < 16; ++q) xw[XROW * q] = z[q].r;
    wave_lds_sync();
#pragma unroll
    for (int m = 0; m < 8; ++m) a[m].r = xr[4 * m];
#pragma unroll
    for (int m = 0; m < 8; ++m) b[m].r = xr[XPOLY + 4 * m];
    wave_lds_sync();
#pragma unroll
    for (int q = 0; q < 16; ++q) xw[XROW * q] = z[q].i;
    wave_lds_sync();
    const TwA ta = load_twa(tw);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int m = 0; m < 8; ++m) a[m].i = xr[4 * m];
    const TwB tb = load_twb(tw);
#pragma unroll
    for (int m = 0; m < 8; ++m) b[m].i = xr[XPOLY + 4 * m];
    __builtin_amdgcn_sched_barrier(0);
    fwd_stages456(a, ta);
    swap_23(a);
    fwd_stages78(a, tb);
    __builtin_amdgcn_sched_barrier(0);
    // s = a K_a + b K_b per channel: the channels the other wavefronts own
    // first, then this one's.
    Cplx s[8];
    const int next = i + 1 < LWE_n ? off + 18 * 8192 : off;  // the next step's batches
    auto mul = [&](const Cplx (&x)[8], auto n_t) {
      constexpr int n = decltype(n_t)::value;
      const int to = (n < 5 ? off : next) + order[(n + 1) % 6];
#pragma unroll
      for (int m = 0; m < 8; ++m) {
        if constexpr (n % 2 == 0) {
          s[m].r = x[m].r * v[m].x;
          s[m].i = x[m].r * v[m].y;
        } else {
          s[m].r = __builtin_fma(x[m].r, v[m].x, s[m].r);
          s[m].i = __builtin_fma(x[m].r, v[m].y, s[m].i);
        }
        s[m].r = __builtin_fma(-x[m].i, v[m].y, s[m].r);
        s[m].i = __builtin_fma(x[m].i, v[m].x, s[m].i);
        key_load(v, key, lane16, to, m);
        if (m & 1) __builtin_amdgcn_sched_barrier(0);
      }
    };
    auto put = [&](double* to) {
      wave_lds_sync();
#pragma unroll
      for (int m = 0; m < 8; ++m) reinterpret_cast<double2*>(to)[m * 64 + lane] = make_double2(s[m].r, s[m].i);
      wave_lds_sync();
    };
    mul(a, std::integral_constant<int, 0>());
    fwd_stages456(b, ta);
    swap_23(b);
    fwd_stages78(b, tb);
    __builtin_amdgcn_sched_barrier(0);
    mul(b, std::integral_constant<int, 1>());
    put(mine);
    mul(a, std::integral_constant<int, 2>());
    mul(b, std::integral_constant<int, 3>());
    put(mine2);
    mul(a, std::integral_constant<int, 4>());
    mul(b, std::integral_constant<int, 5>());
    __syncthreads();
    double2 r1[8], r2[8];
#pragma unroll
    for (int m = 0; m < 8; ++m) r2[m] = reinterpret_cast<const double2*>(in2)[m * 64 + lane];
#pragma unroll
    for (int m = 0; m < 8; ++m) r1[m] = reinterpret_cast<const double2*>(in1)[m * 64 + lane];
    const TwB tbi = load_twb(tw);
    const TwA tai = load_twa(tw);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int m = 0; m < 8; ++m) {
      s[m].r += r1[m].x + r2[m].x;
      s[m].i += r1[m].y + r2[m].y;
    }
    inv_stages87(s, tbi);
    swap_23(s);
    inv_stages654(s, tai);
    double* iw = inv + XROW * rho + ((lane >> 5) << 1) + ((lane >> 4) & 1);
    const double* ir = inv + XROW * 8 * c + l;
    wave_lds_sync();
#pragma unroll
    for (int m = 0; m < 8; ++m) {
      iw[4 * m] = s[m].r;
      iw[XPOLY + 4 * m] = s[m].i;
    }
    wave_lds_sync();
    const TwC tc = load_twc(tw);
    Cplx h[8];
#pragma unroll
    for (int m = 0; m < 8; ++m) {
      h[m].r = ir[XROW * m];
      h[m].i = ir[XPOLY + XROW * m];
    }
    wave_lds_sync();
    __builtin_amdgcn_sched_barrier(0);
    inv_stages3210(h, tc);
    // Register m = (i8 i6 i5), lane (i7 | l): coefficient 32 R + l with
    // R = 8 i8 + 4 i7 + 2 i6 + i5 (real part) and R + 16 (imaginary part).
    uint32_t* ap = s_acc[rot_i][j & 1] + 128 * c + l;
    uint32_t* lo_at = reinterpret_cast<uint32_t*>(lo_words) + 128 * c + l;
    uint32_t old[16], hi[16];
    if (j == 2) {
      constexpr double half = (double)(1 << (LO_SHIFT - 1));
#pragma unroll
      for (int t = 0; t < 16; ++t) {
        const int m = t & 7, R = 8 * (m >> 2) + 2 * ((m >> 1) & 1) + (m & 1) + 16 * (t >> 3);
        const double x = t < 8 ? h[m].r : h[m].i;
        const uint32_t wa = (uint32_t)__builtin_bit_cast(uint64_t, x + magic);
        const uint64_t wb = __builtin_bit_cast(uint64_t, x + (magic + half));
        lo_at[32 * R] = __builtin_amdgcn_sbfe(wa, 0u, (unsigned)LO_SHIFT);
        lo_at[1024 + 32 * R] = __builtin_amdgcn_sbfe(
            __builtin_amdgcn_alignbit((uint32_t)(wb >> 32), (uint32_t)wb, LO_SHIFT), 0u, (unsigned)LO_SHIFT);
      }
    } else {
#pragma unroll
      for (int t = 0; t < 16; ++t) {
        const int m = t & 7, R = 8 * (m >> 2) + 2 * ((m >> 1) & 1) + (m & 1) + 16 * (t >> 3);
        old[t] = ap[32 * R];
        const uint32_t x = (uint32_t)__builtin_bit_cast(uint64_t, (t < 8 ? h[m].r : h[m].i) + magic);
        hi[t] = old[t] + (x << KEY_SHIFT);
      }
    }
    __syncthreads();
    if (j < 2) {
      uint32_t lo[16];
#pragma unroll
      for (int t = 0; t < 16; ++t) {
        const int m = t & 7, R = 8 * (m >> 2) + 2 * ((m >> 1) & 1) + (m & 1) + 16 * (t >> 3);
        lo[t] = lo_at[1024 * j + 32 * R];
      }
#pragma unroll
      for (int t = 0; t < 16; ++t) {
        const int m = t & 7, R = 8 * (m >> 2) + 2 * ((m >> 1) & 1) + (m & 1) + 16 * (t >> 3);
        const uint32_t x = hi[t] + lo[t];
        ap[32 * R] = ap[2 * RING_N + 32 * R] = x;
        ap[RING_N + 32 * R] = 0u - x;
      }
    }
    __syncthreads();
  }
  // SampleExtract: a'_0 = A_0, a'_j = -A_(N-j), b' = B_0.
  if (active) {
    const uint32_t *A = s_acc[rot_i][0] + RING_N;  // -A
    for (int jj = (int)threadIdx.x - rot_i * 192; jj < RING_N; jj += 192)
      I.out[jj] = jj == 0 ? A[-RING_N] : A[RING_N - jj];
    if (j == 0 && lane == 0) I.out[RING_N] = s_acc[rot_i][1][0];
  }
}

// ---------------------------------------------------------------------------
// Blind rotation, six wavefronts per rotation (br6_kernel), one rotation per
// workgroup and CU, for rounds of at most one per CU: wavefront w transforms
// row w (digit w / 2 of polynomial w mod 2) and leaves it in LDS; then half hf
// (i8) of channel ch of the products and of the inverse transform belong to
// wavefront 3 hf + ch; the halves meet in the last stage and the packed
// channel's integers go to the other four through LDS.  Four barriers per
// step.  Bound: the latency of that chain (660 VALU instructions per wavefront,
// two SIMDs carry two of the six); twiddles stay in registers and the step's
// 24 key values per lane are loaded a step ahead.  One rotation takes 2.77 ms,
// 256 take 2.78 ms (3.8 ms before, with four wavefronts and two-prime
// transforms; 3.07 and 3.18 ms with three wavefronts).
// ---------------------------------------------------------------------------
constexpr int INV_TW = 8;          // lane twiddles of the half-size inverse, per half
constexpr int HROW = 17, HCOMP = 16 * HROW;  // its exchange: element e at 17 (e >> 4) + (e & 15)

// 256 of a channel's 512 values (i8 fixed), four registers per lane.
struct HalfTw {
  double r[INV_TW], i[INV_TW];
};
__device__ __forceinline__ void swap_half(Cplx (&z)[4]) {  // register bit 1 <-> lane bit 5, bit 0 <-> lane bit 4
#pragma unroll
  for (int m = 0; m < 2; ++m) {
    swap_lane(z[m].r, z[m + 2].r, false);
    swap_lane(z[m].i, z[m + 2].i, false);
  }
#pragma unroll
  for (int m = 0; m < 4; m += 2) {
    swap_lane(z[m].r, z[m + 1].r, true);
    swap_lane(z[m].i, z[m + 1].i, true);
  }
}
// Two stages: register bit 0 (twiddle e, I times it where register bit 1 is set), then bit 1 (twiddle e + 1).
__device__ __forceinline__ void inv_half2(Cplx (&z)[4], const HalfTw& t, int e) {
  bf_inv<false>(z[0], z[1], t.r[e], t.i[e]);
  bf_inv<true>(z[2], z[3], t.r[e], t.i[e]);
  bf_inv<false>(z[0], z[2], t.r[e + 1], t.i[e + 1]);
  bf_inv<false>(z[1], z[3], t.r[e + 1], t.i[e + 1]);
}

__global__ __launch_bounds__(WARM_THREADS) __attribute__((amdgpu_waves_per_eu(2))) void br6_kernel(
    const BrItem* __restrict__ items, uint32_t count, const FftTables* __restrict__ tables) {
  __shared__ double s_x[6][2 * XPOLY];  // forward exchange, then the transformed digits; then the packed integers
  __shared__ double s_h[6][2 * HCOMP];  // inverse exchanges
  __shared__ uint32_t s_acc[2][3 * RING_N];  // each polynomial p as the window p, -p, p
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int j = w >> 1, c = w & 1;         // forward: digit j of polynomial c
  const int hf = w >= 3, ch = w - 3 * hf;  // products and inverse: half hf (i8) of channel ch
  if (blockIdx.x >= count) {
    key_warm(items, count, blockIdx.x - count, gridDim.x - count);
    return;
  }
  const BrItem I = items[blockIdx.x];
  // Twiddles in registers for the whole rotation.
  const double2* lt = reinterpret_cast<const double2*>(tables->lane) + lane;
  const TwA ta = load_twa(lt);
  const TwB tb = load_twb(lt);
  const TwC tc = load_twc(lt);
  HalfTw th;
#pragma unroll
  for (int e = 0; e < INV_TW; ++e) {
    th.r[e] = tables->half[hf][e][lane][0];
    th.i[e] = tables->half[hf][e][lane][1];
  }
  if (w < 4) {  // acc = (0, X^(-bbar) * mu * (1 + X + ... + X^1023)): four wavefronts, half a polynomial each
    const uint32_t bbar = __builtin_amdgcn_readfirstlane(abar_of(I, LWE_n));
    const uint32_t rot = (2048u - bbar) & 2047u;
#pragma unroll
    for (int R = 0; R < 8; ++R) {
      const uint32_t jj = 512 * (w & 1) + 64 * R + lane;
      const bool neg = (jj < (rot & 1023u)) != (rot >= 1024u);
      const uint32_t v = w < 2 ? 0u : (neg ? (0u - I.mu) : I.mu);
      uint32_t* p = s_acc[w >> 1] + jj;
      p[0] = p[2 * RING_N] = v;
      p[RING_N] = 0u - v;
    }
  }
  const unsigned shift = 32 - BG_BIT * (j + 1);
  const uint32_t offset = (1u << 10) + (j < 2 ? 1u << 17 : 0u) + (j < 1 ? 1u << 24 : 0u);
  const double magic = 6755399441055744.0;  // 1.5 * 2^52
  // Layout 4 backwards: register (i8 i6 i5), lane (i7 | l): row R = 8 i8 + 4 i7 + 2 i6 + i5, +16 for the imaginary part.
  const uint32_t* acc = s_acc[c] + 128 * (lane >> 5) + (lane & 31);
  double* xw = s_x[w] + XROW * 8 * (lane >> 5) + (lane & 31);
  const double* xr = s_x[w] + XROW * (lane & 15) + ((lane >> 5) << 1) + ((lane >> 4) & 1);
  double2* dw = reinterpret_cast<double2*>(s_x[w]) + lane;
  // Half layout: register (i1 i0), lane (i3 i2 | i4 | i7 i6 i5); stored index m 64 + lane' of layout 3.
  const int at = ((lane >> 4) & 1) * 64 + ((lane >> 3) & 1) * 32 + (lane >> 5) * 16 + hf * 8 + (lane & 7);
  const double2* dr = reinterpret_cast<const double2*>(s_x[0]) + at;
  constexpr int DROW = XPOLY;  // double2 between rows of s_x
  // Half exchange: write register (i3 i2), lane (i1 i0 | i4 | i7 i6 i5); read register (i5 i4), lane (i7 i6 | i3..i0).
  double* hw = s_h[w] + HROW * (2 * (lane & 7) + ((lane >> 3) & 1)) + ((lane >> 5) << 1) + ((lane >> 4) & 1);
  const double* hr = s_h[w] + HROW * (8 * (lane >> 5) + 4 * ((lane >> 4) & 1)) + (lane & 15);
  double2* pw = reinterpret_cast<double2*>(s_h[w]) + lane;
  const double2* pr = reinterpret_cast<const double2*>(s_h[hf ? w - 3 : w + 3]) + lane;
  uint32_t* lo_words = reinterpret_cast<uint32_t*>(s_x[0]) + 128 * hf + lane;
  const __amdgpu_buffer_rsrc_t key =
      __builtin_amdgcn_make_buffer_rsrc((void*)I.bk, 0, (int)BK_FFT_BYTES, 0x00027000);
  double2 k[6][4];  // the step's 24 key values of this lane
  auto load = [&](int i, int r) {  // row r: registers (i1 i0) at 0, 128, 256, 384
    const int o = ((i * 6 + r) * FFT_CHANNELS + ch) * 8192;
#pragma unroll
    for (int q = 0; q < 4; ++q)
      k[r][q] = __builtin_bit_cast(
          double2, __builtin_amdgcn_raw_buffer_load_b128(key, at * 16 + (q & 1) * 2048, o + (q >> 1) * 4096, 0));
  };
#pragma unroll
  for (int r = 0; r < 6; ++r) load(0, r);
  uint32_t abars = 0;
  __syncthreads();
  for (int i = 0; i < LWE_n; ++i) {
    if ((i & 63) == 0) abars = i + lane < LWE_n ? abar_of(I, i + lane) : 0u;
    const uint32_t ab = __builtin_amdgcn_readlane(abars, i & 63);
    Cplx z[8];
    {
      const uint32_t* src = acc + ((0u - ab) & (2 * RING_N - 1));
      uint32_t v[16], own[16];
#pragma unroll
      for (int t = 0; t < 16; ++t) {
        const int m = t & 7, R = 8 * (m >> 2) + 2 * ((m >> 1) & 1) + (m & 1) + 16 * (t >> 3);
        v[t] = src[32 * R];
        own[t] = acc[32 * R];
      }
#pragma unroll
      for (int t = 0; t < 16; ++t) {
        const uint32_t D = (v[t] - own[t]) + offset;
        (t < 8 ? z[t & 7].r : z[t & 7].i) = (double)(int)__builtin_amdgcn_sbfe(D, shift, (unsigned)BG_BIT);
      }
    }
    // Stage 0, register bit 2 (i8) <-> lane bit 5 (i7), stages 1-3.
#pragma unroll
    for (int m = 0; m < 4; ++m) bf_fwd<false>(z[m], z[m + 4], W_RE[0], W_IM[0]);
#pragma unroll
    for (int m = 0; m < 4; ++m) {
      swap_lane(z[m].r, z[m + 4].r, false);
      swap_lane(z[m].i, z[m + 4].i, false);
    }
    fwd_stages123(z, tc);
    wave_lds_sync();
#pragma unroll
    for (int m = 0; m < 8; ++m) {
      xw[XROW * m] = z[m].r;
      xw[XPOLY + XROW * m] = z[m].i;
    }
    wave_lds_sync();
#pragma unroll
    for (int m = 0; m < 8; ++m) {
      z[m].r = xr[4 * m];
      z[m].i = xr[XPOLY + 4 * m];
    }
    wave_lds_sync();
    fwd_stages456(z, ta);
    swap_23(z);
    fwd_stages78(z, tb);
#pragma unroll
    for (int m = 0; m < 8; ++m) dw[64 * m] = make_double2(z[m].r, z[m].i);
    __syncthreads();
    // Products of this half of the channel with all six rows.
    Cplx s[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) s[q] = {0.0, 0.0};
    const int next = i + 1 < LWE_n ? i + 1 : i;
#pragma unroll
    for (int r = 0; r < 6; ++r) {
      double2 d[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) d[q] = dr[DROW * r + 128 * q];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        s[q].r = __builtin_fma(d[q].x, k[r][q].x, s[q].r);
        s[q].i = __builtin_fma(d[q].x, k[r][q].y, s[q].i);
        s[q].r = __builtin_fma(-d[q].y, k[r][q].y, s[q].r);
        s[q].i = __builtin_fma(d[q].y, k[r][q].x, s[q].i);
      }
      load(next, r);
    }
    inv_half2(s, th, 0);
    swap_half(s);
    inv_half2(s, th, 2);
    wave_lds_sync();
#pragma unroll
    for (int q = 0; q < 4; ++q) {  // element: row i7..i4, column i3..i0
      hw[4 * q] = s[q].r;
      hw[HCOMP + 4 * q] = s[q].i;
    }
    wave_lds_sync();
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      s[q].r = hr[HROW * q];
      s[q].i = hr[HCOMP + HROW * q];
    }
    wave_lds_sync();
    inv_half2(s, th, 4);
    swap_half(s);
    inv_half2(s, th, 6);
    // Stage 0 joins the halves: this wavefront takes the positions with i7 = hf.
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const Cplx& g = hf ? s[q] : s[2 + q];
      pw[64 * q] = make_double2(g.r, g.i);
    }
    __syncthreads();
    Cplx o[4];  // (i8 i6)
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const double2 g = pr[64 * q];
      const Cplx other{g.x, g.y}, keep = hf ? s[2 + q] : s[q];
      o[q] = hf ? other : keep;
      o[2 + q] = hf ? keep : other;
      bf_inv<false>(o[q], o[2 + q], W_RE[0], W_IM[0]);
    }
    // Coefficient 256 i8 + 128 hf + 64 i6 + lane, +512 for the imaginary part.
    uint32_t x[8];
    uint32_t* ap = s_acc[ch & 1] + 128 * hf + lane;
    if (ch == 2) {
      constexpr double half = (double)(1 << (LO_SHIFT - 1));
#pragma unroll
      for (int t = 0; t < 8; ++t) {
        const double f = t < 4 ? o[t & 3].r : o[t & 3].i;
        const int J = 256 * ((t >> 1) & 1) + 64 * (t & 1) + 512 * (t >> 2);
        const uint32_t wa = (uint32_t)__builtin_bit_cast(uint64_t, f + magic);
        const uint64_t wb = __builtin_bit_cast(uint64_t, f + (magic + half));
        lo_words[J] = __builtin_amdgcn_sbfe(wa, 0u, (unsigned)LO_SHIFT);
        lo_words[1024 + J] = __builtin_amdgcn_sbfe(
            __builtin_amdgcn_alignbit((uint32_t)(wb >> 32), (uint32_t)wb, LO_SHIFT), 0u, (unsigned)LO_SHIFT);
      }
    } else {
#pragma unroll
      for (int t = 0; t < 8; ++t) {
        const int J = 256 * ((t >> 1) & 1) + 64 * (t & 1) + 512 * (t >> 2);
        const uint32_t h = (uint32_t)__builtin_bit_cast(uint64_t, (t < 4 ? o[t & 3].r : o[t & 3].i) + magic);
        x[t] = ap[J] + (h << KEY_SHIFT);
      }
    }
    __syncthreads();
    if (ch < 2) {
#pragma unroll
      for (int t = 0; t < 8; ++t) {
        const int J = 256 * ((t >> 1) & 1) + 64 * (t & 1) + 512 * (t >> 2);
        x[t] += lo_words[1024 * ch + J];
      }
#pragma unroll
      for (int t = 0; t < 8; ++t) {
        const int J = 256 * ((t >> 1) & 1) + 64 * (t & 1) + 512 * (t >> 2);
        ap[J] = ap[2 * RING_N + J] = x[t];
        ap[RING_N + J] = 0u - x[t];
      }
    }
    __syncthreads();
  }
  // SampleExtract: a'_0 = A_0, a'_j = -A_(N-j), b' = B_0.
  const uint32_t* A = s_acc[0] + RING_N;  // -A
  for (int jj = (int)threadIdx.x; jj < RING_N; jj += 384) I.out[jj] = jj == 0 ? A[-RING_N] : A[RING_N - jj];
  if (threadIdx.x == 0) I.out[RING_N] = s_acc[1][0];
}

// ---------------------------------------------------------------------------
// Key switching on the 8-bit matrix cores.
//
// The key switch of gate g subtracts, for every coefficient i < 1024 and
// level j < 8, the key entry K_d of the digit d = d_ij of a'_i + 2^15.  With
// the bits of d, K_d = b0 F_0 + b1 F_1 + b0 b1 F_2 (internal.h), so the sum is
// the product A x F of a 0/1 matrix of 3 columns per (i, j) and the words F;
// split into signed byte planes (F = sum_p 2^(8p) F_p mod 2^32) each plane's
// product is an exact integer (at most 24,576 terms of magnitude <= 128),
// computed by v_mfma_i32_32x32x32_i8, and the word is sum_p 2^(8p) C_p.  (One
// column per digit value, the zero entry included, takes a third more matrix
// work and key bytes, and a correction for unsigned bytes.)
//
// Four coefficients make three MFMA K-blocks: lane n + 32 h supplies for the
// levels j = 4 h + t the words d' = 3 t + f, byte c for coefficient c; with
// the group's digit bytes in one register x (byte c = digits of coefficient c,
// level t in bits 6 - 2t), b0 and b1 of all four are a shift and a mask each.
// The gate rows of the A operand are the lanes' n, the output words of the B
// operand the lanes' n.  A workgroup of 4 wavefronts covers 4 x RT x 32 gates
// and one tile of 32 output words (4 planes = 4 accumulators per 32 gates), or,
// SPLIT, RT x 32 gates with a quarter of the coefficients per wavefront, summed
// in LDS; blockIdx.z takes a range of coefficients, whose partial results are
// added atomically into outputs zeroed first when there is more than one range.
// ---------------------------------------------------------------------------
typedef int v16i __attribute__((ext_vector_type(16)));

// Digit bytes of count gates (input a' = u1 + u2):
// dig[(q * count + g) * 2 + h], byte c = bits [24 - 8h, 32 - 8h) of
// a'_(4q+c) + 2^15, i.e. the digits of levels 4h .. 4h + 3 of coefficient
// 4q + c, most significant first.  With zero_out the outputs are cleared
// (split key switching adds into them).  A workgroup turns a tile of 64 gates
// x 16 groups through LDS: 256-byte runs of a gate are read, 512-byte runs of
// a group written (one thread per (group, gate) read a gate's 16 bytes beside
// 63 others': 16,384 gates 94 us, now 31).
constexpr int PREP_G = 64, PREP_Q = 16;
__global__ __launch_bounds__(256) void ks_prep_kernel(KsSource src, uint32_t from, uint32_t count,
                                                      uint2* __restrict__ dig, int zero_out) {
  __shared__ uint2 s[PREP_Q][PREP_G + 1];
  const uint32_t g0 = blockIdx.x * PREP_G, q0 = blockIdx.y * PREP_Q;
  const uint32_t q = threadIdx.x & 15;
  for (uint32_t r = threadIdx.x >> 4; r < PREP_G; r += 16) {
    const uint32_t g = g0 + r;
    if (g >= count) break;
    const KsItem it = ks_item(src, from + g);
    const g_u32* u1 = (const g_u32*)it.u1 + 4 * (q0 + q);
    const g_u32* u2 = it.u2 ? (const g_u32*)it.u2 + 4 * (q0 + q) : nullptr;
    uint32_t hi = 0, lo = 0;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const uint32_t a = u1[c] + (u2 ? u2[c] : 0u) + 0x8000u;
      hi |= (a >> 24) << (8 * c);
      lo |= ((a >> 16) & 0xFFu) << (8 * c);
    }
    s[q][r] = make_uint2(hi, lo);
    if (zero_out)
#pragma unroll
      for (int c = 0; c < 4; ++c)
        if (4 * (q0 + q) + c < (uint32_t)CT_n) it.out[4 * (q0 + q) + c] = 0u;
  }
  __syncthreads();
  for (uint32_t t = threadIdx.x; t < PREP_G * PREP_Q; t += 256) {
    const uint32_t g = g0 + t % PREP_G, k = t / PREP_G;
    if (g < count) dig[(size_t)(q0 + k) * count + g] = s[k][t % PREP_G];
  }
}

template <int RT, bool SPLIT>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4 / RT))) void ks_mfma_kernel(
    KsSource src, uint32_t from, uint32_t count, const uint32_t* __restrict__ dig, const uint4* __restrict__ ksk,
    uint32_t groups_per_block) {
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t tile = blockIdx.x;
  const uint32_t row0 = (SPLIT ? blockIdx.y : blockIdx.y * 4 + wave) * (RT * 32);
  const uint32_t per_wave = SPLIT ? groups_per_block / 4 : groups_per_block;
  const uint32_t q_begin = blockIdx.z * groups_per_block + (SPLIT ? wave * per_wave : 0), q_end = q_begin + per_wave;
  const int n = lane & 31, h = lane >> 5;
  // Digit words of this lane's gate rows (rows past the last gate read the
  // last gate's digits; their results are not stored).
  const g_u32* dp[RT];
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) dp[rt] = (const g_u32*)dig + (size_t)min(row0 + rt * 32 + n, count - 1) * 2 + h;
  const size_t dstep = (size_t)count * 2;  // words between groups
  v16i acc[RT][4];
#pragma unroll
  for (int rt = 0; rt < RT; ++rt)
#pragma unroll
    for (int p = 0; p < 4; ++p) acc[rt][p] = v16i{};
  // Key fragments: [group][tile][3 blocks][4 planes][64 lanes], one block of
  // four loaded a block ahead of its use.
  const uint4* kb = ksk + (size_t)tile * (3 * 256) + lane;
  auto load_b = [&](uint32_t q, int block, v4i (&b)[4]) {
    const uint4* k = kb + (size_t)q * (KS_TILES * 3 * 256) + block * 256;
#pragma unroll
    for (int p = 0; p < 4; ++p) {
      const uint4 v = k[p * 64];
      b[p] = v4i{(int)v.x, (int)v.y, (int)v.z, (int)v.w};
    }
  };
  uint32_t dcur[RT], dnext[RT];
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) dcur[rt] = dp[rt][(size_t)q_begin * dstep];
  v4i b[3][4];
#pragma unroll
  for (int k = 0; k < 3; ++k) load_b(q_begin, k, b[k]);
  for (uint32_t q = q_begin; q < q_end; ++q) {
    const uint32_t qn = min(q + 1, q_end - 1);
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) dnext[rt] = dp[rt][(size_t)qn * dstep];
    int a[RT][12];
#pragma unroll
    for (int rt = 0; rt < RT; ++rt)
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const uint32_t b0 = (dcur[rt] >> (6 - 2 * t)) & 0x01010101u, b1 = (dcur[rt] >> (7 - 2 * t)) & 0x01010101u;
        a[rt][3 * t] = (int)b0;
        a[rt][3 * t + 1] = (int)b1;
        a[rt][3 * t + 2] = (int)(b0 & b1);
      }
#pragma unroll
    for (int k = 0; k < 3; ++k) {
#pragma unroll
      for (int rt = 0; rt < RT; ++rt)
#pragma unroll
        for (int p = 0; p < 4; ++p)
          acc[rt][p] = __builtin_amdgcn_mfma_i32_32x32x32_i8(
              v4i{a[rt][4 * k], a[rt][4 * k + 1], a[rt][4 * k + 2], a[rt][4 * k + 3]}, b[k][p], acc[rt][p], 0, 0, 0);
      load_b(qn, k, b[k]);
    }
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) dcur[rt] = dnext[rt];
  }
  // Result register r of lane n + 32 h: row 8 (r / 4) + 4 h + r mod 4, word n.
  const uint32_t w = tile * 32 + n;
  auto store = [&](uint32_t g, uint32_t sum) {
    if (g >= count || w >= (uint32_t)CT_n) return;
    const KsItem it = ks_item(src, from + g);
    uint32_t val = 0u - sum;
    if (w == (uint32_t)LWE_n && blockIdx.z == 0) val += it.u1[RING_N] + (it.u2 ? it.u2[RING_N] : 0u) + it.cst;
    if (gridDim.z == 1) it.out[w] = val;
    else atomicAdd(it.out + w, val);
  };
  auto word = [&](int rt, int r) {
    return (uint32_t)acc[rt][0][r] + ((uint32_t)acc[rt][1][r] << 8) + ((uint32_t)acc[rt][2][r] << 16) +
           ((uint32_t)acc[rt][3][r] << 24);
  };
  if constexpr (SPLIT) {
    __shared__ uint32_t s_part[4][RT * 16][64];
#pragma unroll
    for (int rt = 0; rt < RT; ++rt)
#pragma unroll
      for (int r = 0; r < 16; ++r) s_part[wave][rt * 16 + r][lane] = word(rt, r);
    __syncthreads();
#pragma unroll
    for (int k = 0; k < RT * 4; ++k) {
      const int e = wave * RT * 4 + k, rt = e >> 4, r = e & 15;
      store(row0 + rt * 32 + 8 * (r >> 2) + 4 * h + (r & 3),
            s_part[0][e][lane] + s_part[1][e][lane] + s_part[2][e][lane] + s_part[3][e][lane]);
    }
  } else {
#pragma unroll
    for (int rt = 0; rt < RT; ++rt)
#pragma unroll
      for (int r = 0; r < 16; ++r) store(row0 + rt * 32 + 8 * (r >> 2) + 4 * h + (r & 3), word(rt, r));
  }
}

// ---------------------------------------------------------------------------
// Helpers
// ---------------------------------------------------------------------------
__global__ void make_br_items_kernel(BrItem* items, uint32_t count, const uint32_t* a, const uint32_t* b, int32_t ca,
                                     int32_t cb, uint32_t cst, uint32_t mu, uint32_t* out, const void* bk) {
  const uint32_t t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= count) return;
  BrItem it;
  it.a = a + (size_t)t * CT_n;
  it.b = b ? b + (size_t)t * CT_n : nullptr;
  it.out = out + (size_t)t * CT_N;
  it.bk = bk;
  it.ca = ca;
  it.cb = cb;
  it.cst = cst;
  it.mu = mu;
  it.more = nullptr;
  it.n_more = 0;
  it.cm = 0;
  items[t] = it;
}

__global__ void negate_kernel(const uint32_t* a, uint32_t* out, size_t words) {
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < words; i += (size_t)gridDim.x * blockDim.x)
    out[i] = 0u - a[i];
}

// ServerEnc (Alg. 2): ciphertext t of a flat [count][631] array becomes
// pk[t] + (0, Ecd(bit_t)).  bit_t is bit (t mod l) of the int64 value t / l
// (LSB first, two's complement) when `vals` is given, else bytes[t] != 0.
__device__ __forceinline__ uint32_t enc_word(const int64_t* vals, const uint8_t* bytes, uint32_t l, size_t t) {
  const uint32_t bit = vals ? (uint32_t)(((uint64_t)vals[t / l] >> (t % l)) & 1u) : (uint32_t)(bytes[t] != 0);
  return bit ? MU : 0u - MU;
}

// Out of place, 16-byte accesses (pk and out 16-byte aligned): each thread
// issues U loads of four consecutive words (a block's U loads cover U
// consecutive runs of blockDim quads) before it adds the body words and
// stores, so U x 16 bytes per lane are in flight; the last words % 4 words
// are done by the first threads.  IDX is the index type: 32-bit when the
// array has fewer than 2^32 words (cheaper division by 631), else 64-bit.
// Loads and stores are non-temporal: every word is touched once.
__device__ __forceinline__ void add_body(uint4& w, uint32_t r, uint32_t e) {
  switch (CT_n - 1 - r) {
    case 0: w.x += e; break;
    case 1: w.y += e; break;
    case 2: w.z += e; break;
    default: w.w += e; break;
  }
}

template <typename IDX, int U>
__global__ void server_enc_copy_kernel(const uint4* __restrict__ pk, uint4* __restrict__ out, size_t count,
                                       const int64_t* __restrict__ vals, const uint8_t* __restrict__ bytes,
                                       uint32_t l) {
  const IDX words = (IDX)(count * CT_n), quads = words / 4;
  const IDX stride = (IDX)gridDim.x * blockDim.x * U;
  for (IDX q0 = (IDX)blockIdx.x * blockDim.x * U + threadIdx.x; q0 < quads; q0 += stride) {
    uint4 w[U];
#pragma unroll
    for (int k = 0; k < U; ++k) {
      const IDX q = q0 + (IDX)k * blockDim.x;
      if (q < quads) {
        w[k].x = __builtin_nontemporal_load(&pk[q].x);
        w[k].y = __builtin_nontemporal_load(&pk[q].y);
        w[k].z = __builtin_nontemporal_load(&pk[q].z);
        w[k].w = __builtin_nontemporal_load(&pk[q].w);
      }
    }
#pragma unroll
    for (int k = 0; k < U; ++k) {
      const IDX q = q0 + (IDX)k * blockDim.x;
      if (q < quads) {
        const IDX w0 = 4 * q;
        const IDX t = w0 / CT_n;
        const uint32_t r = (uint32_t)(w0 - t * CT_n);  // word index of w.x inside ciphertext t
        if (r >= CT_n - 4) add_body(w[k], r, enc_word(vals, bytes, l, t));  // the body word is one of the four
        __builtin_nontemporal_store(w[k].x, &out[q].x);
        __builtin_nontemporal_store(w[k].y, &out[q].y);
        __builtin_nontemporal_store(w[k].z, &out[q].z);
        __builtin_nontemporal_store(w[k].w, &out[q].w);
      }
    }
  }
  const IDX tid = (IDX)blockIdx.x * blockDim.x + threadIdx.x;
  if (tid < words - 4 * quads) {
    const IDX wi = 4 * quads + tid;
    const IDX t = wi / CT_n;
    uint32_t v = reinterpret_cast<const uint32_t*>(pk)[wi];
    if (wi - t * CT_n == CT_n - 1) v += enc_word(vals, bytes, l, t);
    reinterpret_cast<uint32_t*>(out)[wi] = v;
  }
}

// Word-granular form of the copy for buffers that are not 16-byte aligned.
__global__ void server_enc_word_kernel(const uint32_t* __restrict__ pk, uint32_t* __restrict__ out, size_t count,
                                       const int64_t* __restrict__ vals, const uint8_t* __restrict__ bytes,
                                       uint32_t l) {
  const size_t words = count * CT_n;
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < words; i += (size_t)gridDim.x * blockDim.x) {
    const size_t t = i / CT_n;
    uint32_t v = pk[i];
    if (i - t * CT_n == CT_n - 1) v += enc_word(vals, bytes, l, t);
    out[i] = v;
  }
}

// In place (out == pk): only the body words change.
__global__ void server_enc_inplace_kernel(uint32_t* ct, size_t count, const int64_t* __restrict__ vals,
                                          const uint8_t* __restrict__ bytes, uint32_t l) {
  for (size_t t = (size_t)blockIdx.x * blockDim.x + threadIdx.x; t < count; t += (size_t)gridDim.x * blockDim.x)
    ct[t * CT_n + CT_n - 1] += enc_word(vals, bytes, l, t);
}

// ---------------------------------------------------------------------------
// Fixed scratch of the allocation-free gate call.  Each device holds its own
// copy for the life of the process.  On the host, `scratch` names a host-side
// stand-in, not device memory: host code uses only the address that
// noalloc_scratch_address() returns for the current device.
// ---------------------------------------------------------------------------
static __device__ __align__(256) uint8_t scratch[NOALLOC_BYTES];

int noalloc_scratch_address(void** p) {
  *p = nullptr;
  return (int)hipGetSymbolAddress(p, HIP_SYMBOL(scratch));
}

// ---------------------------------------------------------------------------
// Launchers
// ---------------------------------------------------------------------------
static inline hipStream_t S(void* s) { return reinterpret_cast<hipStream_t>(s); }

int launch_bk_transform(const uint32_t* bk_coeff, void* bk_fft, const FftTables* tables, void* stream) {
  hipLaunchKernelGGL(bk_transform_kernel, dim3(LWE_n * 2 * ELL * FFT_CHANNELS), dim3(256), 0, S(stream), bk_coeff,
                     reinterpret_cast<double2*>(bk_fft), reinterpret_cast<const double4*>(tables->dd));
  return (int)hipGetLastError();
}

int launch_ksk_relayout(const uint32_t* ksk_in, uint32_t* ksk_out, void* stream) {
  hipLaunchKernelGGL(ksk_relayout_kernel, dim3(KS_TILES, KS_GROUPS / 4), dim3(256), 0, S(stream), ksk_in,
                     reinterpret_cast<uint4*>(ksk_out));
  return (int)hipGetLastError();
}

int launch_br(const BrItem* items, uint32_t count, const FftTables* tables, uint32_t waves, uint32_t rot_per_block,
              uint32_t cus, void* stream) {
  if (count == 0) return 0;
  // Workgroups behind the rotations', on the CUs that those leave idle, read the
  // key ahead (key_warm).  A full round of br6 has none and goes without: its
  // own workgroups reading ahead would take 2.84 instead of 3.06 ms for 256
  // rotations with a key from HBM, but 2.81 instead of 2.78 ms otherwise.
  // br1 reads ahead step by step (key_touch) and gains nothing from it.
  const uint32_t blocks = (count + rot_per_block - 1) / rot_per_block;
  const uint32_t ahead = waves > 1 && blocks < cus ? std::min(WARM_BLOCKS, cus - blocks) : 0;
  const dim3 grid(blocks + ahead), block(64 * waves * rot_per_block);
  const double2* tw = reinterpret_cast<const double2*>(tables->lane);
  switch (waves * 16 + rot_per_block) {
    case 16 + 1: hipLaunchKernelGGL(br1_kernel<1>, grid, block, 0, S(stream), items, count, tw); break;
    case 16 + 2: hipLaunchKernelGGL(br1_kernel<2>, grid, block, 0, S(stream), items, count, tw); break;
    case 16 + 4: hipLaunchKernelGGL(br1_kernel<4>, grid, block, 0, S(stream), items, count, tw); break;
    case 16 + 8: hipLaunchKernelGGL(br1_kernel<8>, grid, block, 0, S(stream), items, count, tw); break;
    case 48 + 2: hipLaunchKernelGGL(br3_kernel, grid, block, 0, S(stream), items, count, tw); break;
    case 96 + 1: hipLaunchKernelGGL(br6_kernel, grid, block, 0, S(stream), items, count, tables); break;
    default: return (int)hipErrorInvalidValue;
  }
  return (int)hipGetLastError();
}

int launch_ks_group(const KsSource& src, uint32_t count, const uint32_t* ksk, uint32_t* dig,
                    uint32_t gates_per_block, uint32_t cus, void* stream) {
  if (!(gates_per_block == 128 || gates_per_block == 256 || gates_per_block == 512)) return (int)hipErrorInvalidValue;
  for (uint32_t first = 0; first < count; first += KS_CHUNK) {
    const uint32_t cnt = std::min(KS_CHUNK, count - first);
    // Gates per workgroup (gpb: 256 or 128, at most gates_per_block; registers
    // let a CU hold 512 / gpb such workgroups) and coefficient ranges per gate
    // tile (sp): the pair that minimises the rounds of workgroups the device
    // runs times the cycles of a round on one SIMD -- 384 matrix-core cycles
    // per coefficient for either tile, a quarter more for the smaller one,
    // whose workgroups read the key twice as often (8,197 gates: 607 us with
    // 256, 766 with 128; 1,024: 112 and 111) -- plus the workgroups' epilogues
    // (stores, or atomic adds when the ranges are split).  512 gates per
    // workgroup leave one wavefront per SIMD, whose load waits nothing fills
    // (682 and 158 us).  Up to 64 gates the key's bytes are what counts: the
    // wavefronts of a workgroup then share the gates and split the key, so
    // that each byte is read by one of them.
    uint32_t gpb = 128, best = 1, rows = 1;
    const bool split = cnt <= 64;
    if (split) {
      gpb = cnt <= 32 ? 32 : 64;
      best = 32;
    } else {
      double best_cost = -1;
      for (uint32_t g = std::min(gates_per_block, 256u); g >= 128; g /= 2)
        for (uint32_t sp = 1; sp <= 32; sp *= 2) {
          const uint32_t r = (cnt + g - 1) / g;
          const double rounds = std::ceil((double)r * KS_TILES * sp / (cus * (512 / g)));
          const double cost = rounds * ((double)(RING_N / sp) * (g == 256 ? 384.0 : 480.0) + (sp > 1 ? 8192.0 : 4096.0));
          if (best_cost < 0 || cost < best_cost) {
            gpb = g;
            best = sp;
            rows = r;
            best_cost = cost;
          }
        }
    }
    hipLaunchKernelGGL(ks_prep_kernel, dim3((cnt + PREP_G - 1) / PREP_G, KS_GROUPS / PREP_Q), dim3(256), 0, S(stream),
                       src, first, cnt, reinterpret_cast<uint2*>(dig), best > 1 ? 1 : 0);
    const dim3 grid(KS_TILES, rows, best);
    const uint32_t per = KS_GROUPS / best;
    const uint4* k = reinterpret_cast<const uint4*>(ksk);
    switch (gpb) {
      case 32: hipLaunchKernelGGL((ks_mfma_kernel<1, true>), grid, dim3(256), 0, S(stream), src, first, cnt, dig, k, per); break;
      case 64: hipLaunchKernelGGL((ks_mfma_kernel<2, true>), grid, dim3(256), 0, S(stream), src, first, cnt, dig, k, per); break;
      case 128: hipLaunchKernelGGL((ks_mfma_kernel<1, false>), grid, dim3(256), 0, S(stream), src, first, cnt, dig, k, per); break;
      default: hipLaunchKernelGGL((ks_mfma_kernel<2, false>), grid, dim3(256), 0, S(stream), src, first, cnt, dig, k, per); break;
    }
    const int e = (int)hipGetLastError();
    if (e != 0) return e;
  }
  return 0;
}

int launch_make_br_items(BrItem* items, uint32_t count, const uint32_t* a, const uint32_t* b, int32_t ca, int32_t cb,
                         uint32_t cst, uint32_t mu, uint32_t* out, const void* bk, void* stream) {
  if (count == 0) return 0;
  hipLaunchKernelGGL(make_br_items_kernel, dim3((count + 255) / 256), dim3(256), 0, S(stream), items, count, a, b, ca,
                     cb, cst, mu, out, bk);
  return (int)hipGetLastError();
}

int launch_negate(const uint32_t* a, uint32_t* out, size_t words, void* stream) {
  if (words == 0) return 0;
  hipLaunchKernelGGL(negate_kernel, dim3(1024), dim3(256), 0, S(stream), a, out, words);
  return (int)hipGetLastError();
}

int launch_server_enc(const uint32_t* pk, uint32_t* out, size_t count, const int64_t* vals, const uint8_t* bytes,
                      uint32_t l, void* stream) {
  if (count == 0) return 0;
  const size_t words = count * CT_n;
  if (pk == out) {
    const size_t blocks = std::min<size_t>((count + 255) / 256, 8192);
    hipLaunchKernelGGL(server_enc_inplace_kernel, dim3((uint32_t)blocks), dim3(256), 0, S(stream), out, count, vals,
                       bytes, l);
  } else if ((((uintptr_t)pk | (uintptr_t)out) & 15) == 0) {
    // One 16-byte word per thread in a grid that covers the buffer in one pass
    // (grid-stride only beyond 2^31 - 1 workgroups): measured 6.3 TB/s on a
    // plain copy, against 4.8 TB/s with 4,096 workgroups of 4 words per
    // thread.  The first workgroup also covers the word tail (< 4 words).
    const size_t quads = words / 4;
    const size_t blocks = std::max<size_t>(1, std::min<size_t>((quads + 255) / 256, 0x7fffffff));
    if (words < (1ull << 32))
      hipLaunchKernelGGL((server_enc_copy_kernel<uint32_t, 1>), dim3((uint32_t)blocks), dim3(256), 0, S(stream),
                         reinterpret_cast<const uint4*>(pk), reinterpret_cast<uint4*>(out), count, vals, bytes, l);
    else
      hipLaunchKernelGGL((server_enc_copy_kernel<uint64_t, 1>), dim3((uint32_t)blocks), dim3(256), 0, S(stream),
                         reinterpret_cast<const uint4*>(pk), reinterpret_cast<uint4*>(out), count, vals, bytes, l);
  } else {
    const size_t blocks = std::min<size_t>((words + 255) / 256, 8192);
    hipLaunchKernelGGL(server_enc_word_kernel, dim3((uint32_t)blocks), dim3(256), 0, S(stream), pk, out, count, vals,
                       bytes, l);
  }
  return (int)hipGetLastError();
}

}  // namespace vlp
