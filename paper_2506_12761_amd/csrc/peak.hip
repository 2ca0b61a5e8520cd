// Measured integer peak of the blind rotation's arithmetic.
//
// The algorithmic count of a blind rotation is its modular multiplications:
// per CMux, 8 transforms of (N/2) log2 N butterflies (one multiplication
// each) and 12 N pointwise key products (Section 2.2: the external product
// of a CMux, computed with negacyclic transforms); each is carried out as one
// residue butterfly per prime of the two-prime residue system.  The bound
// such a count is priced against on the integer units can be derived from the
// instruction set (lanes x clock divided by the VALU instructions of one
// multiplication) or measured: this file measures it, with the residue
// butterflies of the cheapest exact integer form (26-bit primes; lazy signed
// Cooley-Tukey forward, Gentleman-Sande inverse, Shoup products), on
// register-resident values, every CU busy and no memory traffic inside the
// loop.  The blind rotation itself uses double-precision transforms (fft.h),
// which need fewer instructions; the rate of their butterflies is measured in the
// same way (fft_peak_kernel).
#include <hip/hip_runtime.h>

#include "fft.h"
#include "vlp.h"

namespace vlp {
namespace {

constexpr uint32_t PEAK_PRIME = 67104769u;  // 32766 * 2^11 + 1 < 2^26

// y w mod p in (-p/2, 3p/2) for |y| < 2^31, a signed twiddle |w| < p/2 and
// wq = floor(w 2^32 / p).
__device__ __forceinline__ uint32_t shoup_s(uint32_t y, uint32_t w, uint32_t wq, uint32_t p) {
  const uint32_t q = (uint32_t)__mulhi((int)y, (int)wq);
  return w * y - q * p;
}
// Cooley-Tukey: (x, y) -> (x + w y, x - w y), never reduced.
__device__ __forceinline__ void bfly_ct(uint32_t& x, uint32_t& y, uint32_t w, uint32_t wq, uint32_t p) {
  const uint32_t u = x;
  const uint32_t t = shoup_s(y, w, wq, p);
  x = u + t;
  y = u - t;
}
// Gentleman-Sande with a negated twiddle: (x, y) -> (x + y, (y - x) w); RED
// reduces the sum (a Shoup product by 1).
template <bool RED>
__device__ __forceinline__ void bfly_gs_neg(uint32_t& x, uint32_t& y, uint32_t w, uint32_t wq, uint32_t p) {
  const uint32_t u = x, v = y;
  x = RED ? shoup_s(u + v, 1u, (uint32_t)((1ull << 32) / p), p) : u + v;
  y = shoup_s(v - u, w, wq, p);
}
// Register of butterfly k of a stage that pairs register r with r | 2^RB.
template <int RB>
__device__ __forceinline__ constexpr int bfly_reg(int k) {
  return ((k >> RB) << (RB + 1)) | (k & ((1 << RB) - 1));
}

constexpr int PEAK_THREADS = 256;
constexpr int PEAK_WAVES_PER_CU = 32;  // 8 per SIMD: enough to hide the multiply latency
constexpr int PEAK_ITERS = 2048;
constexpr int BFLY_PER_ITER = 4 * 8;   // four stages (register strides 8, 4, 2, 1) of 8 butterflies

// One lane's 16 residues, transformed over and over by the stages a
// transform runs inside a lane.
template <bool INV>
__global__ __launch_bounds__(PEAK_THREADS) void butterfly_peak_kernel(uint32_t* out, uint32_t seed, int iters) {
  constexpr uint32_t p = PEAK_PRIME;
  const uint32_t tid = blockIdx.x * PEAK_THREADS + threadIdx.x;
  uint32_t x[16], w[8], wp[8];
#pragma unroll
  for (int r = 0; r < 16; ++r) x[r] = ((seed ^ (tid * 16u + r)) * 2654435761u) % p;
#pragma unroll
  for (int k = 0; k < 8; ++k) {  // signed twiddles |w| < p/2 with floor(w 2^32 / p), as the tables hold
    const int64_t w0 = ((seed + tid) * (2u * k + 3u) + 12345u * k) % p;
    const int64_t ws = w0 > p / 2 ? w0 - (int64_t)p : w0;
    const int64_t n = ws * ((int64_t)1 << 32);
    w[k] = (uint32_t)(int32_t)ws;
    wp[k] = (uint32_t)(int32_t)(n / (int64_t)p - ((n % (int64_t)p != 0 && n < 0) ? 1 : 0));
    // Opaque from here on, as twiddles read from memory are: otherwise the
    // compiler folds their derivation into the products.
    asm volatile("" : "+v"(w[k]), "+v"(wp[k]));
  }
  for (int i = 0; i < iters; ++i) {
    // Forward: the transform's butterflies never reduce, so over the loop's
    // thousands of stages the values leave the residue ranges and wrap
    // modulo 2^32; the instructions, and so their timing, do not depend on
    // the values.  Inverse: sums double the bound three times (2P -> 16P) and
    // the fourth stage reduces them, the pattern of the inverse transform.
#pragma unroll
    for (int k = 0; k < 8; ++k) {  // register stride 8
      const int r = bfly_reg<3>(k);
      if (INV) bfly_gs_neg<false>(x[r], x[r | 8], w[k], wp[k], p); else bfly_ct(x[r], x[r | 8], w[k], wp[k], p);
    }
#pragma unroll
    for (int k = 0; k < 8; ++k) {  // stride 4
      const int r = bfly_reg<2>(k);
      if (INV) bfly_gs_neg<false>(x[r], x[r | 4], w[k], wp[k], p); else bfly_ct(x[r], x[r | 4], w[k], wp[k], p);
    }
#pragma unroll
    for (int k = 0; k < 8; ++k) {  // stride 2
      const int r = bfly_reg<1>(k);
      if (INV) bfly_gs_neg<false>(x[r], x[r | 2], w[k], wp[k], p); else bfly_ct(x[r], x[r | 2], w[k], wp[k], p);
    }
#pragma unroll
    for (int k = 0; k < 8; ++k) {  // stride 1
      const int r = bfly_reg<0>(k);
      if (INV) bfly_gs_neg<true>(x[r], x[r | 1], w[k], wp[k], p); else bfly_ct(x[r], x[r | 1], w[k], wp[k], p);
    }
  }
  uint32_t s = 0;
#pragma unroll
  for (int r = 0; r < 16; ++r) s ^= x[r];
  out[tid] = s;  // keeps the loop live; one word per thread, inside the buffer
}

// The same for the double-precision transforms: one lane's 16 complex values
// through stages 0 to 3 (forward) or 3 to 0 (inverse) of fft.h.  Four stages
// multiply the values by at most 4 in the 2-norm: they start near 2^-500 and are
// brought back every FFT_SCALE iterations, so that they stay normal numbers.
// 16 wavefronts per CU (four per SIMD): a butterfly's chain is three FMAs of 8
// clocks, and 8 independent ones are in each wavefront.  Measured: 5.20 T forward
// and 4.42 T inverse butterflies/s, 79% and 90% of the vector units' issue at
// 2.4 GHz.
constexpr int FFT_PEAK_WAVES_PER_CU = 16;
constexpr int FFT_SCALE = 256;
template <bool INV>
__global__ __launch_bounds__(PEAK_THREADS) void fft_peak_kernel(uint32_t* out, uint32_t seed, int iters) {
  const uint32_t tid = blockIdx.x * PEAK_THREADS + threadIdx.x;
  Cplx z[16];
#pragma unroll
  for (int q = 0; q < 16; ++q)
    z[q] = {(double)(((seed ^ (tid * 32u + q)) * 2654435761u) | 1u) * 0x1p-532,
            (double)(((seed ^ (tid * 32u + 16u + q)) * 2654435761u) | 1u) * 0x1p-532};
  for (int i = 0; i < iters; i += FFT_SCALE) {
    for (int k = 0; k < FFT_SCALE; ++k) {
      if constexpr (INV) {
        inv_stage1<3>(z);
        inv_stage1<2>(z);
        inv_stage1<1>(z);
        inv_stage1<0>(z);
      } else {
        fwd_stage1<0>(z);
        fwd_stage1<1>(z);
        fwd_stage1<2>(z);
        fwd_stage1<3>(z);
      }
    }
#pragma unroll
    for (int q = 0; q < 16; ++q) z[q] = {z[q].r * 0x1p-512, z[q].i * 0x1p-512};
  }
  double s = 0;
#pragma unroll
  for (int q = 0; q < 16; ++q) s += z[q].r + z[q].i;
  out[tid] = (uint32_t)(__builtin_bit_cast(uint64_t, s) >> 32);  // keeps the loop live; one word per thread
}

// Butterflies per second of kernel[0] (forward) and kernel[1] (inverse) on
// `device`, in a grid of waves_per_cu wavefronts per CU.
typedef void (*PeakKernel)(uint32_t*, uint32_t, int);
vlp_status measure(int device, const PeakKernel (&kernel)[2], int waves_per_cu, double (&rate)[2]) {
  int n_dev = 0;
  if (hipGetDeviceCount(&n_dev) != hipSuccess) return VLP_EHIP;
  if (device < 0 || device >= n_dev) return VLP_EINVAL;
  int old = 0;
  if (hipGetDevice(&old) != hipSuccess || hipSetDevice(device) != hipSuccess) return VLP_EHIP;
  int cus = 0;
  uint32_t* out = nullptr;
  hipStream_t st = nullptr;
  hipEvent_t ev[2] = {nullptr, nullptr};
  vlp_status status = VLP_OK;
  do {
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, device) != hipSuccess || cus <= 0) {
      status = VLP_EHIP;
      break;
    }
    const int blocks = cus * waves_per_cu * 64 / PEAK_THREADS;
    if (hipMalloc((void**)&out, (size_t)blocks * PEAK_THREADS * sizeof(uint32_t)) != hipSuccess ||
        hipStreamCreate(&st) != hipSuccess || hipEventCreate(&ev[0]) != hipSuccess ||
        hipEventCreate(&ev[1]) != hipSuccess) {
      status = VLP_EHIP;
      break;
    }
    const double bfly = (double)blocks * PEAK_THREADS * PEAK_ITERS * BFLY_PER_ITER;
    for (int inv = 0; inv < 2 && status == VLP_OK; ++inv) {
      float best = 0;
      for (int rep = 0; rep < 4; ++rep) {  // the first launch warms up; the fastest of the others counts
        if (hipEventRecord(ev[0], st) != hipSuccess) { status = VLP_EHIP; break; }
        hipLaunchKernelGGL(kernel[inv], dim3(blocks), dim3(PEAK_THREADS), 0, st, out, 0x5EEDu + rep, PEAK_ITERS);
        float ms = 0;
        if (hipGetLastError() != hipSuccess || hipEventRecord(ev[1], st) != hipSuccess ||
            hipEventSynchronize(ev[1]) != hipSuccess || hipEventElapsedTime(&ms, ev[0], ev[1]) != hipSuccess) {
          status = VLP_EHIP;
          break;
        }
        if (rep > 0 && (best == 0 || ms < best)) best = ms;
      }
      if (status == VLP_OK) rate[inv] = bfly / (best * 1e-3);
    }
  } while (0);
  if (ev[0]) (void)hipEventDestroy(ev[0]);
  if (ev[1]) (void)hipEventDestroy(ev[1]);
  if (st) (void)hipStreamDestroy(st);
  if (out) (void)hipFree(out);
  (void)hipSetDevice(old);
  return status;
}

}  // namespace
}  // namespace vlp

extern "C" vlp_status vlp_measure_modmul_peak(int device, double* fwd_per_s, double* inv_per_s, double* mixed_per_s) {
  using namespace vlp;
  if (!fwd_per_s || !inv_per_s || !mixed_per_s) return VLP_EINVAL;
  double rate[2] = {0, 0};
  const vlp_status status =
      measure(device, {butterfly_peak_kernel<false>, butterfly_peak_kernel<true>}, PEAK_WAVES_PER_CU, rate);
  if (status != VLP_OK) return status;
  *fwd_per_s = rate[0];
  *inv_per_s = rate[1];
  // A CMux runs six forward transforms and two inverse ones of equal size.
  *mixed_per_s = 8.0 / (6.0 / rate[0] + 2.0 / rate[1]);
  return VLP_OK;
}

extern "C" vlp_status vlp_measure_fft_peak(int device, double* fwd_per_s, double* inv_per_s, double* mixed_per_s) {
  using namespace vlp;
  if (!fwd_per_s || !inv_per_s || !mixed_per_s) return VLP_EINVAL;
  double rate[2] = {0, 0};
  const vlp_status status = measure(device, {fft_peak_kernel<false>, fft_peak_kernel<true>}, FFT_PEAK_WAVES_PER_CU, rate);
  if (status != VLP_OK) return status;
  *fwd_per_s = rate[0];
  *inv_per_s = rate[1];
  // A CMux runs six forward transforms and three inverse ones (its channels).
  *mixed_per_s = 9.0 / (6.0 / rate[0] + 3.0 / rate[1]);
  return VLP_OK;
}
