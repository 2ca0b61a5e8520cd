// Internal types shared by the kernels and the host runtime of libvlp.
#pragma once
#include <stddef.h>
#include <stdint.h>

#include <hip/hip_runtime.h>

namespace vlp {

constexpr int LWE_n = 630;          // LWE dimension (Table 5)
constexpr int RING_N = 1024;        // ring degree
constexpr int BG_BIT = 7;           // gadget base 2^7
constexpr int ELL = 3;              // gadget levels
constexpr int KS_BASEBIT = 2;       // key-switching base 2^2
constexpr int KS_T = 8;             // key-switching levels
constexpr int CT_n = LWE_n + 1;     // words of an LWE_n ciphertext
constexpr int CT_N = RING_N + 1;    // words of an LWE_N ciphertext
constexpr uint32_t MU = 0x20000000u; // 1/8

// Transformed bootstrapping key (fft.h): [630][6 rows][3 channels][8
// registers][64 lanes] complex doubles, each polynomial in the transform's
// order (layout 3, so a wavefront's loads are contiguous), scaled by 1/512.
constexpr size_t BK_ROW_POINTS = (size_t)2 * ELL * 3 * (RING_N / 2);  // complex points of one key row i
constexpr size_t BK_FFT_BYTES = (size_t)LWE_n * BK_ROW_POINTS * 16 + 8192;  // + one batch that is read ahead, not used
// Key-switching key laid out for the 8-bit matrix cores: for every coefficient
// i and level j the three words F_0 = K_1, F_1 = K_2, F_2 = K_3 - K_1 - K_2 of
// its entries K_v = [i][j][v] (mod 2^32; the entry v = 0 is ignored), so that
// K_d = b0 F_0 + b1 F_1 + b0 b1 F_2 for the bits b0, b1 of a digit d.  Each
// word as four signed bytes (F = sum_p 2^(8p) s_p mod 2^32, s_p in [-128,
// 127]).  [256 groups of 4 coefficients][20 tiles of 32 output words][3
// blocks][4 byte planes p][64 lanes][4 words]: lane n + 32 h, word d' = 4 block
// + word = 3 t + f holds, for output word 32 tile + n and level j = 4 h + t,
// byte s_p of F_f of the group's coefficients 0..3 in bytes 0..3; words past
// 630 are zero.
constexpr int KS_TILES = 20;                                           // 640 words / 32
constexpr int KS_GROUPS = RING_N / 4;
constexpr size_t KSK_WORDS = (size_t)KS_GROUPS * KS_TILES * 3 * 4 * 64 * 4;  // u32 words (62,914,560 B)

// One blind rotation: input = (0, cst) + ca * a + cb * b + cm * (more[0] +
// ... + more[n_more - 1]), output the sample-extracted LWE_N ciphertext of
// BlindRotate(input, mu).
struct BrItem {
  const uint32_t* a;
  const uint32_t* b;    // may be null (then cb is ignored)
  uint32_t* out;        // [1025]
  const void* bk;       // transformed bootstrapping key
  int32_t ca, cb;
  uint32_t cst, mu;
  const uint32_t* const* more;  // n_more further operands (k-input XOR), or null
  uint32_t n_more;
  int32_t cm;
};

// One key switch: input = u1 + u2 + (0, cst) in dimension N, output LWE_n.
struct KsItem {
  const uint32_t* u1;
  const uint32_t* u2;   // may be null
  uint32_t* out;        // [631]
  const uint32_t* ksk;  // re-laid key-switching key
  uint32_t cst;
  uint32_t pad;
};

// The key switches of a launch: an array of items in device memory, or (items
// null) elementwise ones, item t being `first` with its ciphertexts advanced t
// places.
struct KsSource {
  const KsItem* items;
  KsItem first;
};

// Fixed device scratch of the allocation-free gate call (vlp_gate_noalloc):
// the sample-extracted outputs of up to 2 blind rotations per gate, then the
// blind-rotation work items and the key-switching digits (2 KiB per gate), for
// at most NOALLOC_MAX_GATES gates per call.  One copy per device, in kernels.hip.
constexpr size_t NOALLOC_MAX_GATES = 1024;
constexpr size_t NOALLOC_EXT_BYTES = 2 * NOALLOC_MAX_GATES * CT_N * 4;   // multiple of 256
constexpr size_t NOALLOC_BYTES = NOALLOC_EXT_BYTES + 2 * NOALLOC_MAX_GATES * sizeof(BrItem) +
                                 NOALLOC_MAX_GATES * RING_N * 2;
// Device address of the current device's copy of that scratch (the HIP error
// of the lookup; call with the device current).
int noalloc_scratch_address(void** p);

// Twiddle tables of the transforms (fft.h): the lane-dependent ones of a
// wavefront, and every stage's as double-doubles {re, re_lo, im, im_lo} at
// index 2^k + block (the key's transform; entry 0 unused).
struct FftTables {
  double lane[11][64][2];
  double half[2][8][64][2];
  double dd[512][4];
};
void make_fft_tables(FftTables* t);
// The tables, made at the first call (0.1 ms) and shared by all contexts of the
// process; safe from several threads.  Made anew for each context they were nearly
// all of the time of creating and destroying one (0.52 ms, now 0.03).
const FftTables& fft_tables();

// Host-side launchers (kernels.hip).  All enqueue on `stream` and return the
// HIP error of the launch.  `tables` is a device pointer.
int launch_bk_transform(const uint32_t* bk_coeff, void* bk_fft, const FftTables* tables, void* stream);
int launch_ksk_relayout(const uint32_t* ksk_in, uint32_t* ksk_out, void* stream);
// Blind rotations by `waves` (1, 3 or 6) wavefronts each, rot_per_block of
// them per workgroup (1 wavefront: 1, 2, 4, 8; 3: 2; 6: 1).
int launch_br(const BrItem* items, uint32_t count, const FftTables* tables, uint32_t waves, uint32_t rot_per_block,
              uint32_t cus, void* stream);
// ServerEnc over a flat [count][631] array; out == pk runs in place.
int launch_server_enc(const uint32_t* pk, uint32_t* out, size_t count, const int64_t* vals, const uint8_t* bytes,
                      uint32_t l, void* stream);
// Key switching of count items on the matrix cores, in launches of at most
// KS_CHUNK gates; dig: device scratch of ks_digit_bytes(count) bytes;
// gates_per_block is the most gates a workgroup takes (128, 256 or 512, the
// last taken as 256, the largest tile), cus the device's CUs.
constexpr uint32_t KS_CHUNK = 16384;
constexpr size_t ks_digit_bytes(size_t count) { return (count < KS_CHUNK ? count : KS_CHUNK) * (RING_N * 2); }
int launch_ks_group(const KsSource& src, uint32_t count, const uint32_t* ksk, uint32_t* dig,
                    uint32_t gates_per_block, uint32_t cus, void* stream);
int launch_make_br_items(BrItem* items, uint32_t count, const uint32_t* a, const uint32_t* b, int32_t ca, int32_t cb,
                         uint32_t cst, uint32_t mu, uint32_t* out, const void* bk, void* stream);
int launch_negate(const uint32_t* a, uint32_t* out, size_t words, void* stream);

}  // namespace vlp
