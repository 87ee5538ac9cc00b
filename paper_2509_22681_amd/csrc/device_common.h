// Device-side helpers shared by the gfx950 kernels of the GR forward.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace flame {

typedef __bf16 bf16_t;
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef _Float16 half_t;
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x4 __attribute__((ext_vector_type(4)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kWave = 64;

__device__ __forceinline__ float to_f32(float v) { return v; }
__device__ __forceinline__ float to_f32(bf16_t v) { return (float)v; }
__device__ __forceinline__ float to_f32(half_t v) { return (float)v; }

// fp16 storage of an fp32 value: round to nearest even, saturating at the largest finite fp16 so
// that an out-of-range activation degrades gracefully instead of turning into inf (and then NaN).
__device__ __forceinline__ half_t to_f16_sat(float v) {
  return (half_t)__builtin_fminf(__builtin_fmaxf(v, -65504.f), 65504.f);
}

template <typename T> __device__ __forceinline__ T from_f32(float v);
template <> __device__ __forceinline__ float from_f32<float>(float v) { return v; }
template <> __device__ __forceinline__ bf16_t from_f32<bf16_t>(float v) { return (bf16_t)v; }  // round to nearest even
template <> __device__ __forceinline__ half_t from_f32<half_t>(float v) { return to_f16_sat(v); }

// silu(x) = x / (1 + exp(-x)) by the hardware's exp2 and reciprocal (about 1 ulp each).  exp2 of a large positive argument gives +inf and the
// result 0, of a large negative one gives 0 and the result x: both limits are the right ones.
__device__ __forceinline__ float silu_fast(float x) {
  float e = __builtin_amdgcn_exp2f(x * -1.4426950408889634f);
  return x * __builtin_amdgcn_rcpf(1.0f + e);
}

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;

// SiLU of an argument that arrives halved: returns silu(x) for s = x / 2.  The attention kernel keeps
// its logits in this form (the factor 1/2 is folded into Q and into the bias table, both exactly):
// silu(x) = x/2 + x^2 r(x^2) then starts from the logit itself, see the polynomial route there.
__device__ __forceinline__ float silu_half_domain(float s) {
  // x / (1 + e^-x) = s / (1/2 + 2^(-2 log2(e) s - 1)): fma, exp2, add, rcp, mul
  return s * __builtin_amdgcn_rcpf(0.5f + __builtin_amdgcn_exp2f(__builtin_fmaf(s, -2.0f * kLog2e, -1.0f)));
}

// SiLU for small arguments.  silu(x) - x/2 is even: silu(x) = x/2 + x^2 r(x^2) with r(u) ~ a1 + a3 u + a5 u^2 (weighted
// least-squares fit of (silu(x) - x/2) / x^2 on [-2, 2]; approximation error 5.3e-4 at |x| = 2, below 2.1e-4 for
// |x| <= 1.5, below 1.3e-4 for |x| <= 1 and below 4.7e-5 for |x| <= 1/4).
constexpr float kPolyA1 = 0.24916259f, kPolyA3 = -0.01916112f, kPolyA5 = 0.00112581f;

// "k-tile blocked" layout of the fp16 activation copy Xh, the projection's operand: inside every block of 64 rows the 32-wide k slices follow one another,
// [row / 64][k / 32][row % 64][k % 32], so the 64 rows x 32 k slice a GEMM k-tile needs is 4 KB of
// contiguous memory and is fetched as whole 128-byte lines.  (Row-major rows of d elements would hand
// the L1 two 64-byte requests per line, and the number of requests in flight is what bounds it.)
__device__ __forceinline__ int64_t blocked_index(int64_t row, int k, int K) {
  return (row >> 6) * 64 * K + (int64_t)(k >> 5) * 2048 + (row & 63) * 32 + (k & 31);
}

// Row order of the MFMA A operand.  Accumulator element e of lane (l32, lhalf) belongs to A-operand
// row 8*(e/4) + 4*lhalf + e%4.  Feeding tile row sigma32(m) = 16*bit2(m) + 4*(m/8) + m%4 into A-operand
// row m turns that into tile row 16*lhalf + e: a lane then owns 16 consecutive outputs (features of
// one token, or tokens of one feature for the feature-major plane) and stores them as two 16-byte
// words, two lanes covering a contiguous 64 bytes.
__device__ __forceinline__ int sigma32(int m) { return ((m & 4) << 2) | ((m >> 3) << 2) | (m & 3); }

// LDS layout of the activations' operand tiles: 64 bytes (32 k) per row.
// byte offset of 16-byte chunk c (0..3) of tile row `row` inside one LDS operand.  Four 64-byte rows share a 256-byte
// group: row bits 0..1 pick the quarter, and the chunk index is XORed with row bits 2..3.  The LDS serves 256 bytes
// = 16 lanes x 16 bytes per clock from 64 banks, and the 16 lanes of a ds_read_b128 that it serves together are not
// 16 consecutive ones: measured on this chip (chip_microbench, the four ds_read_b128 lines), lanes {0-3, 12-15, 20-23,
// 24-27} go together, then {4-7, 8-11, 16-19, 28-31}, and likewise in the upper half of the wavefront.  With this key
// both fragment row orders used below (identity, and sigma32: lane m reads row 16 bit2(m) + 4 (m / 8) + m % 4) put
// the four quads of such a group into four different key values, i.e. 16 different slots: 240 and 225 bytes per clock
// and CU.  (A key with row bit 3 ^ bit 4 in place of bit 3, which is free of conflicts for 16 consecutive lanes,
// measured 127.)
__device__ __forceinline__ int lds_key(int row) { return (row >> 2) & 3; }
__device__ __forceinline__ int lds_off(int row, int c) {
  return (row >> 2) * 256 + ((((row & 3) << 2) | (c ^ lds_key(row))) << 4);
}

// Loads and stores of data that is consumed once, past the caches or (NT = false) through them.
template <bool NT, typename T> __device__ __forceinline__ T load_once(const T *p) {
  if constexpr (NT) return __builtin_nontemporal_load(p);
  else return *p;
}
template <bool NT, typename T> __device__ __forceinline__ void store_once(T v, T *p) {
  if constexpr (NT) __builtin_nontemporal_store(v, p);
  else *p = v;
}

// Layout of the converted projection matrices: MFMA fragments of 32 rows x 16 k, [row / 32][k / 16][lane][8], 1 KB each; lane l holds
// k 8 (l / 32) + 0..7 of row l & 31, or of row sigma32(l & 31) where the rows play operand A.  A fragment is one contiguous
// request, from LDS (free of bank conflicts without a swizzle) as well as from L2 straight into registers.

// An fp32 value as the sum of three bf16 values: each takes the next eight bits (round to nearest, the remainder is exact in fp32), and 8 + 8 + 8
// bits with signs hold the 24 of the mantissa.  Exact for all finite values but those below 2^-110, whose lower parts fall under the range of normal numbers and may be flushed
// (off by less than 2^-125).
// The first two parts end at bf16's largest value, so that what rounds past it leaves a finite remainder, and an infinity (or a NaN) comes out in the last part:
// in the products it then meets the other operand's first part alone, which has that operand's sign.
struct Split3 { bf16x4 p[3]; };
__device__ __forceinline__ Split3 split3(f32x4 v) {
  typedef float f32x2 __attribute__((ext_vector_type(2)));
  constexpr float kBf16Max = 0x1.fep127f;
  Split3 s;
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    f32x2 x = {v[2 * h], v[2 * h + 1]};
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      f32x2 c = x;
      if (i < 2) c = f32x2{__builtin_amdgcn_fmed3f(x[0], -kBf16Max, kBf16Max), __builtin_amdgcn_fmed3f(x[1], -kBf16Max, kBf16Max)};
      const bf16x2 b = __builtin_convertvector(c, bf16x2);       // two values per instruction
      s.p[i][2 * h] = b[0];
      s.p[i][2 * h + 1] = b[1];
      if (i < 2) { x[0] -= (float)b[0]; x[1] -= (float)b[1]; }
    }
  }
  return s;
}

// Number of history keys a query row may look at (the mask of the single-user-multiple-items
// scoring pass): a history row at index q sees keys 0..q, a candidate row sees all L.
__device__ __forceinline__ int visible_history(int is_cand, int q_index, int L) {
  return is_cand ? L : q_index + 1;
}

// Sum over the 64 lanes, delivered to every lane: the butterfly v += v[lane ^ o] for o = 32, 16, 8, 4, 2, 1,
// without the LDS crossbar.  The two widest steps use the half- and row-swap instructions of gfx950 (each
// returns both halves of the exchange, whose sum is the butterfly step in either half); the others are DPP
// operands of the add.  After the step for o, lanes that differ only in bits >= o hold equal values, so a row
// rotation by 4 (resp. 2) reaches a lane that holds exactly what lane ^ 4 (resp. lane ^ 2) holds: every lane
// gets the bits the plain butterfly would give.
__device__ __forceinline__ float wave_sum(float v) {
  {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = __uint_as_float(r[0]) + __uint_as_float(r[1]);
  }
  {
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = __uint_as_float(r[0]) + __uint_as_float(r[1]);
  }
  v += __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(v), 0x128, 0xf, 0xf, false));  // row_ror:8
  v += __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(v), 0x124, 0xf, 0xf, false));  // row_ror:4
  v += __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(v), 0x4e, 0xf, 0xf, false));   // quad_perm 2,3,0,1
  v += __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(v), 0xb1, 0xf, 0xf, false));   // quad_perm 1,0,3,2
  return v;
}

// Exchange between the two lanes that share a query column of a 32x32 accumulator block (lane and lane ^ 32):
// both get the maximum, resp. the sum, of their two values.
__device__ __forceinline__ float pair_max(float v) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float pair_sum(float v) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

}  // namespace flame
