// K3 of a layer and K1 of the next in one kernel, for narrow models (d = 128, 192, 256):
//   X <- X + (LayerNorm_d(O) * U) W2^T + b2,   [U V Q K] <- silu(X W1'^T + b1')
// on 64-row blocks: both act on rows alone, so a workgroup that has made a block's new residual rows can project them at once, from LDS.
//
// What it is for: launches of a few hundred row blocks, which are chains of short kernels.  Each of the two is 16 to 19 us there, of which about 5 are what any launch
// costs and several more its first memory latency, the tail of its last workgroups and (K1) reading the rows back that K3 has just written; the matrix work of both together is 3 us.
// Bound by step 4, whose SiLU (vector instructions) and products take two thirds of the time, and by its steps' latencies.  Step 4 has no barrier: each wavefront has columns and an
// output patch of its own, so that one's SiLU runs beside another's products (with pairs of wavefronts on 64 columns and two barriers a turn d = 256, 320 blocks 37.2 us, without 34.2).
// A launch lasts as long as the compute unit with the most rows, so the row blocks beyond whole rounds go as halves (whole_blocks below; 34.2 -> 29.3 us; d = 192, 384 blocks
// 30.3 -> 28.3 -> 24.3 us).
//
// Eight wavefronts, two workgroups on a compute unit:
//   1. LayerNorm and gate: a row per half wavefront (its 16 to 32 chunks of 16 bytes), eight rows per wavefront, all loads in flight together;
//   2. output projection: wavefront w owns features 32 w .. 32 w + 31 of all rows, W2's fragments from L2 through a register ring;
//   3. residual, through a patch per wavefront: Xh and Xl to memory, and Xh to LDS in the layout in which K1 reads it;
//   4. projection: a wavefront takes 32 columns at a time, W1's fragments from L2 through a register ring, SiLU, and a patch so that whole 64-byte pieces leave.
// Every output is made by the same instructions in the same order as by the two kernels (k3_mfma.hip, gemm_small_kernel in gemm_mfma.hip): bit for bit the same.
#include <type_traits>

#include "device_common.h"
#include "kernels.h"

namespace flame {

namespace {

// Sum over the 32 lanes of a half wavefront, delivered to all of them: wave_sum without its widest step.
__device__ __forceinline__ float half_sum(float v) {
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

constexpr int kPatchBytes = 8 * 4096;          // step 4: 64 rows x 32 columns per wavefront

template <int NK>
constexpr int layer_lds_bytes() { return (64 * 32 * NK * 2 > kPatchBytes ? 64 * 32 * NK * 2 : kPatchBytes) + 64 * 32 * NK * 2; }

// Step 4: [U V Q K] or [V K] of 32 NR rows from LDS (sX: [k / 32][row][32], swizzled), by strips of 32 columns, a wavefront each.  No barrier: the output patches at `patches`, 4 KB per
// wavefront, are the wavefronts' own, so that one's SiLU runs beside another's products.  The order of the strips: U, Q, K, and V last, whose products are the other way round.
// `ready`: the rows are there for everybody and the patches are free; it is called behind the first requests for W1.
template <int NK, int NR, typename Ready>
__device__ __forceinline__ void project_rows(const half_t *__restrict__ W1, const bf16_t *__restrict__ b1, const PlanePtrs &planes, bool all, int64_t ws_rows, int64_t row0, float alpha,
                                             const char *sX, char *patches, int wave, int lane, Ready ready) {
  constexpr int d = 32 * NK, KT = NR * 2048;           // KT: bytes of a k tile of sX
  constexpr int WD = NK < 4 ? NK : 4;                  // k tiles of W1 in flight
  const int l32 = lane & 31, lhalf = lane >> 5;
  const int n_strip = (all ? 4 : 2) * NK, n_rows = n_strip - NK;     // strips (all: U, V, Q and K, else V and K only), and those of the planes that are stored by rows
  char *pb = patches + wave * 4096;
  uint32_t woff = (uint32_t)lane * 16u;
  f16x8 fv[WD][2];
  f32x16 acc[NR];
  const char *wb = nullptr;
  int plane = 0, col = 0, k_rot = 0;
  auto kt_of = [&](int i) { const int k = i + k_rot; return k >= NK ? k - NK : k; };
  auto load_w = [&](int i) {
    asm volatile("" : "+v"(woff));
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) fv[i % WD][ks] = *(const f16x8 *)(wb + kt_of(i) * 2048 + ks * 1024 + woff);
  };
  auto start = [&](int strip) {                        // (past the last strip: that of the last, not used)
    const int h = strip < n_strip ? strip : n_strip - 1;
    const int i = h / NK;
    plane = h >= n_rows ? 1 : !all || i == 2 ? 3 : 2 * i;
    col = (h % NK) * 32;
    k_rot = ((plane * d + (col & ~63)) / (d % 128 == 0 ? 128 : 64)) % NK;   // as in the kernels of K1
    wb = (const char *)(W1 + (int64_t)(plane * d + col) * d);
#pragma unroll
    for (int p = 0; p < WD; ++p) load_w(p);
  };
  start(wave);
  ready();
  int strip = wave;
  auto columns = [&](auto fm_c) {
    constexpr bool FM = decltype(fm_c)::value;         // V is stored feature-major: the rows play operand A
    const int p_now = FM ? 1 : plane, c_now = col;
    const bf16_t *bp = b1 + p_now * d + c_now;
    if (!FM) {
      const bf16x8 b0v = *(const bf16x8 *)(bp + 16 * lhalf), b1v = *(const bf16x8 *)(bp + 16 * lhalf + 8);
#pragma unroll
      for (int i = 0; i < NR; ++i)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[i][e] = (float)(e < 8 ? b0v[e & 7] : b1v[e & 7]);
    } else {
      const float bf = to_f32(bp[l32]);
#pragma unroll
      for (int i = 0; i < NR; ++i)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[i][e] = bf;
    }
    const int ra = FM ? sigma32(l32) : l32;
    const int aoff[2] = {lds_off(ra, lhalf), lds_off(ra, 2 + lhalf)};
    f16x8 fa[2][2][NR];
    auto read_a = [&](int i) {
      int kb = kt_of(i) * KT;
      asm volatile("" : "+s"(kb));
      const char *t = sX + kb;
#pragma unroll
      for (int ks = 0; ks < 2; ++ks)
#pragma unroll
        for (int r = 0; r < NR; ++r) fa[i & 1][ks][r] = *(const f16x8 *)(t + aoff[ks] + r * 2048);
    };
    read_a(0);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < NK; ++i) {
      if (i + 1 < NK) read_a(i + 1);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int ks = 0; ks < 2; ++ks)
#pragma unroll
        for (int r = 0; r < NR; ++r)
          acc[r] = FM ? __builtin_amdgcn_mfma_f32_32x32x16_f16(fa[i & 1][ks][r], fv[i % WD][ks], acc[r], 0, 0, 0)
                      : __builtin_amdgcn_mfma_f32_32x32x16_f16(fv[i % WD][ks], fa[i & 1][ks][r], acc[r], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
      if (i + WD < NK) load_w(i + WD);
      __builtin_amdgcn_sched_barrier(0);
    }
    strip += 8;
    start(strip);                                      // the next columns' first fragments, under the epilogue
    __builtin_amdgcn_sched_barrier(0);
    // patch rows: the tokens, of 32 features, or 32 features, of the tokens
    constexpr int CPR = FM ? 4 * NR : 4, RPI = 64 / CPR;         // 16-byte chunks of a patch row, rows per store
    auto patch = [&](int row, int c) { return CPR == 8 ? row * 128 + ((c ^ ((row >> 1) & 7)) << 4) : lds_off(row, c); };
    auto to_patch = [&](auto scaled) {
      const float sc = alpha * 0.5f;
#pragma unroll
      for (int i = 0; i < NR; ++i)
#pragma unroll
        for (int g = 0; g < 2; ++g) {
          f16x8 o;
#pragma unroll
          for (int q = 0; q < 8; ++q) {
            const float w = silu_fast(acc[i][8 * g + q]);
            o[q] = to_f16_sat(decltype(scaled)::value ? w * sc : w);
          }
          *(f16x8 *)(pb + (FM ? patch(l32, 4 * i + 2 * lhalf + g) : patch(32 * i + l32, 2 * lhalf + g))) = o;
        }
    };
    if (!FM && p_now == 2) to_patch(std::true_type{});
    else to_patch(std::false_type{});
    half_t *P = (half_t *)(FM ? planes.v : p_now == 0 ? planes.u : p_now == 2 ? planes.q : planes.k);
    const int rl4 = lane / CPR, c = lane % CPR;
    const int64_t pitch = (FM ? ws_rows : (int64_t)d) * 2;       // bytes from one patch row to the next: a feature's tokens, or a token's features
    char *dst = (char *)(FM ? P + c_now * ws_rows + row0 : P + row0 * d + c_now);
    uint32_t doff = (uint32_t)(rl4 * pitch) + c * 16u;
    asm volatile("" : "+v"(doff));
#pragma unroll
    for (int it = 0; it < 2 * NR; ++it) *(f16x8 *)(dst + it * RPI * pitch + doff) = *(const f16x8 *)(pb + patch(rl4 + RPI * it, c));
  };
  while (strip < n_rows) columns(std::false_type{});
  while (strip < n_strip) columns(std::true_type{});
}

// NK = d / 32; NR = groups of 32 rows: a whole row block or half of one, the rows from 32 * part on.
// (U is the plane that planes.u overwrites, each workgroup its own rows, which it has read in step 1.)
template <int NK, int NR>
__device__ __forceinline__ void layer_body(const half_t *__restrict__ O, const half_t *U, const bf16_t *__restrict__ gamma, const bf16_t *__restrict__ beta,
                                           const half_t *__restrict__ W2p, const bf16_t *__restrict__ b2, half_t *__restrict__ Xh, half_t *__restrict__ Xl, int lo_is_zero,
                                           const RowBlock rb, int blk, int part, float eps, const half_t *__restrict__ W1, const bf16_t *__restrict__ b1,
                                           const PlanePtrs planes, int all_hist, int all_cand, int64_t ws_rows, float alpha, char *smem) {
  constexpr int d = 32 * NK, NCHUNK = d / 8, NKS = d / 16;
  constexpr int R1 = NR * 64 * d > kPatchBytes ? NR * 64 * d : kPatchBytes;
  char *const sX = smem + R1;                        // gated rows, then patches; behind them the new rows, [k / 32][row][32]
  constexpr int KT = NR * 2048;                      // bytes of a k tile of sX
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, lhalf = lane >> 5;
  const int64_t row0 = (int64_t)blk * kRowAlign + 32 * part;

  // ---- 1: G = (LN(O) * gamma + beta) * U -> LDS (swizzle of k3_mfma.hip)
  auto gkey = [](int r) { return NCHUNK % 16 == 0 ? r & 15 : (r >> 1) & 7; };
  const bool in_row = l32 < NCHUNK;
  const int ch = in_row ? l32 : NCHUNK - 1;
  // (Addresses are a wave-uniform base plus a 32-bit lane offset throughout; the empty asm keeps the compiler from making 64-bit vector addresses of them.)
  constexpr int NQ = 2 * NR;                         // row pairs of a wavefront, and 16-row groups of the block
  f16x8 ov[NQ], uv[NQ];
  {
    const char *ob = (const char *)(O + row0 * d), *ub = (const char *)(U + row0 * d);
    uint32_t off = (uint32_t)((wave * 2 * NQ + lhalf) * d + ch * 8) * 2u;
    asm volatile("" : "+v"(off));
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      ov[q] = *(const f16x8 *)(ob + q * 4 * d + off);
      uv[q] = *(const f16x8 *)(ub + q * 4 * d + off);
    }
  }
  const bf16x8 gv = *(const bf16x8 *)(gamma + ch * 8), bv = *(const bf16x8 *)(beta + ch * 8);
  // what does not depend on step 1 is requested ahead of it: the first fragments of W2
  constexpr int PD = 8;
  const bool proj = wave < NK;                       // this wavefront's feature block exists
  const int fb = proj ? wave : NK - 1;
  const char *wp = (const char *)(W2p + (int64_t)fb * 512);     // + ks * NK * 1024 + 16 lane
  uint32_t woff = (uint32_t)lane * 16u;
  f16x8 fw[PD];
  asm volatile("" : "+v"(woff));
#pragma unroll
  for (int p = 0; p < PD - 1; ++p) fw[p] = *(const f16x8 *)(wp + p * NK * 1024 + woff);
  __builtin_amdgcn_sched_barrier(0);
  {
    float v[NQ][8], mu[NQ], rstd[NQ];
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      float sum = 0.f;
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        v[q][k] = in_row ? (float)ov[q][k] : 0.f;
        sum += v[q][k];
      }
      mu[q] = sum;
    }
#pragma unroll
    for (int q = 0; q < NQ; ++q) mu[q] = half_sum(mu[q]) * (1.0f / d);
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      float sq = 0.f;
      if (in_row) {
#pragma unroll
        for (int k = 0; k < 8; ++k) { const float t = v[q][k] - mu[q]; sq += t * t; }
      }
      rstd[q] = sq;
    }
#pragma unroll
    for (int q = 0; q < NQ; ++q) rstd[q] = rsqrtf(half_sum(rstd[q]) * (1.0f / d) + eps);
    if (in_row) {
#pragma unroll
      for (int q = 0; q < NQ; ++q) {
        const int r = wave * 2 * NQ + 2 * q + lhalf;
        const bool pad = 32 * part + r >= rb.n_valid;              // padding rows carry a zero branch so that they stay finite
        f16x8 o;
#pragma unroll
        for (int k = 0; k < 8; ++k) o[k] = to_f16_sat(((v[q][k] - mu[q]) * rstd[q] * (float)gv[k] + (float)bv[k]) * (float)uv[q][k]);
        asm volatile("" : "+v"(o));                    // (keeps the select a select: a branch around every element is what the compiler makes of it otherwise)
#pragma unroll
        for (int k = 0; k < 8; ++k) o[k] = pad ? (half_t)0.f : o[k];
        *(f16x8 *)(smem + r * (d * 2) + ((ch ^ gkey(r)) << 4)) = o;
      }
    }
  }
  __syncthreads();

  // ---- 2 (the residual rows are requested behind W2's last fragments)
  const int rl = lane >> 2, cc = lane & 3, n = fb * 32 + 8 * cc;   // step 3: rows rl + 16 it of 32, eight features n ..
  f16x8 xh[NQ], xl[NQ];
  char *const xhb = (char *)(Xh + (int64_t)blk * kRowAlign * d + fb * 2048 + part * 1024), *const xlb = (char *)(Xl + row0 * d + fb * 32);     // the block's slice of Xh, k-tile blocked, and of Xl
  uint32_t xho = (uint32_t)(rl * 32 + 8 * cc) * 2u, xlo = (uint32_t)(rl * d + 8 * cc) * 2u;
  auto load_x = [&](int t) {
    asm volatile("" : "+v"(xho), "+v"(xlo));
    xh[t] = *(const f16x8 *)(xhb + t * 1024 + xho);
    xl[t] = *(const f16x8 *)(xlb + t * 32 * d + xlo);           // (not used in the first layer, whose input rows are exact in Xh)
  };
  f32x16 acc[NR];
#pragma unroll
  for (int i = 0; i < NR; ++i)
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[i][e] = 0.f;
  if (proj) {
    f16x8 fa[2][NR];
    auto read_g = [&](int set, int ks) {
#pragma unroll
      for (int i = 0; i < NR; ++i) {
        const int r = 32 * i + l32;
        fa[set][i] = *(const f16x8 *)(smem + r * (d * 2) + (((2 * ks + lhalf) ^ gkey(r)) << 4));
      }
    };
    read_g(0, 0);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks) {
      asm volatile("" : "+v"(woff));
      if (ks + PD - 1 < NKS) fw[(ks + PD - 1) % PD] = *(const f16x8 *)(wp + (ks + PD - 1) * NK * 1024 + woff);
      else if (ks + PD - 1 < NKS + NQ) load_x(ks + PD - 1 - NKS);
      if (ks + 1 < NKS) read_g((ks + 1) & 1, ks + 1);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = 0; i < NR; ++i) acc[i] = __builtin_amdgcn_mfma_f32_32x32x16_f16(fw[ks % PD], fa[ks & 1][i], acc[i], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  __syncthreads();                                     // everybody has read G

  // ---- 3
  if (proj) {
    char *pb = smem + wave * 4096;                     // 32 rows x 32 features, fp32, 16-byte chunks XOR-swizzled by row
    auto pkey = [](int row) { return (row >> 1) & 7; };
    const bf16x8 bvw = *(const bf16x8 *)(b2 + n);
    if (lo_is_zero) {
#pragma unroll
      for (int t = 0; t < NQ; ++t)
#pragma unroll
        for (int q = 0; q < 8; ++q) xl[t][q] = (half_t)0.f;
    }
#pragma unroll
    for (int i = 0; i < NR; ++i) {
#pragma unroll
      for (int gq = 0; gq < 4; ++gq) {
        const int c = 2 * gq + lhalf;
        const f32x4 v = {acc[i][4 * gq], acc[i][4 * gq + 1], acc[i][4 * gq + 2], acc[i][4 * gq + 3]};
        *(f32x4 *)(pb + l32 * 128 + ((c ^ pkey(l32)) << 4)) = v;
      }
#pragma unroll
      for (int it = 0; it < 2; ++it) {
        const int row = 16 * it + rl, t = 2 * i + it;
        f16x8 oh, ol;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const f32x4 v = *(const f32x4 *)(pb + row * 128 + (((2 * cc + h) ^ pkey(row)) << 4));
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const float x = ((float)xh[t][4 * h + q] + (float)xl[t][4 * h + q]) + (v[q] + (float)bvw[4 * h + q]);
            oh[4 * h + q] = to_f16_sat(x);
            ol[4 * h + q] = to_f16_sat(x - (float)oh[4 * h + q]);
          }
        }
        *(f16x8 *)(xhb + t * 1024 + xho) = oh;
        *(f16x8 *)(xlb + t * 32 * d + xlo) = ol;
        *(f16x8 *)(sX + fb * KT + lds_off(32 * i + row, cc)) = oh;
      }
    }
  }
  // ---- 4
  project_rows<NK, NR>(W1, b1, planes, rb.kind ? all_cand : all_hist, ws_rows, row0, alpha, sX, smem, wave, lane, []() { __syncthreads(); });
}

// The first n_whole workgroups take a row block each, those behind them half of one.
template <int NK>
__global__ __launch_bounds__(512, 4) void layer_kernel(const half_t *__restrict__ O, const half_t *U, const bf16_t *__restrict__ gamma, const bf16_t *__restrict__ beta,
                                                       const half_t *__restrict__ W2p, const bf16_t *__restrict__ b2, half_t *__restrict__ Xh, half_t *__restrict__ Xl, int lo_is_zero,
                                                       const RowBlock *__restrict__ blocks, const int32_t *__restrict__ blk_list, int blk_first, float eps,
                                                       const half_t *__restrict__ W1, const bf16_t *__restrict__ b1, PlanePtrs planes, int all_hist, int all_cand, int64_t ws_rows,
                                                       float alpha, int n_whole) {
  extern __shared__ __attribute__((aligned(256))) char smem[];
  const int i = blockIdx.x, h = i - n_whole, item = h < 0 ? i : n_whole + (h >> 1);
  const int blk = blk_list ? blk_list[item] : blk_first + item;
  if (h < 0) layer_body<NK, 2>(O, U, gamma, beta, W2p, b2, Xh, Xl, lo_is_zero, blocks[blk], blk, 0, eps, W1, b1, planes, all_hist, all_cand, ws_rows, alpha, smem);
  else layer_body<NK, 1>(O, U, gamma, beta, W2p, b2, Xh, Xl, lo_is_zero, blocks[blk], blk, h & 1, eps, W1, b1, planes, all_hist, all_cand, ws_rows, alpha, smem);
}

}  // namespace

// At every size of d = 128, 192 and 256: forwards of 4 layers on two kernels a layer / on this one (us), by 64-row blocks (the two kernels stream past 1024, 682 and 512 of them):
//   d = 128: 5: 86 / 72, 100: 104 / 86, 320: 150 / 119, 1025: 324 / 268, 1140: 347 / 282, 1278: 372 / 309, 8200: 1821 / 1688;
//   d = 192: 5: 96 / 81, 130: 149 / 127, 510: 262 / 205, 684: 333 / 274, 768: 350 / 287, 852: 398 / 336, 2050: 790 / 710;
//   d = 256: 5: 90 / 87, 65: 124 / 113, 160: 147 / 136, 510: 302 / 267, 561: 356 / 305, 639: 384 / 325, 1025: 589 / 515, 8200: 3735 / 3661.
// (Stores and loads past the caches make it slower in launches that stream, too: d = 192, 1280 blocks 454 -> 480 us, d = 256, 640 blocks 330 -> 342.)
bool layer_fused(int d) { return d == 128 || d == 192 || d == 256; }

// Row blocks that a workgroup takes whole; each of the others is two workgroups of half of it.  Beyond a multiple of the compute units, blocks that fit them as halves, one each, go
// as halves: the most rows on a compute unit are then half a block fewer.  (Twice the traffic of weights for those; more of them would not shorten the longest.)
static int whole_blocks(int n_blk) {
  constexpr int kUnits = 256;
  const int rest = n_blk % kUnits;
  return 2 * rest <= kUnits ? n_blk - rest : n_blk;
}

template <int NK>
static hipError_t layer_limit() {
  static std::atomic<uint64_t> done{0};
  return raise_lds_limit(reinterpret_cast<const void *>(&layer_kernel<NK>), layer_lds_bytes<NK>(), done);
}

hipError_t layer_setup(int d) { return d == 128 ? layer_limit<4>() : d == 192 ? layer_limit<6>() : d == 256 ? layer_limit<8>() : hipSuccess; }

void launch_layer(const void *O, const void *U, const void *gamma, const void *beta, const void *W2p_layer, const void *b2, void *Xh, void *Xl, bool lo_is_zero,
                  const RowBlock *blocks, const int32_t *blk_list, int n_blk, int blk_first, const void *W1h_next, const void *b1_next, PlanePtrs planes, bool all_hist, bool all_cand,
                  const Shape &sh, hipStream_t s) {
  if (n_blk <= 0) return;
  const int n_whole = whole_blocks(n_blk);
#define LAYER_CASE(NK) layer_kernel<NK><<<n_whole + 2 * (n_blk - n_whole), 512, layer_lds_bytes<NK>(), s>>>((const half_t *)O, (const half_t *)U, (const bf16_t *)gamma, \
    (const bf16_t *)beta, (const half_t *)W2p_layer, (const bf16_t *)b2, (half_t *)Xh, (half_t *)Xl, lo_is_zero ? 1 : 0, blocks, blk_list, blk_first, sh.eps, \
    (const half_t *)W1h_next, (const bf16_t *)b1_next, planes, all_hist ? 1 : 0, all_cand ? 1 : 0, sh.ws_rows, sh.alpha, n_whole)
  if (sh.d == 128) LAYER_CASE(4);
  else if (sh.d == 192) LAYER_CASE(6);
  else LAYER_CASE(8);
#undef LAYER_CASE
}

}  // namespace flame
