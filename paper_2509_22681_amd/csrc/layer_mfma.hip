// K3 of a layer and K1 of the next in one kernel, for narrow models (d = 128, 192, 256) in launches that do not stream:
//   X <- X + (LayerNorm_d(O) * U) W2^T + b2,   [U V Q K] <- silu(X W1'^T + b1')
// on 64-row blocks: both act on rows alone, so a workgroup that has made a block's new residual rows can project them at once, from LDS.
//
// What it is for: launches of a few hundred row blocks, which are chains of short kernels.  Each of the two is 16 to 19 us there, of which about 5 are what any launch
// costs and several more its first memory latency, the tail of its last workgroups and (K1) reading the rows back that K3 has just written; the matrix work of both together is 3 us.
// Measured, K3 + K1 of a layer -> one launch: d = 256, 320 blocks 36 -> 36 to 37 us and a launch less, d = 192, 320 blocks 35 -> 28 to 29; the forward 226 -> 217 and 1311 -> 1125 us.
// Bound by its steps' latencies: of 39 thousand cycles per workgroup 7 go to step 1, 4 to step 2, 5 to step 3, 19 to step 4 (8 of them its products) and the rest to barriers.
//
// Eight wavefronts, two workgroups on a compute unit:
//   1. LayerNorm and gate: a row per half wavefront (its 16 to 32 chunks of 16 bytes), eight rows per wavefront, all loads in flight together;
//   2. output projection: wavefront w owns features 32 w .. 32 w + 31 of all 64 rows, W2's fragments from L2 through a register ring;
//   3. residual, through a patch per wavefront: Xh and Xl to memory, and Xh to LDS in the layout in which K1 reads it;
//   4. projection: a pair of wavefronts takes 64 columns at a time, W1's fragments from L2 through a register ring, SiLU, and a patch per pair so that whole lines leave.
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

constexpr int kPatchBytes = 4 * 8192;          // step 4: 64 rows x 64 columns per pair of wavefronts

template <int NK>
constexpr int layer_lds_bytes() { return (64 * 32 * NK * 2 > kPatchBytes ? 64 * 32 * NK * 2 : kPatchBytes) + 64 * 32 * NK * 2; }

// NK = d / 32.  (U is the plane that planes.u overwrites, each workgroup its own rows, which it has read in step 1: no __restrict__.)
template <int NK>
__global__ __launch_bounds__(512, 4) void layer_kernel(const half_t *__restrict__ O, const half_t *U, const bf16_t *__restrict__ gamma, const bf16_t *__restrict__ beta,
                                                       const half_t *__restrict__ W2p, const bf16_t *__restrict__ b2, half_t *__restrict__ Xh, half_t *__restrict__ Xl, int lo_is_zero,
                                                       const RowBlock *__restrict__ blocks, const int32_t *__restrict__ blk_list, int blk_first, float eps,
                                                       const half_t *__restrict__ W1, const bf16_t *__restrict__ b1, PlanePtrs planes, int all_hist, int all_cand, int64_t ws_rows,
                                                       float alpha) {
  constexpr int d = 32 * NK, NCHUNK = d / 8, NKS = d / 16;
  constexpr int R1 = 64 * d * 2 > kPatchBytes ? 64 * d * 2 : kPatchBytes;
  extern __shared__ __attribute__((aligned(256))) char smem[];     // gated rows, then patches; behind them the new rows
  char *const sX = smem + R1;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, lhalf = lane >> 5;
  const int blk = blk_list ? blk_list[blockIdx.x] : blk_first + blockIdx.x;
  const RowBlock rb = blocks[blk];
  const int64_t row0 = (int64_t)blk * kRowAlign;

  // ---- 1: G = (LN(O) * gamma + beta) * U -> LDS (swizzle of k3_mfma.hip)
  auto gkey = [](int r) { return NCHUNK % 16 == 0 ? r & 15 : (r >> 1) & 7; };
  const bool in_row = l32 < NCHUNK;
  const int ch = in_row ? l32 : NCHUNK - 1;
  // (Addresses are a wave-uniform base plus a 32-bit lane offset throughout; the empty asm keeps the compiler from making 64-bit vector addresses of them.)
  f16x8 ov[4], uv[4];
  {
    const char *ob = (const char *)(O + row0 * d), *ub = (const char *)(U + row0 * d);
    uint32_t off = (uint32_t)((wave * 8 + lhalf) * d + ch * 8) * 2u;
    asm volatile("" : "+v"(off));
#pragma unroll
    for (int q = 0; q < 4; ++q) {
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
    float v[4][8], mu[4], rstd[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      float sum = 0.f;
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        v[q][k] = in_row ? (float)ov[q][k] : 0.f;
        sum += v[q][k];
      }
      mu[q] = sum;
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) mu[q] = half_sum(mu[q]) * (1.0f / d);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      float sq = 0.f;
      if (in_row) {
#pragma unroll
        for (int k = 0; k < 8; ++k) { const float t = v[q][k] - mu[q]; sq += t * t; }
      }
      rstd[q] = sq;
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) rstd[q] = rsqrtf(half_sum(rstd[q]) * (1.0f / d) + eps);
    if (in_row) {
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int r = wave * 8 + 2 * q + lhalf;
        const bool pad = r >= rb.n_valid;              // padding rows carry a zero branch so that they stay finite
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
  f16x8 xh[4], xl[4];
  char *const xhb = (char *)(Xh + row0 * d + fb * 2048), *const xlb = (char *)(Xl + row0 * d + fb * 32);     // the block's slice of Xh, k-tile blocked, and of Xl
  uint32_t xho = (uint32_t)(rl * 32 + 8 * cc) * 2u, xlo = (uint32_t)(rl * d + 8 * cc) * 2u;
  auto load_x = [&](int t) {
    asm volatile("" : "+v"(xho), "+v"(xlo));
    xh[t] = *(const f16x8 *)(xhb + t * 1024 + xho);
    xl[t] = *(const f16x8 *)(xlb + t * 32 * d + xlo);           // (not used in the first layer, whose input rows are exact in Xh)
  };
  f32x16 acc[2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[i][e] = 0.f;
  if (proj) {
    f16x8 fa[2][2];
    auto read_g = [&](int set, int ks) {
#pragma unroll
      for (int i = 0; i < 2; ++i) {
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
      else if (ks + PD - 1 < NKS + 4) load_x(ks + PD - 1 - NKS);
      if (ks + 1 < NKS) read_g((ks + 1) & 1, ks + 1);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = 0; i < 2; ++i) acc[i] = __builtin_amdgcn_mfma_f32_32x32x16_f16(fw[ks % PD], fa[ks & 1][i], acc[i], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  __syncthreads();                                     // everybody has read G

  // ---- 4, its first requests: W1's fragments of the first columns.  Columns of 64 (a "half" of the tile in gemm_small_kernel) over the planes that the block needs
  const int pair = wave >> 1;
  const bool all = rb.kind ? all_cand : all_hist;      // U, V, Q and K, or V and K only
  constexpr int CPP = d / 64;                          // halves per plane
  const int n_half = (all ? 4 : 2) * CPP;
  constexpr int WD = NK < 4 ? NK : 4;                  // k tiles of W1 in flight
  f16x8 fv[WD][2];
  const char *wb = nullptr;
  int plane = 0, col = 0, k_rot = 0;
  auto kt_of = [&](int i) { const int k = i + k_rot; return k >= NK ? k - NK : k; };
  auto load_w = [&](int i) {
    asm volatile("" : "+v"(woff));
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) fv[i % WD][ks] = *(const f16x8 *)(wb + kt_of(i) * 2048 + ks * 1024 + woff);
  };
  // in order: U, Q, K, and V last, whose products are the other way round
  const int n_rows = n_half - CPP;                     // halves of the planes that are stored by rows
  auto start = [&](int half) {                         // (past the last half: that of the last, not used)
    const int h = half < n_half ? half : n_half - 1;
    const int i = h / CPP;
    plane = h >= n_rows ? 1 : !all || i == 2 ? 3 : 2 * i;
    col = (h % CPP) * 64;
    k_rot = ((plane * d + col) / (d % 128 == 0 ? 128 : 64)) % NK;   // as in the kernels of K1
    wb = (const char *)(W1 + ((int64_t)(plane * d + col) / 32 + (wave & 1)) * 32 * d);
#pragma unroll
    for (int p = 0; p < WD; ++p) load_w(p);
  };

  // ---- 3
  if (proj) {
    char *pb = smem + wave * 4096;                     // 32 rows x 32 features, fp32, 16-byte chunks XOR-swizzled by row
    auto pkey = [](int row) { return (row >> 1) & 7; };
    const bf16x8 bvw = *(const bf16x8 *)(b2 + n);
    if (lo_is_zero) {
#pragma unroll
      for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int q = 0; q < 8; ++q) xl[t][q] = (half_t)0.f;
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) {
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
        *(f16x8 *)(sX + fb * 4096 + lds_off(32 * i + row, cc)) = oh;
      }
    }
  }
  start(pair);
  __syncthreads();                                     // the new rows are complete, and everybody has left the patches

  // ---- 4
  char *pb = smem + pair * 8192;
  int half = pair;
  auto columns = [&](auto fm_c) {
    constexpr bool FM = decltype(fm_c)::value;         // V is stored feature-major: the rows play operand A
    const int p_now = FM ? 1 : plane, c_now = col;
    const bf16_t *bp = b1 + p_now * d + c_now + (wave & 1) * 32;
    if (!FM) {
      const bf16x8 b0v = *(const bf16x8 *)(bp + 16 * lhalf), b1v = *(const bf16x8 *)(bp + 16 * lhalf + 8);
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[i][e] = (float)(e < 8 ? b0v[e & 7] : b1v[e & 7]);
    } else {
      const float bf = to_f32(bp[l32]);
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[i][e] = bf;
    }
    const int ra = FM ? sigma32(l32) : l32;
    const int aoff[2] = {lds_off(ra, lhalf), lds_off(ra, 2 + lhalf)};
    f16x8 fa[2][2][2];
    auto read_a = [&](int i) {
      int kb = kt_of(i) * 4096;
      asm volatile("" : "+s"(kb));
      const char *t = sX + kb;
#pragma unroll
      for (int ks = 0; ks < 2; ++ks)
#pragma unroll
        for (int r = 0; r < 2; ++r) fa[i & 1][ks][r] = *(const f16x8 *)(t + aoff[ks] + r * 2048);
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
        for (int r = 0; r < 2; ++r)
          acc[r] = FM ? __builtin_amdgcn_mfma_f32_32x32x16_f16(fa[i & 1][ks][r], fv[i % WD][ks], acc[r], 0, 0, 0)
                      : __builtin_amdgcn_mfma_f32_32x32x16_f16(fv[i % WD][ks], fa[i & 1][ks][r], acc[r], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
      if (i + WD < NK) load_w(i + WD);
      __builtin_amdgcn_sched_barrier(0);
    }
    half += 4;
    start(half);                                       // the next columns' first fragments (as built, under the epilogue for V; for U, Q and K the compiler moves them behind its barrier)
    __builtin_amdgcn_sched_barrier(0);
    const float sc = alpha * 0.5f;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int g = 0; g < 2; ++g) {
        f16x8 o;
#pragma unroll
        for (int q = 0; q < 8; ++q) {
          const float w = silu_fast(acc[i][8 * g + q]);
          o[q] = to_f16_sat(!FM && p_now == 2 ? w * sc : w);
        }
        const int row = FM ? (wave & 1) * 32 + l32 : 32 * i + l32;
        const int c = FM ? 4 * i + 2 * lhalf + g : 4 * (wave & 1) + 2 * lhalf + g;
        *(f16x8 *)(pb + row * 128 + ((c ^ ((row >> 1) & 7)) << 4)) = o;
      }
    __syncthreads();
    half_t *P = (half_t *)(FM ? planes.v : p_now == 0 ? planes.u : p_now == 2 ? planes.q : planes.k);
    const int ht = tid & 127, c = ht & 7;
    const int64_t pitch = (FM ? ws_rows : (int64_t)d) * 2;       // bytes from one patch row to the next: a feature's tokens, or a token's features
    char *dst = (char *)(FM ? P + c_now * ws_rows + row0 : P + row0 * d + c_now);
    uint32_t doff = (uint32_t)((ht >> 3) * pitch) + c * 16u;
    asm volatile("" : "+v"(doff));
#pragma unroll
    for (int it = 0; it < 4; ++it) {
      const int r = (ht >> 3) + 16 * it;
      const f16x8 v = *(const f16x8 *)(pb + r * 128 + ((c ^ ((r >> 1) & 7)) << 4));
      *(f16x8 *)(dst + it * 16 * pitch + doff) = v;
    }
    __syncthreads();
  };
  // every pair takes the same number of turns, that is of barriers
  while (half < n_rows) columns(std::false_type{});
  while (half < n_half) columns(std::true_type{});
  for (; half - pair < n_half; half += 4) {
    __syncthreads();
    __syncthreads();
  }
}

}  // namespace

// Where the chain of launches costs more than a chain of steps in one workgroup: up to the row blocks that stream (kStreamBytes), and from
//   d = 128   the first        (4 layers, whole forward, unfused -> fused: 2 blocks 77 -> 75 us, 128: 104 -> 94, 512: 190 -> 161, 1000: 311 -> 276),
//   d = 192   64 blocks        (2: 87 -> 91, 32: 96 -> 97, 64: 111 -> 106, 256: 162 -> 140, 512: 263 -> 230),
//   d = 256  160 blocks        (2: 81 -> 102, 64: 114 -> 126, 128: 141 -> 142, 192: 163 -> 151, 512: 323 -> 291).
// Below, a block's d / 64 turns of columns one after another are longer than K1's small tiles side by side on a chip that is mostly idle.
constexpr int kLayerFrom192 = 64, kLayerFrom256 = 160;
bool layer_fused(int d, int n_blk) {
  const int from = d == 128 ? 1 : d == 192 ? kLayerFrom192 : kLayerFrom256;
  return (d == 128 || d == 192 || d == 256) && n_blk >= from && (int64_t)n_blk * kRowAlign * d * 2 <= kStreamBytes;
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
#define LAYER_CASE(NK) layer_kernel<NK><<<n_blk, 512, layer_lds_bytes<NK>(), s>>>((const half_t *)O, (const half_t *)U, (const bf16_t *)gamma, (const bf16_t *)beta, (const half_t *)W2p_layer, \
    (const bf16_t *)b2, (half_t *)Xh, (half_t *)Xl, lo_is_zero ? 1 : 0, blocks, blk_list, blk_first, sh.eps, (const half_t *)W1h_next, (const bf16_t *)b1_next, planes, all_hist ? 1 : 0, \
    all_cand ? 1 : 0, sh.ws_rows, sh.alpha)
  if (sh.d == 128) LAYER_CASE(4);
  else if (sh.d == 192) LAYER_CASE(6);
  else LAYER_CASE(8);
#undef LAYER_CASE
}

}  // namespace flame
