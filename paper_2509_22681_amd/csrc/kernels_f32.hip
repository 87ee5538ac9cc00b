// fp32 instantiation of the GR block.  It serves the 1e-4 parity case and every shape the fp16 kernels do not cover.  The projections run on the
// bf16 matrix instruction with operands split into three parts (see gemm_f32_kernel), attention on the fp32 matrix instruction (32 x 32 x 2: fp32
// operands and accumulator, the arithmetic of a chain of FMAs).
//
// Operand layout of the fp32 instruction: acc[i][j] += sum over two k slots of A[i][k] B[j][k]; lane l
// supplies row l & 31 of either operand for k slot l >> 5.  A lane reads four consecutive floats of its row at offset
// 4 (l >> 5) of every group of eight, which feeds four instructions (slots {8 g + t, 8 g + 4 + t}) from one 16-byte load.
// Accumulator element e of a lane is row 8 (e / 4) + 4 (l >> 5) + e % 4 of A, row l & 31 of B.
#include <type_traits>

#include "device_common.h"
#include "kernels.h"

namespace flame {

namespace {

__device__ __forceinline__ void mfma_f32_k8(const f32x4 a, const f32x4 b, f32x16 &acc) {
#pragma unroll
  for (int t = 0; t < 4; ++t) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a[t], b[t], acc, 0, 0, 0);
}

// Four consecutive floats p[k..k+3], zero where k >= K.  VEC: rows are 16-byte aligned and K is a multiple of 4.
template <bool VEC>
__device__ __forceinline__ f32x4 load4(const float *p, int k, int K) {
  f32x4 v = {0.f, 0.f, 0.f, 0.f};
  if constexpr (VEC) {
    if (k < K) v = *(const f32x4 *)(p + k);
  } else {
#pragma unroll
    for (int t = 0; t < 4; ++t)
      if (k + t < K) v[t] = p[k + t];
  }
  return v;
}

// silu(x) = x / (1 + exp(-x)) with the reciprocal by the hardware's estimate and one Newton step (within an ulp of the quotient, a third of its
// instructions).  Where exp(-x) overflows (x below about -88.7) the estimate is 0 and its error no number: held to the most that an estimate is off by, it adds nothing
// and the result is -0, as the quotient's.  (Between there and -87.3 the estimate is subnormal and may be flushed: 0 in place of 1e-36.)  -inf gives NaN, as the quotient.
__device__ __forceinline__ float silu_newton(float x) {
  const float t = 1.0f + __expf(-x);
  const float r = __builtin_amdgcn_rcpf(t);
  const float e = fmaxf(__builtin_fmaf(-t, r, 1.0f), -1e-6f);
  return x * __builtin_fmaf(e, r, r);
}

// Sum over the 16 lanes of a row of lanes, delivered to all of them.
__device__ __forceinline__ float row16_sum(float v) {
  v += __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(v), 0x128, 0xf, 0xf, false));  // row_ror:8
  v += __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(v), 0x124, 0xf, 0xf, false));  // row_ror:4
  v += __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(v), 0x122, 0xf, 0xf, false));  // row_ror:2
  v += __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(v), 0x121, 0xf, 0xf, false));  // row_ror:1
  return v;
}

}  // namespace

// ---------------------------------------------------------------------------------------------
// C[m][n] = sum_k A[m][k] W[n][k] + bias[n] on 64-row blocks.  256 threads = WM x WN wavefronts of MB x NB blocks of 32 x 32 outputs; k in chunks of 32.
// Both operands are split into three bf16 values, and six of the nine products run on the bf16 matrix instruction (32 x 32 x 16, fp32
// accumulators), the small ones first; left out are three, of up to 2^-25 of the product each (a part is up to 2^-8 of the one before it) and 2^-24 together.  6 x 32 cycles for 16 k against 8 x 64 on the fp32 instruction, and the sums
// are rounded less often (a product of bf16 values is exact, and 16 k go into an accumulator at a time instead of 2).
// PACKED: W arrives split and packed by fragments (split_w in misc.hip), by LDS-DMA, a chunk ahead through two stages; else (64 x 64 tiles only: callers without room for the packed copy) it is split here, like A,
// on the way from registers to LDS.  The split is the same, so the two agree bit for bit.  (Forwards that fill the static workspace so, against 128 x 128 tiles on the fp32
// instruction: d = 128, 4 layers 354 -> 327 us, d = 256, 4 layers 470 -> 379, d = 512, 2 layers 364 -> 273.)
// LDS rows of A are 64 bytes per part, 16-byte chunks XOR-swizzled over groups of four rows (key: row bits 2..3), which the fragment reads take
// without bank conflicts.  Tiles of 64 rows have two stages for A, tiles of 128 one (two workgroups on a compute unit, one's staging under
// the other's matrix work).
// EPI 0: planes[p][m][n] = silu(C) with A = X.
// EPI 1: X[m][n] += C with A = (LayerNorm(O) * gamma + beta) * U, made while the chunk is staged: the statistics of the 64
//        rows come first (mean, then the centred second moment), and the gated rows never travel through memory.
// 20 480 rows, d = 256: K1 116 -> 82 us per launch against the fp32 instruction (its work alone is 26 us; a workgroup spends a third of its time on splitting A and on its
// requests, and two are resident on a compute unit), 45 us where only V and K are needed; the output projection, whose row statistics come first, 45 -> 38.  Error of the scores
// against 64 bits 0.87 of what it was (geometric mean of 24 outputs of widths 64 to 256, of which two rose, by 4 and 7 %).
// ---------------------------------------------------------------------------------------------
// (A, U, gamma, beta and W carry no __restrict__: loads that the compiler knows to be unchanging may pass any fence, and the counted waits for W need the requests in order.)
// NI (EPI 1): 16-byte loads per lane and row that the statistics keep in registers, ceil(K / 64) at least; 0: any K, in two reads of the rows.
template <int EPI, int WM, int WN, int MB, int NB, bool PACKED, bool VEC, int NI, bool SCORE = false>
__global__ __launch_bounds__(256, MB * NB == 4 ? 2 : 1) void gemm_f32_kernel(const float *A, const float *U, const float *gamma,
                                                       const float *beta, const RowBlock *__restrict__ blocks, float eps,
                                                       const void *Wv, const float *__restrict__ bias, float *__restrict__ out,
                                                       const int32_t *__restrict__ blk_list, int blk_first, int n_blk, int d, int n_planes, int plane0, int plane_step,
                                                       int64_t plane_stride, int y2, const int32_t *__restrict__ blk_list2, int n_blk2,
                                                       const float *__restrict__ w_s = nullptr, float b_s = 0.f, float *__restrict__ scores = nullptr) {
  static_assert(WM * WN == 4, "four wavefronts");
  constexpr int BM = 32 * WM * MB, BN = 32 * WN * NB, BK = 32, TB = BM / 64, LPT = BM / 32;   // tile, k chunk, 64-row blocks, 16-byte loads of A per thread
  constexpr int AST = TB == 1 ? 2 : 1, APART = BM * BK * 2, ASTAGE = 3 * APART, WSTAGE = 3 * BN * BK * 2;
  __shared__ __attribute__((aligned(256))) char lds[AST * ASTAGE + 2 * WSTAGE];
  __shared__ float s_mu[EPI == 1 ? 64 : 1], s_rstd[EPI == 1 ? 64 : 1];
  static_assert(EPI == 0 || TB == 1, "row statistics are kept for one block of rows");
  static_assert(PACKED || (BM == 64 && BN == 64), "raw W: 64 x 64 tiles");
  char *const ldsw = lds + AST * ASTAGE;
  const int K = d, dp = (d + 31) / 32 * 32, pb = dp / 32;      // 32-column blocks per plane
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / WN, wn = wave % WN, l32 = lane & 31, lhalf = lane >> 5;
  // 32-column block b of the launch, counted over its planes: matrix (plane) and block in it; blocks past the last repeat it and are not stored
  int cy = blockIdx.y;
  if (EPI == 0 && cy >= y2) {                              // the second part of the launch: U and Q of its own blocks
    cy -= y2;
    plane0 = 0;
    blk_list = blk_list2;
    n_blk = n_blk2;
    if ((int)blockIdx.x * TB >= n_blk) return;
  }
  const int nb_all = n_planes * pb, cb0 = cy * (BN / 32);
  auto plane_of = [&](int b) { return plane0 + min(b, nb_all - 1) / pb * plane_step; };
  auto block_of = [&](int b) { return min(b, nb_all - 1) % pb; };
  int64_t row0[TB];
  bool present[TB];
#pragma unroll
  for (int t = 0; t < TB; ++t) {
    const int i = blockIdx.x * TB + t;
    present[t] = i < n_blk;
    const int ic = present[t] ? i : n_blk - 1;
    row0[t] = (int64_t)(blk_list ? blk_list[ic] : blk_first + ic) * kRowAlign;
  }
  int n_valid = kRowAlign;
  if constexpr (EPI == 1) {
    n_valid = blocks[row0[0] / kRowAlign].n_valid;
    if constexpr (NI > 0) {
      // statistics: 16 lanes per row, four rows of a wavefront at a time, all of its rows' loads in flight together
      // (up to 16 x 16 bytes per lane), so that the memory latency is paid once or twice and not once per row
      constexpr int RB = NI > 4 ? 2 : 4;             // row groups per round
      const int c16 = lane & 15, rq = lane >> 4;
#pragma unroll
      for (int g0 = 0; g0 < 4; g0 += RB) {
        f32x4 v[RB][NI];
        float mu[RB], sq[RB];
#pragma unroll
        for (int g = 0; g < RB; ++g)
#pragma unroll
          for (int i = 0; i < NI; ++i)
            v[g][i] = load4<true>(A + (row0[0] + wave * 16 + 4 * (g0 + g) + rq) * K, 4 * (c16 + 16 * i), K);
#pragma unroll
        for (int g = 0; g < RB; ++g) {
          mu[g] = 0.f;
#pragma unroll
          for (int i = 0; i < NI; ++i) mu[g] += (v[g][i][0] + v[g][i][1]) + (v[g][i][2] + v[g][i][3]);
        }
#pragma unroll
        for (int g = 0; g < RB; ++g) mu[g] = row16_sum(mu[g]) / (float)K;
#pragma unroll
        for (int g = 0; g < RB; ++g) {
          sq[g] = 0.f;
#pragma unroll
          for (int i = 0; i < NI; ++i)
            if (4 * (c16 + 16 * i) < K) {
#pragma unroll
              for (int t = 0; t < 4; ++t) { const float c = v[g][i][t] - mu[g]; sq[g] += c * c; }
            }
        }
#pragma unroll
        for (int g = 0; g < RB; ++g) {
          const float rstd = rsqrtf(row16_sum(sq[g]) / (float)K + eps);
          const int r = wave * 16 + 4 * (g0 + g) + rq;
          if (c16 == 0) { s_mu[r] = mu[g]; s_rstd[r] = rstd; }
        }
      }
    } else {
      for (int b = 0; b < 4; ++b) {
        const int r = wave * 16 + 4 * b;
        const float *o = A + (row0[0] + r) * K;
        float s[4] = {0.f, 0.f, 0.f, 0.f};
        for (int k = lane; k < K; k += 64)
#pragma unroll
          for (int q = 0; q < 4; ++q) s[q] += o[(int64_t)q * K + k];
#pragma unroll
        for (int q = 0; q < 4; ++q) s[q] = wave_sum(s[q]) / (float)K;
        float v[4] = {0.f, 0.f, 0.f, 0.f};
        for (int k = lane; k < K; k += 64)
#pragma unroll
          for (int q = 0; q < 4; ++q) { const float c = o[(int64_t)q * K + k] - s[q]; v[q] += c * c; }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          v[q] = rsqrtf(wave_sum(v[q]) / (float)K + eps);
          if (lane == 0) { s_mu[r + q] = s[q]; s_rstd[r + q] = v[q]; }
        }
      }
    }
    __syncthreads();
  }
  // staging: thread (row = tid / 8 + 32 i, chunk = tid % 8) brings 16 bytes of A.  The loads stay as they come until split():
  // an operand made in fetch() would wait for its loads ahead of the matrix work that is there to hide them.
  // VEC loads are unconditional, at a clamped address where the matrix ends, and zeroed in split() (a branch around each costs more).
  const int sr = tid >> 3, sc = tid & 7;
  f32x4 ra[2][LPT], ru[2][EPI == 1 ? LPT : 1], rg[2], rb[2], rw[2][PACKED ? 1 : 2];   // chunks of even and of odd index
  float mu[EPI == 1 ? LPT : 1], rstd[EPI == 1 ? LPT : 1];
  if constexpr (EPI == 1) {
#pragma unroll
    for (int i = 0; i < LPT; ++i) { mu[i] = s_mu[sr + 32 * i]; rstd[i] = s_rstd[sr + 32 * i]; }
  }
  auto load = [&](const float *p, int k) { return VEC ? *(const f32x4 *)(p + min(k, K - 4)) : load4<false>(p, k, K); };
  auto fetch = [&](auto set_c, int k0) {
    constexpr int F = decltype(set_c)::value;
    const int k = k0 + 4 * sc;
    if constexpr (EPI == 1) { rg[F] = load(gamma, k); rb[F] = load(beta, k); }
#pragma unroll
    for (int i = 0; i < LPT; ++i) {
      const int r = sr + 32 * i;
      const int64_t m = row0[TB == 1 ? 0 : r >> 6] + (r & 63);
      ra[F][i] = load(A + m * K, k);
      if constexpr (EPI == 1) ru[F][i] = load(U + m * K, k);
    }
    if constexpr (!PACKED) {
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const int c = min(block_of(cb0 + i) * 32 + sr, d - 1);      // (columns past the matrix are computed and not stored)
        rw[F][i] = load((const float *)Wv + ((int64_t)plane_of(cb0 + i) * d + c) * K, k);
      }
    }
  };
  Split3 pa[LPT], pw[PACKED ? 1 : 2];
  auto split = [&](auto set_c, int k0) {
    constexpr int F = decltype(set_c)::value;
    const bool inside = !VEC || k0 + 4 * sc < K;
    const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < LPT; ++i) {
      f32x4 v = ra[F][i];
      if constexpr (EPI == 1) {
#pragma unroll
        for (int t = 0; t < 4; ++t) v[t] = ((v[t] - mu[i]) * rstd[i] * rg[F][t] + rb[F][t]) * ru[F][i][t];
      }
      pa[i] = split3(inside && (EPI == 0 || sr + 32 * i < n_valid) ? v : zero);
    }
    if constexpr (!PACKED) {
#pragma unroll
      for (int i = 0; i < 2; ++i) pw[i] = split3(inside ? rw[F][i] : zero);
    }
  };
  // byte offset of 16-byte chunk c (0..3) of tile row r inside a part of A
  auto off = [](int r, int c) { return (r >> 2) * 256 + ((((r & 3) << 2) | (c ^ ((r >> 2) & 3))) << 4); };
  auto store = [&](int ast, int wst) {
#pragma unroll
    for (int i = 0; i < LPT; ++i)
#pragma unroll
      for (int p = 0; p < 3; ++p) *(bf16x4 *)(lds + ast * ASTAGE + p * APART + off(sr + 32 * i, sc >> 1) + (sc & 1) * 8) = pa[i].p[p];
    if constexpr (!PACKED) {                            // into the fragments' places: k 4 sc .. + 3 of column 32 i + sr
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int p = 0; p < 3; ++p)
          *(bf16x4 *)(ldsw + wst * WSTAGE + (i * 6 + (sc >> 2) * 3 + p) * 1024 + (((sc >> 1) & 1) * 32 + sr) * 16 + (sc & 1) * 8) = pw[i].p[p];
    }
  };
  // W of a chunk: six fragments (two of 16 k, three parts) per 32-column block, 6 KB in one piece; fragment q of the tile belongs to wavefront q % 4
  typedef __attribute__((address_space(1))) const void gvoid;
  typedef __attribute__((address_space(3))) void lvoid;
  auto request_w = [&](int kc, int st) {
    if constexpr (PACKED) {
#pragma unroll
      for (int i = 0; i < 6 * (BN / 32) / 4; ++i) {
        const int q = wave + 4 * i, b = cb0 + q / 6;
        const char *src = (const char *)Wv + (((int64_t)plane_of(b) * pb + block_of(b)) * (dp / 16) + 2 * kc) * 3072 + (q % 6) * 1024;
        __builtin_amdgcn_global_load_lds((gvoid *)(src + lane * 16), (lvoid *)(ldsw + st * WSTAGE + q * 1024), 16, 0, 0);
      }
    }
  };
  // W of the chunk requested last has landed: behind it at least the rows of one chunk were fetched (without 16-byte loads they are as many as the matrix has, and the
  // wait is for all).  pin() keeps requests in the order in which they are counted.
  auto pin = [&]() { asm volatile("" ::: "memory"); __builtin_amdgcn_sched_barrier(0); };
  auto wait_w = [&]() { asm volatile("s_waitcnt vmcnt(%0)" ::"n"(VEC && PACKED ? (EPI == 1 ? 2 * LPT + 2 : LPT) : 0) : "memory"); };
  f32x16 acc[MB][NB];
#pragma unroll
  for (int i = 0; i < MB; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;
  typedef std::integral_constant<int, 0> EVEN;
  typedef std::integral_constant<int, 1> ODD;
  const int nk = dp / BK;
  request_w(0, 0);
  pin();
  fetch(EVEN{}, 0);
  if (nk > 1) fetch(ODD{}, BK);
  pin();
  // the residual's values of this lane, requested ahead of the k loop (read one by one between its stores they would cost a
  // memory latency each)
  float xr[EPI == 1 ? MB : 1][EPI == 1 ? NB : 1][16];
  if constexpr (EPI == 1) {
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
      for (int j = 0; j < NB; ++j) {
        const float *x = out + (row0[0] + (wm * MB + i) * 32 + 4 * lhalf) * d + min((cb0 + wn * NB + j) * 32 + l32, d - 1);
#pragma unroll
        for (int e = 0; e < 16; ++e) xr[i][j][e] = x[(int64_t)(8 * (e >> 2) + (e & 3)) * d];
      }
  }
  split(EVEN{}, 0);
  store(0, 0);
  wait_w();                                              // W of chunk 0 has landed
  __syncthreads();
  // The rows come from far away (past the L2s, several thousand cycles under load): they are fetched two chunks ahead, W (from an L2) one.  As built, the look-ahead of the rows is lost:
  // a __syncthreads with LDS-DMA pending waits for all loads, and with EPI 1 such a wait stands ahead of a chunk's first LDS read.
  auto chunk = [&](auto parity_c, auto ahead_c, const int kc) {
    constexpr bool AHEAD = decltype(ahead_c)::value;     // there is a chunk after the next
    constexpr int PAR = decltype(parity_c)::value, ast = AST == 2 ? PAR : 0, wst = PAR;
    std::integral_constant<int, PAR ^ 1> other;
    if (AHEAD || kc + 1 < nk) request_w(kc + 1, wst ^ 1);           // everybody left that stage at the barrier that opened this chunk
    pin();
    if constexpr (AHEAD) fetch(parity_c, (kc + 2) * BK);
    pin();                                                 // the requests stay ahead of the matrix work
    auto multiply = [&](int s) {
      bf16x8 fa[MB][3], fw[NB][3];
#pragma unroll
      for (int p = 0; p < 3; ++p) {
#pragma unroll
        for (int i = 0; i < MB; ++i) fa[i][p] = *(const bf16x8 *)(lds + ast * ASTAGE + p * APART + off((wm * MB + i) * 32 + l32, 2 * s + lhalf));
#pragma unroll
        for (int j = 0; j < NB; ++j) fw[j][p] = *(const bf16x8 *)(ldsw + wst * WSTAGE + ((wn * NB + j) * 6 + s * 3 + p) * 1024 + lane * 16);
      }
      constexpr int PA[6] = {2, 0, 1, 1, 0, 0}, PW[6] = {0, 2, 1, 0, 1, 0};
#pragma unroll
      for (int q = 0; q < 6; ++q)
#pragma unroll
        for (int i = 0; i < MB; ++i)
#pragma unroll
          for (int j = 0; j < NB; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[i][PA[q]], fw[j][PW[q]], acc[i][j], 0, 0, 0);
    };
    multiply(0);
    __builtin_amdgcn_sched_barrier(0);
    // the next chunk is split under the second half of the matrix work (where its parts are stored unconditionally; else the compiler moves the split to the store)
    multiply(1);
    split(other, (kc + 1) * BK);                                // (behind the last chunk: of what was fetched for it, and not stored)
    __builtin_amdgcn_sched_group_barrier(0x100, 3 * (MB + NB), 0);
#pragma unroll
    for (int i = 0; i < 6 * MB * NB; ++i) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x002, EPI == 1 ? 8 : 5, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
    if (AST == 1) __syncthreads();                         // everybody has left the stage of A
    if (AHEAD || kc + 1 < nk) store(AST == 2 ? ast ^ 1 : 0, wst ^ 1);
    // W of the next chunk has landed
    if constexpr (AHEAD) wait_w();
    else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
  };
  // The last two chunks, which fetch no rows and wait for all, are code of their own: what is waited for never depends on a branch.  (As a branch in the loop: base_f32 676 us per
  // forward, with the last chunk's rows fetched over again so that the count holds 690, so 654.)
  typedef std::true_type AHEAD;
  typedef std::false_type TAIL;
  int kc = 0;
  for (; kc + 3 < nk; kc += 2) {
    chunk(EVEN{}, AHEAD{}, kc);
    chunk(ODD{}, AHEAD{}, kc + 1);
  }
  if (kc + 2 < nk) {
    chunk(EVEN{}, AHEAD{}, kc);
    chunk(ODD{}, TAIL{}, kc + 1);
    chunk(EVEN{}, TAIL{}, kc + 2);
  } else {
    chunk(EVEN{}, TAIL{}, kc);
    if (kc + 1 < nk) chunk(ODD{}, TAIL{}, kc + 1);
  }
  if constexpr (SCORE) {
    // The last layer of a model of up to 64 features: the workgroup has its candidates' whole rows, which only the score head reads.  Sums in the order of score_kernel: columns n
    // and n + 32 first (the two wavefronts of the rows, through the free stage of A), then the 32 lanes.
    static_assert(EPI == 1 && WM == 2 && WN == 2 && MB == 1 && NB == 1, "a row block of 64 features");
    const int n = wn * 32 + l32;
    const bool inside = n < d;
    const float w = inside ? w_s[n] : 0.f, bn = inside ? bias[n] : 0.f;
    float p[16];
#pragma unroll
    for (int e = 0; e < 16; ++e) p[e] = inside ? __builtin_fmaf(xr[0][0][e] + (acc[0][0][e] + bn), w, 0.f) : 0.f;
    __syncthreads();
    float *part = (float *)lds + (wm * 16 * 64 + lane);
    if (wn == 1) {
#pragma unroll
      for (int e = 0; e < 16; ++e) part[e * 64] = p[e];
    }
    __syncthreads();
    if (wn == 0) {
      const int src = blocks[row0[0] / kRowAlign].src_row;
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        float v = p[e] + part[e * 64];
        const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
        v = row16_sum(__uint_as_float(r[0]) + __uint_as_float(r[1]));
        const int row = wm * 32 + 8 * (e >> 2) + 4 * lhalf + (e & 3);
        if (l32 == 0 && row < n_valid) scores[src + row] = v + b_s;
      }
    }
    return;
  }
  // a lane holds one output column and 16 rows: 32 lanes write 128 contiguous bytes of a row
#pragma unroll
  for (int j = 0; j < NB; ++j) {
    const int b = cb0 + wn * NB + j, plane = plane_of(b), n = block_of(b) * 32 + l32;
    if (b >= nb_all || n >= d) continue;
    const float bn = bias[(int64_t)plane * d + n];
    float *col = out + plane * plane_stride + n;           // (EPI 1: one matrix, its plane is X)
#pragma unroll
    for (int i = 0; i < MB; ++i) {
      const int r32 = (wm * MB + i) * 32, blk = TB == 1 ? 0 : r32 >> 6;
      if (!present[blk]) continue;
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int64_t m = row0[blk] + (r32 & 63) + 8 * (e >> 2) + 4 * lhalf + (e & 3);
        const float v = acc[i][j][e] + bn;
        if constexpr (EPI == 0) col[m * d] = silu_newton(v);
        else col[m * d] = xr[i][j][e] + v;
      }
    }
  }
}

// 16-byte loads of the operands: rows of the workspaces start on 16 bytes when d does; weights where the caller put them
static bool vec4_rows(int d, const void *p) { return d % 4 == 0 && (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

// W, W2: the matrices of the layer, as they are or (packed) split and packed by fragments
void launch_uvqk_f32(const float *X, const void *W1, bool packed, const float *b1, float *planes, const int32_t *blk_list, int n_blk, int blk_first, int plane_mask,
                     const int32_t *uq_list, int n_uq, const Shape &sh, hipStream_t s) {
  if (n_blk <= 0) return;
  // all planes, or every other one: U and Q, V and K
  const bool all = plane_mask == 0xF;
  const int np = all ? 4 : 2, plane0 = plane_mask == 0xA ? 1 : 0, step = all ? 1 : 2, nb = np * ((sh.d + 31) / 32);
#define UVQK_CASE(WM, WN, MB, NB, PK, VV) do { const int y = (nb + WN * NB - 1) / (WN * NB); \
    gemm_f32_kernel<0, WM, WN, MB, NB, PK, VV, 0><<<dim3((n_blk + WM * MB / 2 - 1) / (WM * MB / 2), n_uq > 0 ? 2 * y : y), 256, 0, s>>>( \
      X, nullptr, nullptr, nullptr, nullptr, 0.f, W1, b1, planes, blk_list, blk_first, n_blk, sh.d, np, plane0, step, sh.ws_rows * sh.d, y, uq_list, n_uq); } while (0)
  const bool vec = sh.d % 4 == 0;
  if (packed) {
    // 128 x 128 tiles halve the operand traffic; a launch needs enough of them for two per compute unit
    const bool big = (int64_t)((n_blk + 1) / 2) * ((nb + 3) / 4) >= 512;
    if (vec) { if (big) UVQK_CASE(2, 2, 2, 2, true, true); else UVQK_CASE(2, 2, 1, 1, true, true); }
    else UVQK_CASE(2, 2, 1, 1, true, false);
  } else {
    if (vec && vec4_rows(sh.d, W1)) UVQK_CASE(2, 2, 1, 1, false, true);
    else UVQK_CASE(2, 2, 1, 1, false, false);
  }
#undef UVQK_CASE
}

bool outproj_scores_f32(const float *gamma, const float *beta, const void *W2, bool packed, const Shape &sh) {
  return sh.d <= 64 && vec4_rows(sh.d, gamma) && vec4_rows(sh.d, beta) && (packed || vec4_rows(sh.d, W2));
}

void launch_outproj_f32(const float *O, const float *U, const float *gamma, const float *beta, const void *W2, bool packed, const float *b2, float *X,
                        const RowBlock *blocks, const int32_t *blk_list, int n_blk, int blk_first, const float *w_s, float b_s, float *scores, const Shape &sh, hipStream_t s) {
  if (n_blk <= 0) return;
  const int nb = (sh.d + 31) / 32;
  if (scores) {
#define OUT_SCORE(PK) gemm_f32_kernel<1, 2, 2, 1, 1, PK, true, 1, true><<<dim3(n_blk, 1), 256, 0, s>>>( \
      O, U, gamma, beta, blocks, sh.eps, W2, b2, X, blk_list, blk_first, n_blk, sh.d, 1, 0, 1, 0, 1 << 30, nullptr, 0, w_s, b_s, scores)
    if (packed) OUT_SCORE(true);
    else OUT_SCORE(false);
#undef OUT_SCORE
    return;
  }
#define OUT_CASE(WM, WN, MB, NB, PK, VV, NI) gemm_f32_kernel<1, WM, WN, MB, NB, PK, VV, NI><<<dim3(n_blk, (nb + WN * NB - 1) / (WN * NB)), 256, 0, s>>>( \
      O, U, gamma, beta, blocks, sh.eps, W2, b2, X, blk_list, blk_first, n_blk, sh.d, 1, 0, 1, 0, 1 << 30, nullptr, 0)
#define OUT_WIDTHS(PK) do { \
    if (sh.d <= 64) OUT_CASE(2, 2, 1, 1, PK, true, 1); \
    else if (sh.d <= 128) OUT_CASE(2, 2, 1, 1, PK, true, 2); \
    else if (sh.d <= 256) OUT_CASE(2, 2, 1, 1, PK, true, 4); \
    else if (sh.d <= 512) OUT_CASE(2, 2, 1, 1, PK, true, 8); \
    else OUT_CASE(2, 2, 1, 1, PK, true, 0); } while (0)
  const bool vec = vec4_rows(sh.d, gamma) && vec4_rows(sh.d, beta);
  if (packed) {
    if (!vec) OUT_CASE(2, 2, 1, 1, true, false, 0);
    // 64 x 128 tiles where they have no empty columns and there are as many as two rounds of the chip at two per compute unit.  Forwards of five layers with 64 x 64 tiles / with
    // these (us), 64-row blocks: d = 256: 128: 326 / 329, 192: 451 / 450, 256: 560 / 535, 512: 1063 / 1006; d = 128: 256: 240 / 242, 320: 331 / 333, 512: 435 / 421;
    // with empty columns, d = 192: 128: 254 / 261, 512: 714 / 722; d = 160: 512: 585 / 594.
    else if (nb % 4 == 0 && sh.d <= 256 && (int64_t)n_blk * nb >= 2048) {
      if (sh.d <= 128) OUT_CASE(1, 4, 2, 1, true, true, 2);
      else OUT_CASE(1, 4, 2, 1, true, true, 4);
    } else OUT_WIDTHS(true);
  } else {
    if (vec && vec4_rows(sh.d, W2)) OUT_WIDTHS(false);
    else OUT_CASE(2, 2, 1, 1, false, false, 0);
  }
#undef OUT_WIDTHS
#undef OUT_CASE
}

// ---------------------------------------------------------------------------------------------
// Attention.  One workgroup = 64 query rows of one head, four wavefronts: two groups of 32 rows, each served by two wavefronts
// that take every other block of 32 keys and add up at the end (in a fixed order).  Transposed products as in the fp16
// kernel: S^T = K Q^T puts 16 keys of one query into a lane, in the very slots that O^T += V^T P^T takes as its B operand
// (instruction e of a block multiplies keys 8 (e / 4) + e % 4 and + 4), so the weights never leave their registers.
// STAGED (heads of exactly 32 or 64): K and V arrive by LDS-DMA in tiles of 64 keys, two stages, the next tile requested while this one is
// multiplied.  A lane's 16 bytes of a K row from global memory are 32 lines per instruction, 360 requests per block of 32 keys and
// wavefront, and the compute unit has too few of them in flight to feed the matrix instruction; through LDS a wavefront makes 64 for a tile.
// 32 x (512 + 128), 4 heads of 64: 106 -> 91 us per launch (43 at the matrix rate), the candidates alone 31 -> 33 us.
// Other widths read their operands straight from global memory, without a barrier.  Heads of 129 to 256 hold 256 accumulators and the query
// row's fragments in registers, one wavefront per SIMD, and do not fit: 375 to 397 registers spill (51 to 54 at a width of exactly 256).  They are
// the slow ones for it, 32 x (256 + 64) on 2 heads 167 us per launch at a width of 160 and 73 at 256, against 32 at 128 (with one
// wavefront per query row and plain FMAs 4171, 6574 and 3108).
// DB = 32-wide blocks of the head; EXACT: the head is exactly 32 DB wide (vector loads), else elements past it count as zero.
// A lane's V operand of block b is feature DB * row + b, so that one load brings a lane's features of all blocks.
// ---------------------------------------------------------------------------------------------
template <int DB, bool EXACT, bool SOFTMAX>
__global__ __launch_bounds__(256) void attn_f32_kernel(const float *__restrict__ U_V_Q_K, const float *__restrict__ bias_lh,
                                                       const float *__restrict__ tscale_h,
                                                       float *__restrict__ O, const AttnItem *__restrict__ items, int n_items,
                                                       int d, int dh, int D, float alpha, int64_t plane_stride) {
  constexpr int NG = 4 * DB;                         // groups of eight features
  constexpr int DBR = DB < 4 ? DB : 4;               // head blocks that leave per round at the end
  constexpr int PITCH = 32 * DBR + 4;                // floats per row of the output patch of 32 query rows
  // STAGED: two LDS stages of a tile of 64 keys, K rows and V rows of RB bytes, 16-byte chunks XOR-swizzled by row.  The output patches
  // and the row states reuse them once the keys are done.
  constexpr bool STAGED = EXACT && DB <= 2;
  constexpr int RB = 128 * DB, CH = RB / 16, TILE = 64 * RB, STAGE = 2 * TILE;
  constexpr int PATCH_BYTES = 2 * 32 * PITCH * 4, TAIL_BYTES = PATCH_BYTES + (2 * 2 * 64 + 2 * 2 * 32) * 4;
  constexpr int LDS_BYTES = STAGED && 2 * STAGE > TAIL_BYTES ? 2 * STAGE : TAIL_BYTES;
  __shared__ __attribute__((aligned(256))) char lds[LDS_BYTES];
  float (*const s_patch)[32 * PITCH] = (float (*)[32 * PITCH])lds;
  float (*const s_state)[2][64] = (float (*)[2][64])(lds + PATCH_BYTES);
  float (*const s_row)[2][32] = (float (*)[2][32])(lds + PATCH_BYTES + 2 * 2 * 64 * 4);
  auto lkey = [](int row) { return CH == 16 ? row & 15 : (row >> 1) & 7; };
  const int item = blockIdx.z * gridDim.y + blockIdx.y;   // heads of an item side by side: the longest items of all heads start first
  if (item >= n_items) return;
  const AttnItem it = items[item];
  const int h = blockIdx.x;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int l32 = lane & 31, lhalf = lane >> 5;
  const int qg = wave & 1, split = wave >> 1;
  const float *Vp = U_V_Q_K + 1 * plane_stride + h * dh;
  const float *Qp = U_V_Q_K + 2 * plane_stride + h * dh;
  const float *Kp = U_V_Q_K + 3 * plane_stride + h * dh;
  const float *bias = bias_lh + (int64_t)h * D;
  const int q0 = qg * 32;
  const bool active = q0 < it.n_q;
  const int q_local = q0 + l32;
  const bool row_valid = q_local < it.n_q;
  const int64_t qrow = it.q_row + (row_valid ? q_local : it.n_q - 1);        // clamped for the loads
  const int q_index = it.is_cand ? it.L : it.q_pos + q_local;
  const int n_vis = row_valid ? visible_history(it.is_cand, q_index, it.L) : 0;
  const int vis_max = active ? (it.is_cand ? it.L : min(it.q_pos + q0 + 32, it.n_kv)) : 0;
  // every row of this group sees all keys before vis_min (no row does where the tile ends inside the group)
  const int vis_min = q0 + 32 > it.n_q ? 0 : it.is_cand ? it.L : it.q_pos + q0 + 1;
  constexpr float kNeg = -1.0e30f;                   // a finite stand-in for -inf
  const float ts = SOFTMAX ? tscale_h[h] : 0.f;
  float m_run = kNeg, l_run = 0.f;                   // softmax: running maximum of my row, and the sum over this lane's keys
  // features 8 g + 4 lhalf + 0..3 of a row
  auto row4 = [&](const float *row, int g) {
    const int k = 8 * g + 4 * lhalf;
    if constexpr (EXACT) return *(const f32x4 *)(row + k);
    f32x4 v = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int t = 0; t < 4; ++t)
      if (k + t < dh) v[t] = row[k + t];
    return v;
  };
  f32x4 fq[NG];
#pragma unroll
  for (int g = 0; g < NG; ++g) fq[g] = row4(Qp + qrow * d, g);
  f32x16 oacc[DB];
#pragma unroll
  for (int b = 0; b < DB; ++b)
#pragma unroll
    for (int e = 0; e < 16; ++e) oacc[b][e] = 0.f;
  f32x4 fk[NG];
  auto load_k = [&](int k0) {
#pragma unroll
    for (int g = 0; g < NG; ++g) fk[g] = row4(Kp + ((int64_t)it.kv_row + k0 + l32) * d, g);
  };
  // One block of 32 keys: S^T, weights, O^T; fv[e][b] = feature DB l32 + b of key 8 (e / 4) + 4 lhalf + e % 4, bz the keys' bias.
  float fv[16][DB], bz[16];
  auto load_bias = [&](int k0) {
#pragma unroll
    for (int e = 0; e < 16; ++e) bz[e] = bias[max(0, min(D - 1, q_index - (k0 + 8 * (e >> 2) + 4 * lhalf + (e & 3))))];
  };
  float pw[16];
  auto weigh = [&](int k0, const f32x16 &sacc) {
    float p[16];
    if constexpr (SOFTMAX) {
      float mt = kNeg;
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int c = k0 + 8 * (e >> 2) + 4 * lhalf + (e & 3);
        p[e] = c < n_vis ? (alpha * sacc[e] + bz[e]) * ts : kNeg;
        mt = fmaxf(mt, p[e]);
      }
      const float m_new = fmaxf(m_run, pair_max(mt));
      const float sc = expf(m_run - m_new);
      m_run = m_new;
      l_run *= sc;
#pragma unroll
      for (int b = 0; b < DB; ++b)
#pragma unroll
        for (int e = 0; e < 16; ++e) oacc[b][e] *= sc;
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int c = k0 + 8 * (e >> 2) + 4 * lhalf + (e & 3);
        p[e] = expf(p[e] - m_new);
        asm volatile("" : "+v"(p[e]));     // (keeps the mask below a select: see the other branch)
        p[e] = c < n_vis ? p[e] : 0.f;
        l_run += p[e];
      }
    } else {
      // (all weights first, then the mask: written as one conditional expression, the compiler branches around every single weight and
      // runs sixteen dependent chains one after another: a short launch, 32 x 128 candidates on 512 keys, 33.8 -> 31.0 us)
#pragma unroll
      for (int e = 0; e < 16; ++e) p[e] = silu_newton(alpha * sacc[e] + bz[e]);
      if (k0 + 32 > vis_min) {
#pragma unroll
        for (int e = 0; e < 16; ++e) p[e] = k0 + 8 * (e >> 2) + 4 * lhalf + (e & 3) < n_vis ? p[e] : 0.f;
      }
    }
#pragma unroll
    for (int e = 0; e < 16; ++e) pw[e] = p[e];
  };
  auto add_pv = [&]() {
#pragma unroll
    for (int e = 0; e < 16; ++e)
#pragma unroll
      for (int b = 0; b < DB; ++b) oacc[b] = __builtin_amdgcn_mfma_f32_32x32x2f32(fv[e][b], pw[e], oacc[b], 0, 0, 0);
  };
  if constexpr (STAGED) {
    typedef __attribute__((address_space(1))) const void gvoid;
    typedef __attribute__((address_space(3))) void lvoid;
    constexpr int RPI = 1024 / RB, NI = 64 / RPI / 4;    // rows per request, requests per wavefront and operand
    static_assert(4 * RPI % 16 == 0, "a wavefront's requests of one tile share their swizzle key");
    const int rq = wave * RPI + lane / CH;               // tile row of this lane in its first request
    const uint32_t off = (uint32_t)(rq * d + (((lane % CH) ^ lkey(rq)) << 2)) * 4u;
    auto request = [&](int st, int k0) {
#pragma unroll
      for (int i = 0; i < NI; ++i) {
        const int64_t r = (int64_t)(it.kv_row + k0 + 4 * RPI * i) * d;
        char *dst = lds + st * STAGE + (wave + 4 * i) * 1024;
        __builtin_amdgcn_global_load_lds((gvoid *)((const char *)(Kp + r) + off), (lvoid *)dst, 16, 0, 0);
        __builtin_amdgcn_global_load_lds((gvoid *)((const char *)(Vp + r) + off), (lvoid *)(dst + TILE), 16, 0, 0);
      }
    };
    // this lane's K row, and its V bytes of a row whose index has bit 2 clear (the half wavefront adds 4 rows)
    const int kr = 32 * split + l32;
    const int ka = kr * RB + ((lhalf ^ lkey(kr)) << 4);
    const int va = 4 * lhalf * RB + (((DB * l32 / 4) ^ lkey(4 * lhalf)) << 4) + (DB * l32 % 4) * 4;
    const int n_tiles = (it.n_kv + 63) / 64;             // the same for all wavefronts
    if (n_tiles > 0) request(0, 0);
    for (int t = 0; t < n_tiles; ++t) {
      const int k0 = 64 * t + 32 * split;
      const bool work = k0 < vis_max;
      const char *sk = lds + (t & 1) * STAGE, *sv = sk + TILE;
      // tile t has landed for everybody, and everybody has left tile t - 1, whose stage takes tile t + 1
      // (the builtin: the compiler knows it and sees that the query rows have landed too)
      __builtin_amdgcn_s_waitcnt(0x0f70);                // vmcnt(0)
      asm volatile("" ::: "memory");
      __builtin_amdgcn_s_barrier();
      if (work) load_bias(k0);
      if (t + 1 < n_tiles) request((t + 1) & 1, 64 * (t + 1));
      __builtin_amdgcn_sched_barrier(0);
      if (!work) continue;
#pragma unroll
      for (int g = 0; g < NG; ++g) fk[g] = *(const f32x4 *)(sk + (ka ^ (g << 5)));
      f32x16 sacc;
#pragma unroll
      for (int e = 0; e < 16; ++e) sacc[e] = 0.f;
#pragma unroll
      for (int g = 0; g < NG; ++g) mfma_f32_k8(fk[g], fq[g], sacc);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int r0 = 8 * (e >> 2) + (e & 3);           // + 32 split: a multiple of the key's period
        const float *v = (const float *)(sv + (32 * split + r0) * RB + (va ^ (lkey(r0) << 4)));
        if constexpr (DB == 2) { const float2 w = *(const float2 *)v; fv[e][0] = w.x; fv[e][1] = w.y; }
        else fv[e][0] = *v;
      }
      weigh(k0, sacc);
      add_pv();
    }
    __syncthreads();                                     // everybody has left the last tile
  } else {
    const int first = split * 32, pitch = 64;
    if (first < vis_max) load_k(first);
    for (int k0 = first; k0 < vis_max; k0 += pitch) {
      // V and the bias of this block are requested ahead of its S, K of the next block ahead of its V^T P
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const float *vr = Vp + ((int64_t)it.kv_row + k0 + 8 * (e >> 2) + 4 * lhalf + (e & 3)) * d + DB * l32;
        if constexpr (EXACT && DB == 4) { const f32x4 v = *(const f32x4 *)vr; for (int b = 0; b < DB; ++b) fv[e][b] = v[b]; }
        else {
#pragma unroll
          for (int b = 0; b < DB; ++b) fv[e][b] = EXACT || DB * l32 + b < dh ? vr[b] : 0.f;
        }
      }
      load_bias(k0);
      f32x16 sacc;
#pragma unroll
      for (int e = 0; e < 16; ++e) sacc[e] = 0.f;
#pragma unroll
      for (int g = 0; g < NG; ++g) mfma_f32_k8(fk[g], fq[g], sacc);
      if (k0 + pitch < vis_max) load_k(k0 + pitch);
      weigh(k0, sacc);
      add_pv();
    }
  }
  // ---- the two wavefronts of a row group add up, and the rows leave as whole lines: a lane holds scattered features of one
  // query, so the sums pass through a patch of rows in LDS.
  float s_mine = 1.f, s_other = 1.f;
  if constexpr (SOFTMAX) {
    if (split == 1) { s_state[qg][0][lane] = m_run; s_state[qg][1][lane] = l_run; }
    __syncthreads();
    if (split == 0) {
      const float m_o = s_state[qg][0][lane], l_o = s_state[qg][1][lane];
      const float m_new = fmaxf(m_run, m_o);
      s_mine = expf(m_run - m_new);
      s_other = expf(m_o - m_new);
      m_run = m_new;
      l_run = l_run * s_mine + l_o * s_other;
    }
  }
  if (split == 0) {
    // what a row's sum is multiplied by, and the weight of its own V row: a candidate is one more key for itself, at distance
    // 0.  (By vector arithmetic on its own rows only: no other candidate's values come near it.)
    float p = 0.f;
    if (it.is_cand) {
      float dot = 0.f;
#pragma unroll
      for (int g = 0; g < NG; ++g) {
        const f32x4 k = row4(Kp + qrow * d, g);
#pragma unroll
        for (int t = 0; t < 4; ++t) dot = fmaf(fq[g][t], k[t], dot);
      }
      const float logit = alpha * pair_sum(dot) + bias[0];
      if constexpr (SOFTMAX) {
        const float z = logit * ts, m_new = fmaxf(m_run, z), sc = expf(m_run - m_new);
        p = expf(z - m_new);
        l_run = l_run * sc + (lhalf == 0 ? p : 0.f);
        s_mine *= sc;
        s_other *= sc;
      } else {
        p = silu_newton(logit);
      }
    }
    float inv = 1.f;
    if constexpr (SOFTMAX) inv = 1.0f / pair_sum(l_run);
    if (lhalf == 0) { s_row[qg][0][l32] = p; s_row[qg][1][l32] = inv; }
  }
  float *patch = s_patch[qg];
#pragma unroll
  for (int b0 = 0; b0 < DB; b0 += DBR) {
    if (b0 > 0) __syncthreads();                     // the round before has left
    if (split == 1) {
#pragma unroll
      for (int e = 0; e < 16; ++e)
#pragma unroll
        for (int b = 0; b < DBR; ++b) patch[l32 * PITCH + DBR * (8 * (e >> 2) + 4 * lhalf + (e & 3)) + b] = oacc[b0 + b][e];
    }
    __syncthreads();
    if (split == 0) {
#pragma unroll
      for (int e = 0; e < 16; ++e)
#pragma unroll
        for (int b = 0; b < DBR; ++b) {
          float *o = patch + l32 * PITCH + DBR * (8 * (e >> 2) + 4 * lhalf + (e & 3)) + b;
          *o = SOFTMAX ? oacc[b0 + b][e] * s_mine + *o * s_other : oacc[b0 + b][e] + *o;
        }
    }
    __syncthreads();
    // 128 threads write the 32 rows of their group, 16 bytes each
    const int rows = min(32, it.n_q - q0);
    for (int i = split * 64 + lane; i < rows * 8 * DBR; i += 128) {
      const int r = i / (8 * DBR), c = 4 * (i % (8 * DBR));                 // floats c .. c + 3 of the patch row
      const int f = DB == DBR ? c : (c / DBR) * DB + b0 + c % DBR;          // the features they are
      const int64_t at = (int64_t)(it.q_row + q0 + r) * d + f;
      f32x4 v = *(const f32x4 *)(patch + r * PITCH + c);
      const float p = s_row[qg][0][r], inv = s_row[qg][1][r];
      if (it.is_cand) {
#pragma unroll
        for (int t = 0; t < 4; ++t) v[t] = fmaf(p, EXACT || f + t < dh ? Vp[at + t] : 0.f, v[t]);
      }
      if constexpr (SOFTMAX) v *= inv;
      float *o = O + h * dh + at;
      if constexpr (EXACT) *(f32x4 *)o = v;
      else {
#pragma unroll
        for (int t = 0; t < 4; ++t)
          if (f + t < dh) o[t] = v[t];
      }
    }
  }
}

void launch_attn_f32(const float *planes, const float *bias_lh, const float *tscale_h, float *O, const AttnItem *items,
                     int n_items, const Shape &sh, hipStream_t s) {
  if (n_items <= 0) return;
  constexpr int kGridY = 32768;        // a launch takes at most 65 535 workgroups along y
  const dim3 grid(sh.H, n_items < kGridY ? n_items : kGridY, (n_items + kGridY - 1) / kGridY);
#define ATTN_CASE(DBV, EX, SM) attn_f32_kernel<DBV, EX, SM><<<grid, 256, 0, s>>>(planes, bias_lh, tscale_h, O, items, n_items, sh.d, sh.dh, sh.D, sh.alpha, sh.ws_rows * sh.d)
#define ATTN_WIDTH(DBV) do { const bool ex = sh.dh == 32 * DBV; \
    if (sh.softmax) { if (ex) ATTN_CASE(DBV, true, true); else ATTN_CASE(DBV, false, true); } \
    else { if (ex) ATTN_CASE(DBV, true, false); else ATTN_CASE(DBV, false, false); } } while (0)
  if (sh.dh <= 32) ATTN_WIDTH(1);
  else if (sh.dh <= 64) ATTN_WIDTH(2);
  else if (sh.dh <= 128) ATTN_WIDTH(4);
  else ATTN_WIDTH(8);
#undef ATTN_WIDTH
#undef ATTN_CASE
}

}  // namespace flame
