// Small bandwidth-bound kernels of the GR forward: input assembly, bias-table expansion,
// LayerNorm * U gating, score head, and the debug evaluation of the mask predicate.
#include <algorithm>

#include "device_common.h"
#include "kernels.h"

namespace flame {

hipError_t raise_lds_limit(const void *kernel, int bytes, std::atomic<uint64_t> &done) {
  int dev = -1;
  if (const hipError_t e = hipGetDevice(&dev); e != hipSuccess) return e;
  const uint64_t bit = dev >= 0 && dev < 64 ? (uint64_t)1 << dev : 0;
  if (done.load() & bit) return hipSuccess;
  const hipError_t e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
  if (e == hipSuccess) done.fetch_or(bit);
  return e;
}

// ---------------------------------------------------------------------------------------------
// Prologue of a pass: what its kernels read that is neither an embedding nor a weight as the caller holds it.  Independent pieces, in one launch, since each alone is a
// few microseconds of launch for next to no work:
//   * plan tables of a small plan, from pinned host memory to the device (larger ones are copied ahead of the launch);
//   * assembly of the token rows;
//   * the projection matrices in the operand layouts of the products;
//   * the bias table by distance, and the logit scales of softmax attention.
// A workgroup does one of them, by its index.
// Before, each was a launch or a copy of its own: 32 x (512 + 128), d = 256, bf16 252 -> 231 us per forward, in fp32 671 -> 656; one request of 64 + 16 in fp32 stays
// at 48 to 55 us, the launches saved going into the split of its weights.
// ---------------------------------------------------------------------------------------------

// Assembly: the token matrix of a request is its history rows followed by its candidate rows
// (Section 2.1: candidates are appended after the behaviour sequence).  A workgroup takes a quarter of a 64-row
// block of the padded workspace, so that a small batch spreads over many compute units; rows past n_valid are zero so that they stay finite downstream.
// fp32 path: X is row-major fp32.  MFMA path: the residual is held as two fp16 words, Xh = fp16(X) (k-tile blocked, the
// projection's operand) and Xl = fp16(X - Xh); embeddings are exact in Xh, so assembly writes Xh only and the first layer
// treats Xl as zero.
constexpr int kSlices = 4;
__device__ __forceinline__ void assemble_f32(const RowBlock rb, int b, int slice, const float *hist, const float *cand, float *X, int d, bool vec) {
  constexpr int rows = kRowAlign / kSlices;
  const int r0 = slice * rows;
  const float *src = (rb.kind ? cand : hist) + ((int64_t)rb.src_row + r0) * d;
  float *dst = X + ((int64_t)b * kRowAlign + r0) * d;
  const int n = rows * d, nv = (rb.n_valid - r0) * d;      // nv <= 0: a slice of padding rows
  if (vec) {                                               // 16 bytes per lane
#pragma unroll 4
    for (int i = threadIdx.x * 4; i < n; i += 1024) {
      f32x4 v = {0.f, 0.f, 0.f, 0.f};
      if (i < nv) v = *(const f32x4 *)(src + i);
      *(f32x4 *)(dst + i) = v;
    }
  } else {
    for (int i = threadIdx.x; i < n; i += 256) dst[i] = i < nv ? src[i] : 0.f;
  }
}

__device__ __forceinline__ void assemble_bf16(const RowBlock rb, int b, int slice, const bf16_t *hist, const bf16_t *cand, half_t *Xh, int d) {
  const bf16_t *src = rb.kind ? cand : hist;
  const int cpr = d / 8;                                   // 16-byte chunks per row
  constexpr int rows = kRowAlign / kSlices;
  const int r0 = slice * rows;
  const int64_t row_base = (int64_t)b * kRowAlign;
#pragma unroll 4
  for (int i = threadIdx.x; i < rows * cpr; i += 256) {
    const int r = r0 + i / cpr, c = i % cpr;
    bf16x8 v;
#pragma unroll
    for (int k = 0; k < 8; ++k) v[k] = (bf16_t)0.f;
    if (r < rb.n_valid) v = *(const bf16x8 *)(src + ((int64_t)rb.src_row + r) * d + c * 8);
    f16x8 o;
#pragma unroll
    for (int k = 0; k < 8; ++k) o[k] = to_f16_sat((float)v[k]);
    *(f16x8 *)(Xh + blocked_index(row_base + r, c * 8, d)) = o;
  }
}

// bf16 -> fp16 copies of the projection matrices.  The MFMA path works on fp16 operands: with eight
// to sixteen layers the 2^-9 rounding of bf16 intermediates alone puts about 1e-2 rms (5e-2 worst
// case) on the scores, fp16's 2^-12 keeps them ten times closer; weights of magnitude >= 2^-14 are
// represented exactly either way.
__device__ __forceinline__ f16x8 to_f16x8(const bf16x8 v) {
  f16x8 o;
#pragma unroll
  for (int k = 0; k < 8; ++k) o[k] = to_f16_sat((float)v[k]);
  return o;
}

// Chunk i (16 bytes) of a matrix packed fragment by fragment (device_common.h): whole lines are written; the reads, two 16-byte pieces of 32 rows per
// fragment, come back from L1 for the fragments of the next k.  planes: the rows are U | V | Q | K of K rows each, layer after layer (V's rows play operand
// B in the projection, all others A).
__device__ __forceinline__ void pack_w(const bf16_t *in, half_t *out, int64_t i, int K, bool planes) {
  const int lane = (int)(i & 63);
  const int64_t f = i >> 6, nb = f / (K / 16);          // fragment, 32-row block
  const int ks = (int)(f % (K / 16));
  const bool plays_a = !(planes && (nb * 32 / K) % 4 == 1);
  const int64_t row = nb * 32 + (plays_a ? sigma32(lane & 31) : lane & 31);
  *(f16x8 *)(out + i * 8) = to_f16x8(*(const bf16x8 *)(in + row * K + ks * 16 + 8 * (lane >> 5)));
}

// Chunk i of the fused K3's copy: W2p[layer][ks][cb][lane][0..7] = W2[32*cb + lane%32][16*ks + 8*(lane/32) + 0..7]
__device__ __forceinline__ void pack_w2(const bf16_t *W2, half_t *W2p, int64_t i, int d) {
  const int64_t per_layer = (int64_t)d * d / 8, l = i / per_layer, c = i % per_layer, t = c >> 6;
  const int lane = (int)(c & 63), cb = (int)(t % (d / 32)), ks = (int)(t / (d / 32));
  *(f16x8 *)(W2p + i * 8) = to_f16x8(*(const bf16x8 *)(W2 + l * d * d + (int64_t)(32 * cb + (lane & 31)) * d + 16 * ks + 8 * (lane >> 5)));
}

// fp32 path: the projection matrices as bf16 parts, fragment by fragment, [matrix][row / 32][k / 16][part][lane][8], 1 KB per fragment; lane l holds k 8 (l / 32) + 0..7
// of row l & 31.  Matrices of d x d, rows and k padded with zeros to multiples of 32: the n1 planes of W1, then W2's matrices.  Item i: 16 bytes of each of the three parts.
__device__ __forceinline__ void split_w(const float *W1, const float *W2, char *out, int64_t i, int n1, int d) {
  const int dp = (d + 31) / 32 * 32, kf = dp / 16;
  const int64_t per = (int64_t)dp * dp / 8;
  const int lane = (int)(i & 63), mat = (int)(i / per);
  const int f = (int)(i % per >> 6), rb = f / kf, ks = f % kf;
  const int row = rb * 32 + (lane & 31), k = ks * 16 + 8 * (lane >> 5);
  const float *src = (mat < n1 ? W1 + (int64_t)mat * d * d : W2 + (int64_t)(mat - n1) * d * d) + (int64_t)row * d;
  f32x4 v[2];
#pragma unroll
  for (int t = 0; t < 8; ++t) v[t >> 2][t & 3] = row < d && k + t < d ? src[k + t] : 0.f;
  const Split3 s0 = split3(v[0]), s1 = split3(v[1]);
  char *dst = out + (((int64_t)mat * per >> 6) + f) * 3072 + lane * 16;
#pragma unroll
  for (int p = 0; p < 3; ++p) {
    *(bf16x4 *)(dst + p * 1024) = s0.p[p];
    *(bf16x4 *)(dst + p * 1024 + 8) = s1.p[p];
  }
}

int64_t split_w_bytes(int d, int n_layers) { const int64_t dp = (d + 31) / 32 * 32; return 5 * n_layers * dp * dp * 6; }

__global__ __launch_bounds__(256) void prologue_kernel(const Prologue p, int wg_tables, int wg_rows, int wg_w, int64_t n_w1, int64_t n_w, bool vec) {
  int wg = blockIdx.x;
  if (wg < wg_tables) {
    const int i = wg * 256 + threadIdx.x;
    if (i < p.n_table_words / 4) ((uint4 *)p.tables_dst)[i] = ((const uint4 *)p.tables_src)[i];
    return;
  }
  wg -= wg_tables;
  if (wg < wg_rows) {
    const int t = wg / kSlices, slice = wg % kSlices;
    const int b = p.list ? p.list[t] : t;
    const RowBlock rb = p.blocks[b];
    if (p.dtype == FLAME_GR_BF16) assemble_bf16(rb, b, slice, (const bf16_t *)p.hist, (const bf16_t *)p.cand, (half_t *)p.Xh, p.d);
    else assemble_f32(rb, b, slice, (const float *)p.hist, (const float *)p.cand, p.X, p.d, vec);
    return;
  }
  wg -= wg_rows;
  if (wg < wg_w) {
    for (int64_t i = (int64_t)wg * 256 + threadIdx.x; i < n_w; i += (int64_t)wg_w * 256) {
      if (p.dtype != FLAME_GR_BF16) split_w((const float *)p.w1, (const float *)p.w2, (char *)p.Ws, i, 4 * p.n_layers, p.d);
      else if (i < n_w1) pack_w((const bf16_t *)p.w1, (half_t *)p.W1h, i, p.d, true);
      else if (p.W2p) pack_w2((const bf16_t *)p.w2, (half_t *)p.W2p, i - n_w1, p.d);
      else pack_w((const bf16_t *)p.w2, (half_t *)p.W2h, i - n_w1, p.d, false);
    }
    return;
  }
  wg -= wg_w;
  // bias[lh][distance] = rab[lh][bucket(distance)]: the attention kernels index the bias by distance (D is a power of two)
  const int step = ((int)gridDim.x - wg_tables - wg_rows - wg_w) * 256, n_lh = p.n_layers * p.H, shift = 31 - __builtin_clz(p.D);
  for (int64_t i = wg * 256 + threadIdx.x; i < (int64_t)n_lh * p.D; i += step)
    p.bias[i] = p.rab[(i >> shift) * p.n_buckets + p.bucket_tab[i & (p.D - 1)]] * p.bias_scale;
  if (p.tscale)
    for (int i = wg * 256 + threadIdx.x; i < n_lh; i += step) p.tscale[i] = p.logit_factor / p.temperature[i];
}

void launch_prologue(const Prologue &p, hipStream_t s) {
  auto workgroups = [](int64_t items, int64_t most) { return (int)std::min((items + 255) / 256, most); };
  const int wg_tables = p.tables_src ? workgroups(p.n_table_words / 4, 1 << 20) : 0, wg_rows = p.n_blk * kSlices;
  int64_t n_w1 = 0, n_w = 0;
  int wg_bias = 0;
  if (p.w1) {
    const int64_t dd8 = (int64_t)p.d * p.d / 8;                       // (MFMA path: d % 64 == 0)
    if (p.dtype == FLAME_GR_BF16) { n_w1 = 4 * p.n_layers * dd8; n_w = 5 * p.n_layers * dd8; }
    else if (p.Ws) n_w = split_w_bytes(p.d, p.n_layers) / 48;
    wg_bias = std::max(1, workgroups((int64_t)p.n_layers * p.H * p.D, 2048));
  }
  const int wg_w = workgroups(n_w, 2048), grid = wg_tables + wg_rows + wg_w + wg_bias;
  if (grid == 0) return;
  const bool vec = p.d % 4 == 0 && ((reinterpret_cast<uintptr_t>(p.hist) | reinterpret_cast<uintptr_t>(p.cand)) & 15u) == 0;
  prologue_kernel<<<grid, 256, 0, s>>>(p, wg_tables, wg_rows, wg_w, n_w1, n_w, vec);
}

// ---------------------------------------------------------------------------------------------
// The candidates' final residual rows, in candidate order (the input of a fusion / head stage).
// ---------------------------------------------------------------------------------------------
// Xh != nullptr: the residual is the pair (Xh blocked, Xl row-major) of the MFMA path (d a multiple of 8 there, 16-byte loads), else fp32 X.
// Four row slices per block, so that a batch of a hundred blocks fills the chip: memory latency bounds it.  128 blocks, d = 192: 21 -> 4.7 us
// against one workgroup per block and one element per lane.
__global__ __launch_bounds__(256) void gather_hidden_kernel(const float *__restrict__ X, const half_t *__restrict__ Xh,
                                                            const half_t *__restrict__ Xl, const RowBlock *__restrict__ blocks,
                                                            const int32_t *__restrict__ cand_blocks, float *__restrict__ hidden, int d) {
  const int b = cand_blocks[blockIdx.x];
  const RowBlock rb = blocks[b];
  const int rows = kRowAlign / gridDim.y, r0 = blockIdx.y * rows;
  const int n = (min(rb.n_valid, r0 + rows) - r0) * d;       // <= 0: a slice of padding rows
  const int64_t row0 = (int64_t)b * kRowAlign + r0;
  float *dst = hidden + ((int64_t)rb.src_row + r0) * d;
  if (Xh) {
    const bool vec = (reinterpret_cast<uintptr_t>(hidden) & 15u) == 0;      // the caller's array; d % 8 == 0 keeps its rows on 16 bytes
#pragma unroll 4
    for (int i = threadIdx.x * 8; i < n; i += 2048) {
      const f16x8 h = *(const f16x8 *)(Xh + blocked_index(row0 + i / d, i % d, d)), l = *(const f16x8 *)(Xl + row0 * d + i);
      f32x4 o[2];
#pragma unroll
      for (int k = 0; k < 8; ++k) o[k >> 2][k & 3] = (float)h[k] + (float)l[k];
      if (vec) {
        *(f32x4 *)(dst + i) = o[0];
        *(f32x4 *)(dst + i + 4) = o[1];
      } else {
#pragma unroll
        for (int k = 0; k < 8; ++k) dst[i + k] = o[k >> 2][k & 3];
      }
    }
  } else {
    for (int i = threadIdx.x; i < n; i += 256) dst[i] = X[row0 * d + i];
  }
}

void launch_gather_hidden(const float *X, const void *Xh, const void *Xl, const RowBlock *blocks, const int32_t *cand_blocks, int n_cblk,
                          float *hidden, int d, hipStream_t s) {
  if (n_cblk > 0) gather_hidden_kernel<<<dim3(n_cblk, 4), 256, 0, s>>>(X, (const half_t *)Xh, (const half_t *)Xl, blocks, cand_blocks, hidden, d);
}

// Debug capture: the residual rows [row_begin, row_end) of the MFMA path as fp32 (Xh + Xl, exact).
__global__ __launch_bounds__(256) void residual_to_f32_kernel(const half_t *__restrict__ Xh, const half_t *__restrict__ Xl,
                                                              float *__restrict__ out, int64_t first, int64_t n, int d) {
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
    const int64_t e = first + i;
    out[e] = (float)Xh[blocked_index(e / d, (int)(e % d), d)] + (float)Xl[e];
  }
}

void launch_residual_to_f32(const void *Xh, const void *Xl, float *out, int64_t row_begin, int64_t row_end, int d, hipStream_t s) {
  const int64_t n = (row_end - row_begin) * d;
  if (n <= 0) return;
  const int grid = (int)((n + 255) / 256 > 4096 ? 4096 : (n + 255) / 256);
  residual_to_f32_kernel<<<grid, 256, 0, s>>>((const half_t *)Xh, (const half_t *)Xl, out, row_begin * d, n, d);
}

// ---------------------------------------------------------------------------------------------
// G = (LayerNorm_d(O) * gamma + beta) * U.  One wavefront per row, statistics in fp32 by wavefront
// reduction (mean first, then the centred second moment: biased variance).
// ---------------------------------------------------------------------------------------------
template <typename T, typename TW, int MAXV>   // T: activations (O, U, G); TW: stored weights (gamma, beta)
__global__ __launch_bounds__(256) void ln_gate_kernel(const T *__restrict__ O, const T *__restrict__ U,
                                                      const TW *__restrict__ gamma, const TW *__restrict__ beta,
                                                      T *__restrict__ G, const RowBlock *__restrict__ blocks,
                                                      const int32_t *__restrict__ blk_list, int blk_first, int d,
                                                      float eps) {
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int rb = blockIdx.x >> 4;                       // 16 workgroups of 4 rows per 64-row block
  const int blk = blk_list ? blk_list[rb] : blk_first + rb;
  const int in_blk = (blockIdx.x & 15) * 4 + wave;
  const int64_t row = (int64_t)blk * kRowAlign + in_blk;
  if (in_blk >= blocks[blk].n_valid) {                  // padding row: keep it finite (zero branch)
    for (int k = lane; k < d; k += 64) G[row * d + k] = from_f32<T>(0.f);
    return;
  }
  const T *o = O + row * d;
  float v[MAXV];
  float sum = 0.f;
#pragma unroll
  for (int i = 0; i < MAXV; ++i) {
    const int k = lane + i * 64;
    v[i] = k < d ? to_f32(o[k]) : 0.f;
    sum += v[i];
  }
  const float mu = wave_sum(sum) / (float)d;
  float sq = 0.f;
#pragma unroll
  for (int i = 0; i < MAXV; ++i) {
    const int k = lane + i * 64;
    const float c = k < d ? v[i] - mu : 0.f;
    sq += c * c;
  }
  const float rstd = rsqrtf(wave_sum(sq) / (float)d + eps);
#pragma unroll
  for (int i = 0; i < MAXV; ++i) {
    const int k = lane + i * 64;
    if (k < d) {
      const float y = ((v[i] - mu) * rstd * to_f32(gamma[k]) + to_f32(beta[k])) * to_f32(U[row * d + k]);
      G[row * d + k] = from_f32<T>(y);
    }
  }
}

template <typename T, typename TW>
static void ln_gate_dispatch(const void *O, const void *U, const void *g, const void *b, void *G,
                             const RowBlock *blocks, const int32_t *blk_list, int n_blk, int blk_first, int d, float eps, hipStream_t s) {
  const int grid = n_blk * 16;
#define LN_CASE(MV) ln_gate_kernel<T, TW, MV><<<grid, 256, 0, s>>>((const T *)O, (const T *)U, (const TW *)g, (const TW *)b, (T *)G, blocks, blk_list, blk_first, d, eps)
  if (d <= 64) LN_CASE(1);
  else if (d <= 128) LN_CASE(2);
  else if (d <= 256) LN_CASE(4);
  else if (d <= 512) LN_CASE(8);
  else if (d <= 1024) LN_CASE(16);
  else LN_CASE(64);
#undef LN_CASE
}

void launch_ln_gate(const void *O, const void *U, const void *gamma, const void *beta, void *G,
                    const RowBlock *blocks, const int32_t *blk_list, int n_blk, int blk_first, int d, float eps, hipStream_t s) {
  if (n_blk <= 0) return;
  ln_gate_dispatch<half_t, bf16_t>(O, U, gamma, beta, G, blocks, blk_list, n_blk, blk_first, d, eps, s);
}

// ---------------------------------------------------------------------------------------------
// Score head: one logit per candidate row, written in the caller's candidate order.
// ---------------------------------------------------------------------------------------------
template <typename T>
__global__ __launch_bounds__(256) void score_kernel(const float *__restrict__ X, const half_t *__restrict__ Xh,
                                                    const half_t *__restrict__ Xl, const T *__restrict__ w_s, float b_s,
                                                    const RowBlock *__restrict__ blocks, const int32_t *__restrict__ cblk,
                                                    float *__restrict__ scores, int d) {
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int blk = cblk[blockIdx.x >> 4];
  const RowBlock rb = blocks[blk];
  const int i = (blockIdx.x & 15) * 4 + wave;
  if (i >= rb.n_valid) return;
  const int64_t row = (int64_t)blk * kRowAlign + i;
  float acc = 0.f;
  if constexpr (sizeof(T) == 2) {
    // MFMA path: 8 features per lane and step, 16-byte loads (8 consecutive k sit together in the blocked word too)
    for (int k = lane * 8; k < d; k += 512) {
      const f16x8 h8 = *(const f16x8 *)(Xh + blocked_index(row, k, d)), l8 = *(const f16x8 *)(Xl + row * d + k);
      const bf16x8 w8 = *(const bf16x8 *)(w_s + k);
#pragma unroll
      for (int q = 0; q < 8; ++q) acc += ((float)h8[q] + (float)l8[q]) * (float)w8[q];
    }
  } else {
    for (int k = lane; k < d; k += 64) acc += X[row * d + k] * to_f32(w_s[k]);
  }
  acc = wave_sum(acc);
  if (lane == 0) scores[rb.src_row + i] = acc + b_s;
}

void launch_scores(int dtype, const float *X, const void *Xh, const void *Xl, const void *w_s, float b_s, const RowBlock *blocks,
                   const int32_t *cand_blocks, int n_cblk, float *scores, int d, hipStream_t s) {
  if (n_cblk <= 0) return;
  if (dtype == FLAME_GR_BF16)
    score_kernel<bf16_t><<<n_cblk * 16, 256, 0, s>>>(nullptr, (const half_t *)Xh, (const half_t *)Xl, (const bf16_t *)w_s, b_s, blocks, cand_blocks, scores, d);
  else
    score_kernel<float><<<n_cblk * 16, 256, 0, s>>>(X, nullptr, nullptr, (const float *)w_s, b_s, blocks, cand_blocks, scores, d);
}

// ---------------------------------------------------------------------------------------------
// Helpers of the entry point that works in a static workspace (no allocation, no copies): the bucket
// table computed on the device, plan tables delivered as kernel arguments, and the spare rows behind
// a batch cleared (whole-tile key loads may read them; they must hold finite values).
// ---------------------------------------------------------------------------------------------
__device__ __forceinline__ int ilog2_dev(int v) { return 31 - __builtin_clz(v); }

// Same integers as the host planner's bucket function (documented in flame_gr.h).
__global__ __launch_bounds__(256) void bucket_table_kernel(int nb, int D, int32_t *__restrict__ out) {
  const int half = nb / 2;
  const int lo = ilog2_dev(half), hi = ilog2_dev(D);
  const int octaves = hi > lo ? hi - lo : 0;
  int sub = lo;
  while (sub > 0 && octaves * (1 << sub) > half) --sub;
  for (int t = blockIdx.x * 256 + threadIdx.x; t < D; t += gridDim.x * 256) {
    int b = t;
    if (t >= half) {
      const int oct = ilog2_dev(t);
      b = half + (oct - lo) * (1 << sub) + ((t - (1 << oct)) >> (oct - sub));
    }
    out[t] = b;
  }
}

void launch_bucket_table(int n_buckets, int D, int32_t *out, hipStream_t s) {
  const int grid = (D + 255) / 256 > 64 ? 64 : (D + 255) / 256;
  bucket_table_kernel<<<grid, 256, 0, s>>>(n_buckets, D, out);
}

__global__ __launch_bounds__(256) void upload_words_kernel(UploadWords src, int n, uint32_t *__restrict__ dst) {
  for (int i = threadIdx.x; i < n; i += 256) dst[i] = src.w[i];
}

void launch_upload_words(const void *host_src, size_t bytes, void *dst, hipStream_t s) {
  const uint32_t *src = (const uint32_t *)host_src;
  uint32_t *out = (uint32_t *)dst;
  size_t n = bytes / 4;                        // every plan table is an array of 32-bit integers
  while (n > 0) {
    UploadWords u;
    const int m = (int)(n < (size_t)UploadWords::kWords ? n : (size_t)UploadWords::kWords);
    for (int i = 0; i < m; ++i) u.w[i] = src[i];
    upload_words_kernel<<<1, 256, 0, s>>>(u, m, out);
    src += m; out += m; n -= m;
  }
}

// K plane rows [row0, row0 + n) and the same token columns of the feature-major V plane <- 0
__global__ __launch_bounds__(256) void clear_spare_kernel(half_t *__restrict__ K, half_t *__restrict__ Vt, int d, int64_t ws_rows,
                                                          int64_t row0, int n) {
  const int64_t total = (int64_t)n * d;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < total; i += (int64_t)gridDim.x * 256) {
    K[row0 * d + i] = (half_t)0.f;
    Vt[(i / n) * ws_rows + row0 + i % n] = (half_t)0.f;
  }
}

void launch_clear_spare(void *K, void *Vt, int d, int64_t ws_rows, int64_t row0, int n, hipStream_t s) {
  if (n <= 0) return;
  const int64_t total = (int64_t)n * d;
  const int grid = (int)((total + 255) / 256 > 1024 ? 1024 : (total + 255) / 256);
  clear_spare_kernel<<<grid, 256, 0, s>>>((half_t *)K, (half_t *)Vt, d, ws_rows, row0, n);
}

// ---------------------------------------------------------------------------------------------
// Debug: the mask predicate and bucket table as the attention kernels see them.
// ---------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void debug_mask_kernel(int L, int M, const int32_t *__restrict__ tab, int D,
                                                         uint8_t *__restrict__ mask, int32_t *__restrict__ bucket) {
  const int N = L + M;
  const int64_t total = (int64_t)N * N;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < total; i += (int64_t)gridDim.x * 256) {
    const int r = (int)(i / N), c = (int)(i % N);
    const int is_cand = r >= L;
    const int q_index = is_cand ? L : r;
    bool ok;
    int delta;
    if (c < L) {
      ok = c < visible_history(is_cand, q_index, L);
      delta = q_index - c;
    } else {
      ok = is_cand && c == r;   // among candidate keys a candidate sees itself only
      delta = 0;
    }
    mask[i] = ok ? 1 : 0;
    if (bucket) bucket[i] = ok ? tab[delta < D ? delta : D - 1] : -1;
  }
}

void launch_debug_mask(int L, int M, const int32_t *bucket_tab, int D, uint8_t *mask, int32_t *bucket, hipStream_t s) {
  const int64_t total = (int64_t)(L + M) * (L + M);
  if (total == 0) return;
  int grid = (int)((total + 255) / 256 > 4096 ? 4096 : (total + 255) / 256);
  debug_mask_kernel<<<grid, 256, 0, s>>>(L, M, bucket_tab, D, mask, bucket);
}

}  // namespace flame
