// K3 of the GR block, fused: X <- X + (LayerNorm_d(O) * U) W2^T + b2.
//
// The residual stream X lives in HBM as two fp16 words per element: Xh = fp16(X), the k-tile blocked operand copy that the
// next layer's projection reads anyway, and Xl = fp16(X - Xh) (row-major), together 22 significant bits, so that
// this kernel reads 4 and writes 4 bytes per element instead of reading 4 and writing 6 (fp32 X plus the operand copy).
//
// LayerNorm, the U gate, the output projection and the residual run in one kernel (the fusion of
// layer normalisation with the following linear projection that Section 3.2 describes), so the
// gated activations never travel through HBM.  The kernel is HBM-bound by construction (per row it
// must read O and U and read-modify-write X: 12 bytes per element against 2*d flops), so the
// design aims at streaming, not at MFMA utilisation:
//   * one workgroup = one 64-row block of the workspace, all d output features (d <= 512 per pass);
//   * phase 1: each wavefront normalises 16 rows (one row per wavefront-wide 16-byte load, statistics
//     by wavefront reduction in fp32: mean, then centred second moment) and writes the gated fp16 rows
//     into LDS, 16-byte chunks XOR-swizzled with the row's low four bits so that the MFMA operand reads are
//     conflict free (the LDS serves 16 lanes x 16 bytes per clock from 64 banks);
//   * phase 2: each wavefront owns d/4 output features; the W2 operand comes straight from L2 in a
//     fragment-major packed layout (one coalesced 1 KB read per MFMA operand, prepared once per forward
//     by the prologue), so LDS holds only the activations and two workgroups fit on a CU;
//   * phase 3: residual add in fp32 (X = Xh + Xl, exact in fp32) and split into the two fp16 words again, after a
//     transposition of the accumulators through LDS so that the residual is read and written in whole lines.
#include "device_common.h"
#include "kernels.h"

namespace flame {

namespace {

// NWV wavefronts per workgroup, NBW 32-feature blocks per wavefront: d = 32 * NBW * NWV (four wavefronts for
// d = 128, 256, 512; three for d = 96, 192, 384; twice as many for d = 384 and 512 where a workgroup has a compute unit to itself).  A workgroup takes RH 32-row halves of a 64-row block; its rows are dealt out
// RPW per wavefront in phase 1 (with three wavefronts the last one has rows to spare, which it skips).
// CS workgroups share the rows (blockIdx.y): each repeats phase 1 and takes 1/CS of every wavefront's feature
// blocks through phases 2 and 3.  RH = 2, CS = 1 is for launches that fill the chip.  RH = 1 and CS > 1 are for launches with few
// row blocks, where a workgroup sits alone on its CU and its run time, not the chip's bandwidth, is what counts: half the
// rows are one round of loads per wavefront, and everything that does not depend on phase 1 (the first W2 fragments, the
// residual rows) is requested ahead of it.  Every output element is computed exactly as with RH = 2, CS = 1.
// NT: O, U and the residual pair bypass the caches (consumed once; data of this size would push W2's fragments and K1's operands
// out of L2).  Small batches are better off leaving them there for the next kernel (see launch_k3).
// k3_dense: half blocks with uncut features are for a few hundred row blocks, more than two workgroups per CU.  Three wavefronts per SIMD hold
// them all at once, where two run a second, nearly empty round; the registers for that come from the residual rows, which are
// requested behind phase 1 instead of ahead of it, and a shorter W2 ring.  384 row blocks, two wavefronts against three: d = 256 24.0 -> 20.1 us, d = 192
// 25.2 -> 19.8 us per launch.
constexpr bool k3_dense(int nwv, int cs, int rh, int nbw) { return nwv < 6 && rh == 1 && cs == 1 && nbw == 2; }
template <int NWV, int NBW, int CS, int RH, bool NT>
__global__ __launch_bounds__(64 * NWV, k3_dense(NWV, CS, RH, NBW) ? 3 : 2) void k3_fused_kernel(const half_t *__restrict__ O, const half_t *__restrict__ U,
                                                          const bf16_t *__restrict__ gamma, const bf16_t *__restrict__ beta,
                                                          const half_t *__restrict__ W2p, const bf16_t *__restrict__ b2,
                                                          half_t *__restrict__ Xh, half_t *__restrict__ Xl, int lo_is_zero,
                                                          const RowBlock *__restrict__ blocks, const int32_t *__restrict__ blk_list,
                                                          int blk_first, float eps) {
  constexpr int d = 32 * NBW * NWV;
  constexpr int ROWS = 32 * RH;                  // rows of this workgroup
  constexpr int RB4 = 4;                         // rows per batch of phase 1
  constexpr int RPW = (ROWS + NWV * RB4 - 1) / (NWV * RB4) * RB4;   // rows per wavefront in phase 1 (with three wavefronts a few too many)
  constexpr bool EVEN = RPW * NWV == ROWS;
  constexpr bool EARLY = RH == 1;                // requests that do not wait for phase 1 go out ahead of it
  constexpr bool DENSE = k3_dense(NWV, CS, RH, NBW);  // (but the residual behind it)
  constexpr int NCHUNK = d / 8;                  // 16-byte chunks per row
  // Swizzle key of the gated rows in LDS.  A row of d fp16 is NCHUNK chunks; the MFMA operand reads take one chunk
  // column of 16 consecutive rows.  With NCHUNK a multiple of 16 the row pitch is a multiple of 256 bytes and the
  // low four row bits spread those reads over the 16 slots; with NCHUNK = 24 (d = 192, pitch 384 bytes: odd and
  // even rows already sit 128 bytes apart) three bits of row / 2 do, and the XOR stays inside a group of 8 chunks.
  auto gkey = [](int r) { return NCHUNK % 16 == 0 ? r & 15 : (r >> 1) & 7; };
  constexpr int CPL = (NCHUNK + 63) / 64;        // chunks per lane in phase 1
  extern __shared__ __attribute__((aligned(16))) char smem[];   // sG: ROWS x d fp16, swizzled

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, lhalf = lane >> 5;
  const int bx = RH == 2 ? (int)blockIdx.x : (int)blockIdx.x >> 1, half0 = RH == 2 ? 0 : (int)blockIdx.x & 1;
  const int blk = blk_list ? blk_list[bx] : blk_first + bx;
  const int n_valid = blocks[blk].n_valid - 32 * half0;
  const int64_t row0 = (int64_t)blk * kRowAlign + 32 * half0;

  // ---- phase 1: G = (LN(O) * gamma + beta) * U -> LDS
  // Rows are taken four at a time, and the loads of the next four are issued before the current
  // four are normalised: with one row in flight per wavefront the kernel would run at the latency,
  // not the bandwidth, of HBM.
  f16x8 ov[2][RB4][CPL], uv[2][RB4][CPL];
  auto issue = [&](int set, int batch) {
#pragma unroll
    for (int q = 0; q < RB4; ++q)
#pragma unroll
      for (int c = 0; c < CPL; ++c) {
        const int ch = lane + 64 * c;
        if (ch < NCHUNK) {
          const int rr = wave * RPW + batch * RB4 + q;
          const int64_t off = (row0 + (EVEN || rr < ROWS ? rr : ROWS - 1)) * d + ch * 8;
          ov[set][q][c] = load_once<NT>((const f16x8 *)(O + off));
          uv[set][q][c] = load_once<NT>((const f16x8 *)(U + off));
        }
      }
  };
  float g[CPL][8], bt[CPL][8];
  auto load_affine = [&]() {
#pragma unroll
    for (int c = 0; c < CPL; ++c) {
      const int ch = lane + 64 * c;
      if (ch < NCHUNK) {
        const bf16x8 gv = *(const bf16x8 *)(gamma + ch * 8), bv = *(const bf16x8 *)(beta + ch * 8);
#pragma unroll
        for (int k = 0; k < 8; ++k) { g[c][k] = (float)gv[k]; bt[c][k] = (float)bv[k]; }
      }
    }
  };
  if (!EARLY) load_affine();
  issue(0, 0);
  if (EARLY && RPW / RB4 > 1) issue(1, 1);

  static_assert(NBW % CS == 0, "feature blocks of a wavefront divide among the workgroups of a row block");
  constexpr int NB2 = NBW / CS;                  // feature blocks per wavefront in this workgroup
  const int fb0 = wave * NBW + (CS > 1 ? (int)blockIdx.y * NB2 : 0);   // first of them
  constexpr int NKS = d / 16;
  // The W2 fragments come from L2, whose latency is several times the 8 MFMAs of a k-step: they are requested
  // PD - 1 k-steps ahead into a register ring (scheduling barriers keep the compiler from sinking the requests
  // back to their first use); the activations come from LDS, one step ahead.
  constexpr int PD = !EARLY || DENSE || NB2 > 2 ? 4 : NKS % 8 == 0 ? 8 : 4;
  static_assert(NKS % PD == 0, "k-steps are walked in groups of the ring depth");
  const half_t *wp = W2p + ((int64_t)fb0 * 64 + lane) * 8;      // + (ks * (d/32) + j) * 512
  f16x8 fw[PD][NB2], fa[2][RH];
  auto first_w2 = [&]() {
#pragma unroll
    for (int p = 0; p < PD - 1; ++p)
#pragma unroll
      for (int j = 0; j < NB2; ++j) fw[p][j] = *(const f16x8 *)(wp + ((int64_t)p * (d / 32) + j) * 512);
  };
  constexpr int WF = 32 * NB2;                      // features per wavefront (in this workgroup)
  constexpr int CPR = WF / 4;                       // 16-byte fp32 chunks per patch row
  constexpr int RPI = 64 / CPR;                     // patch rows per instruction
  constexpr int NIT = 32 / RPI;
  constexpr int XB = NIT < 8 ? NIT : 8;             // residual rows requested ahead
  const int rl = lane / CPR, cc = lane % CPR;
  const int n = fb0 * 32 + 4 * cc;                  // this lane's 4 features in the read-out
  // lo_is_zero: the first layer, whose input rows are embeddings (exact in Xh): Xl is not read, only written
  f16x4 xh[XB], xl[XB];
  auto load_x = [&](int i, int t, int it) {
    const int64_t m = row0 + 32 * i + rl + (int64_t)it * RPI;
    xh[t] = load_once<NT>((const f16x4 *)(Xh + blocked_index(m, n, d)));
    xl[t] = f16x4{(half_t)0.f, (half_t)0.f, (half_t)0.f, (half_t)0.f};
    if (!lo_is_zero) xl[t] = load_once<NT>((const f16x4 *)(Xl + m * d + n));
  };
  if (EARLY) {
    __builtin_amdgcn_sched_barrier(0);
    first_w2();
    if (!DENSE) {
#pragma unroll
      for (int t = 0; t < XB; ++t) load_x(0, t, t);
    }
    __builtin_amdgcn_sched_barrier(0);
  }
  if (EARLY) load_affine();
#pragma unroll
  for (int batch = 0; batch < RPW / RB4; ++batch) {
    const int set = batch & 1;
    if (batch + 1 < RPW / RB4 && !(EARLY && batch == 0)) issue(set ^ 1, batch + 1);
    __builtin_amdgcn_sched_barrier(0);
    // the four rows go through each step together, so that their reduction chains overlap
    float v[RB4][CPL][8], mu[RB4], rstd[RB4];
#pragma unroll
    for (int q = 0; q < RB4; ++q) {
      float sum = 0.f;
#pragma unroll
      for (int c = 0; c < CPL; ++c)
#pragma unroll
        for (int k = 0; k < 8; ++k) {
          v[q][c][k] = lane + 64 * c < NCHUNK ? (float)ov[set][q][c][k] : 0.f;
          sum += v[q][c][k];
        }
      mu[q] = sum;
    }
#pragma unroll
    for (int q = 0; q < RB4; ++q) mu[q] = wave_sum(mu[q]) * (1.0f / d);
#pragma unroll
    for (int q = 0; q < RB4; ++q) {
      float sq = 0.f;
#pragma unroll
      for (int c = 0; c < CPL; ++c)
        if (lane + 64 * c < NCHUNK) {
#pragma unroll
          for (int k = 0; k < 8; ++k) { const float t = v[q][c][k] - mu[q]; sq += t * t; }
        }
      rstd[q] = sq;
    }
#pragma unroll
    for (int q = 0; q < RB4; ++q) rstd[q] = rsqrtf(wave_sum(rstd[q]) * (1.0f / d) + eps);
#pragma unroll
    for (int q = 0; q < RB4; ++q) {
      const int r = wave * RPW + batch * RB4 + q;
      if (!EVEN && r >= ROWS) continue;            // a spare row of the last wavefront
      const bool pad = r >= n_valid;               // padding rows carry a zero branch so that they stay finite
#pragma unroll
      for (int c = 0; c < CPL; ++c) {
        const int ch = lane + 64 * c;
        if (ch < NCHUNK) {
          f16x8 o;
#pragma unroll
          for (int k = 0; k < 8; ++k)
            o[k] = pad ? (half_t)0.f : to_f16_sat(((v[q][c][k] - mu[q]) * rstd[q] * g[c][k] + bt[c][k]) * (float)uv[set][q][c][k]);
          *(f16x8 *)(smem + r * (d * 2) + ((ch ^ gkey(r)) << 4)) = o;
        }
      }
    }
    __builtin_amdgcn_sched_barrier(0);
  }
  __syncthreads();

  // ---- phase 2: acc[token][feature] over k; features of this wavefront: fb0 * 32 .. + 32 * NB2 - 1
  f32x16 acc[RH][NB2];
#pragma unroll
  for (int i = 0; i < RH; ++i)
#pragma unroll
    for (int j = 0; j < NB2; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;
  if (!EARLY) first_w2();
  if (DENSE) {
#pragma unroll
    for (int t = 0; t < XB; ++t) load_x(0, t, t);
    __builtin_amdgcn_sched_barrier(0);
  }
#pragma unroll
  for (int i = 0; i < RH; ++i) {
    const int r = 32 * i + l32;
    fa[0][i] = *(const f16x8 *)(smem + r * (d * 2) + ((lhalf ^ gkey(r)) << 4));
  }
  __builtin_amdgcn_sched_barrier(0);
  for (int ks0 = 0; ks0 < NKS; ks0 += PD) {
#pragma unroll
    for (int u = 0; u < PD; ++u) {
      const int ks = ks0 + u;
      const int cur = u & 1, nxt = cur ^ 1;
      const int kw = ks + PD - 1 < NKS ? ks + PD - 1 : NKS - 1;
      const int kn = ks + 1 < NKS ? ks + 1 : ks;
#pragma unroll
      for (int j = 0; j < NB2; ++j) fw[(u + PD - 1) % PD][j] = *(const f16x8 *)(wp + ((int64_t)kw * (d / 32) + j) * 512);
#pragma unroll
      for (int i = 0; i < RH; ++i) {
        const int r = 32 * i + l32;
        fa[nxt][i] = *(const f16x8 *)(smem + r * (d * 2) + (((2 * kn + lhalf) ^ gkey(r)) << 4));
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = 0; i < RH; ++i)
#pragma unroll
        for (int j = 0; j < NB2; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(fw[u][j], fa[cur][i], acc[i][j], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    }
  }

  // ---- phase 3: residual.  In the accumulators a lane holds one token and scattered features, and only
  // two lanes share a row, so direct X accesses would be 32-byte pieces (the memory path is bound by the
  // number of requests, not only by bytes).  Each wavefront passes its 32 x (32 NBW) patch through a
  // private slice of the now free LDS (16-byte chunks XOR-swizzled by row) and then walks it row by
  // row: 16 bytes per lane, whole lines of X, 64-byte runs of the blocked fp16 copy.
  __syncthreads();                                  // every wavefront has finished reading G
  char *pb = smem + wave * (32 * WF * 4);
  // chunk XOR key: 16 consecutive rows of one chunk column use each of the 16 slots of 256 bytes once
  auto pkey = [](int row) { return CPR == 8 ? (row >> 1) & 7 : row & 15; };
  f32x4 bvf;
  {
    const bf16x4 bv = *(const bf16x4 *)(b2 + n);
#pragma unroll
    for (int q = 0; q < 4; ++q) bvf[q] = (float)bv[q];
  }
#pragma unroll
  for (int i = 0; i < RH; ++i) {
    if (!EARLY) {
#pragma unroll
      for (int t = 0; t < XB; ++t) load_x(i, t, t);
    }
#pragma unroll
    for (int j = 0; j < NB2; ++j)
#pragma unroll
      for (int gq = 0; gq < 4; ++gq) {
        const int c = 8 * j + 2 * gq + lhalf;
        const f32x4 v = {acc[i][j][4 * gq], acc[i][j][4 * gq + 1], acc[i][j][4 * gq + 2], acc[i][j][4 * gq + 3]};
        *(f32x4 *)(pb + l32 * (WF * 4) + ((c ^ pkey(l32)) << 4)) = v;
      }
#pragma unroll
    for (int it = 0; it < NIT; ++it) {
      const int row = it * RPI + rl;
      const f32x4 v = *(const f32x4 *)(pb + row * (WF * 4) + ((cc ^ pkey(row)) << 4));
      const f16x4 h4 = xh[it % XB], l4 = xl[it % XB];
      if (it + XB < NIT) load_x(i, it % XB, it + XB);
      f16x4 oh, ol;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const float x = ((float)h4[q] + (float)l4[q]) + (v[q] + bvf[q]);
        oh[q] = to_f16_sat(x);
        ol[q] = to_f16_sat(x - (float)oh[q]);
      }
      const int64_t m = row0 + 32 * i + row;
      store_once<NT>(oh, (f16x4 *)(Xh + blocked_index(m, n, d)));
      store_once<NT>(ol, (f16x4 *)(Xl + m * d + n));
    }
  }
}

}  // namespace

// the gated rows, and after them a 32-row fp32 patch of every wavefront's features
static size_t k3_lds_bytes(int d, int cs, int rh) { const size_t g = (size_t)32 * rh * d * 2, patch = (size_t)32 * (d / cs) * 4; return g > patch ? g : patch; }

bool k3_fused_supported(int d) { return d == 128 || d == 192 || d == 256 || d == 384 || d == 512; }

// Few row blocks: half blocks, with the features cut as long as that leaves one workgroup per compute unit at most (lone workgroups,
// latency), then half blocks with uncut features.  Microseconds per launch, whole blocks / half blocks / half blocks with features cut
// in two / in four, all with three or four wavefronts:
//   d = 512: 16 blocks 21.1 / 15.8 / 12.0 / 10.1, 64: 22.6 / 17.1 / 13.2 / 13.9, 66: 22.1 / 16.1, 128: 24.1 / 18.6 / 22.3 / 21.6, 256: 28.5 / 26.9
//   d = 384: 16: 25.4 / - / - / 12.2, 64: 26.1 / - / 14.2, 66: 26.7 / 16.5, 256: 29.8 / 23.9
//   d = 256: 16: 16.4 / 11.0 / 9.8, 64: 17.2 / 11.6 / 10.9, 66: 17.1 / 11.7, 128: 18.1 / 12.7, 256: 19.2 / 16.2
//   d = 192: 16: 20.0 / 12.4 / 11.5, 64: 20.5 / 12.9 / 12.0, 66: 20.4 / 13.0, 256: 21.7 / 16.0
//   d = 128 (one feature block per wavefront, never cut): 16: 13.9 / 9.6, 256: 15.6 / 12.5
// d = 384 and 512: a workgroup alone on its compute unit leaves each SIMD one wavefront; with six or eight of them half as wide the rows' phase is half as long and two
// wavefronts share a SIMD.  Forwards of 8 layers, three or four wavefronts (by the rule above) / twice as many, features cut in two / uncut (us):
//   d = 512: 22 blocks 242.6 / 242.6 / 263.9, 25: 256.9 / 251.4 / 275.8, 36: 326 / 315 / 335, 60: 449 / 438 / 456, 70: 382 / 394 / 365, 110: 446 / 462 / 432, 150: 574 / 600 / 584
//   d = 384: 10: 204 / 196 / 214, 40: 320 / 302 / 320, 64: 405 / 385 / 405, 70: 339 / 355 / 320, 110: 383 / 406 / 367, 150: 450 / 498 / 472
// Past kK3HalfBlocks = 384 row blocks, three workgroups for each of the 256 compute units, a fourth has to wait its turn:
//   384 / 386 / 448 blocks: d = 128 17.4 / 16.5, 17.5 / 18.3, 17.7 / 18.4;  d = 256 23.5 / 20.1, 23.4 / 23.3, 24.2 / 24.6;
//   d = 384 36.7 / 35.2, 37.3 / 38.4, 38.2 / 40.2;  d = 512 38.2 / 39.1, 38.3 / 43.6, 40.9 / 46.0
// (d = 192, whose workgroups have three wavefronts and find room for a fourth, keeps the common limit although half blocks measure ahead beyond
// it: 448 25.8 / 22.4, 640 32.4 / 28.0, 1024 44.2 / 38.5, 1536 52.8 / 52.5, 2048 68.4 / 69.1.)
// Whole blocks also where the launch streams (kStreamBytes): from 257 blocks at d = 512 and 342 at d = 384, where the two are
// level (d = 512: 258 37.6 / 37.0, 342 37.8 / 37.6; d = 384: 342 36.0 / 34.0); at those widths no whole block reads through the caches.
template <int NWV, int NB>
static void launch_k3(const half_t *O, const half_t *U, const bf16_t *gamma, const bf16_t *beta, const half_t *W2p, const bf16_t *b2, half_t *Xh, half_t *Xl,
                      int lo_is_zero, const RowBlock *blocks, const int32_t *blk_list, int n_blk, int blk_first, float eps, hipStream_t s) {
  constexpr int d = 32 * NB * NWV;
  const bool nt = (int64_t)n_blk * kRowAlign * d * 2 > kStreamBytes;
#define K3_LAUNCH(CSV, RHV, NTV) k3_fused_kernel<NWV, NB, CSV, RHV, NTV><<<dim3(n_blk * (3 - RHV), CSV), 64 * NWV, k3_lds_bytes(d, CSV, RHV), s>>>( \
    O, U, gamma, beta, W2p, b2, Xh, Xl, lo_is_zero, blocks, blk_list, blk_first, eps)
  if constexpr (NB == 4) {
#define K3_WIDE(CSV) k3_fused_kernel<2 * NWV, 2, CSV, 1, false><<<dim3(2 * n_blk, CSV), 128 * NWV, k3_lds_bytes(d, CSV, 1), s>>>( \
    O, U, gamma, beta, W2p, b2, Xh, Xl, lo_is_zero, blocks, blk_list, blk_first, eps)
    if (d == 512 && n_blk <= kK3CutInFour) {
      if constexpr (d == 512) K3_LAUNCH(4, 1, false);
      return;
    }
    if (n_blk <= kK3OneEach) {
      if (n_blk <= kK3CutInTwo) K3_WIDE(2);
      else K3_WIDE(1);
      return;
    }
#undef K3_WIDE
  }
  if (NB < 4 && n_blk <= kK3CutInTwo) K3_LAUNCH((NB == 2 ? 2 : 1), 1, false);
  else if (n_blk <= kK3HalfBlocks && !nt) K3_LAUNCH(1, 1, false);
  else {
    constexpr bool kWholeOnlyStreams = (int64_t)(kK3HalfBlocks + 1) * kRowAlign * d * 2 > kStreamBytes;
    if (kWholeOnlyStreams || nt) K3_LAUNCH(1, 2, true);
    else if constexpr (!kWholeOnlyStreams) K3_LAUNCH(1, 2, false);
  }
#undef K3_LAUNCH
}

void launch_k3_fused(const void *O, const void *U, const void *gamma, const void *beta, const void *W2p_layer, const void *b2,
                     void *Xh, void *Xl, bool lo_is_zero, const RowBlock *blocks, const int32_t *blk_list, int n_blk, int blk_first,
                     const Shape &sh, hipStream_t s) {
  if (n_blk <= 0) return;
#define K3_CASE(NWV, NB) launch_k3<NWV, NB>((const half_t *)O, (const half_t *)U, (const bf16_t *)gamma, (const bf16_t *)beta, (const half_t *)W2p_layer, \
    (const bf16_t *)b2, (half_t *)Xh, (half_t *)Xl, lo_is_zero ? 1 : 0, blocks, blk_list, n_blk, blk_first, sh.eps, s)
  if (sh.d == 512) K3_CASE(4, 4);
  else if (sh.d == 384) K3_CASE(3, 4);
  else if (sh.d == 256) K3_CASE(4, 2);
  else if (sh.d == 192) K3_CASE(3, 2);
  else K3_CASE(4, 1);
#undef K3_CASE
}

}  // namespace flame
