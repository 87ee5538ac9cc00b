// MFMA projections of the GR block for gfx950 (fp16 operands, fp32 accumulation):
//   K1  [U V Q K] = silu(X W1^T + b1)            (SiLU fused as the GEMM epilogue)
//   K3b X <- X + G W2^T + b2                     (residual fused as the GEMM epilogue; X is held as the two fp16 words
//                                                 Xh = fp16(X), k-tile blocked, and Xl = fp16(X - Xh), row-major)
// Both are C[m][n] = sum_k A[m][k] W[n][k].
//
// Tiling.  A 128x128 tile re-reads 1 byte of operand per 64 flop, which at MFMA speed is twice what
// the L2 delivers (measured about 19 TB/s), so the block tile is 256 x BN (BN = 128 where d allows):
// 256 threads = 4 wavefronts in a 2x2 arrangement, each owning 128 x BN/2 as 4 x (BN/64) blocks of
// v_mfma_f32_32x32x16_f16.  Two workgroups share a CU: with K = d as short as 512 the fixed cost of a
// tile (pipeline fill, epilogue) is a third of its time and only another resident workgroup hides it
// (a 256 x 256 tile at one workgroup per CU measured slower for exactly that reason).
//
// Pipeline (the role the cp.async pipeline plays in Section 3.2): k advances in steps of 32 through a
// ring of three LDS stages filled by LDS-DMA loads (global_load_lds_dwordx4: no staging registers,
// lane i of an instruction lands at base + 16 i).  Iteration kt waits for its own DMA of tile kt, passes
// one barrier (tile kt complete for everybody, tile kt-1 vacated by everybody), requests tile kt+2
// into the vacated stage - two iterations of flight time - and multiplies tile kt; the fragment reads
// of the second 16-deep step are issued behind the first MFMAs of the first step, so that they run
// under matrix work and nothing waits on them early.  LDS rows of A are 64 bytes; 16-byte chunks are
// XOR-swizzled over groups of 256 bytes (each DMA lane fetches the chunk that belongs in its slot: lds_off), which
// makes the fragment reads bank-conflict free without padding; W comes packed by fragments and needs no swizzle.
//
// Rows are addressed through 64-row blocks so that the same kernel runs on a contiguous range or on
// a list of candidate blocks (last-layer pruning).
#include <type_traits>

#include "device_common.h"
#include "kernels.h"

namespace flame {

namespace {

constexpr int BM = 256;
constexpr int BK = 32;
constexpr int RB = BM / kRowAlign;      // 64-row blocks per row tile

struct PlaneSel { int id[4]; int n; };

// XOR key of the chunk index in an epilogue patch whose rows hold CPR 16-byte chunks (8: 128-byte rows,
// two per 256-byte group; 4: 64-byte rows, four per group): 16 consecutive rows of one chunk column use
// every slot of the 256 bytes once.
template <int CPR>
__device__ __forceinline__ int patch_key(int row) { return CPR == 8 ? (row >> 1) & 7 : (row >> 2) & 3; }

// NT: the planes are stored past the caches (kStreamBytes).  (A template argument: of two stores in the branches of an if the compiler makes
// one, and drops the hint.)
template <int BN, int EPI, bool NT>
__global__ __launch_bounds__(256, 2) void gemm_mfma_kernel(
    const half_t *__restrict__ A, const half_t *__restrict__ W, const bf16_t *__restrict__ bias,
    PlanePtrs planes, half_t *__restrict__ Xl, half_t *__restrict__ Xh, int lo_is_zero,
    const int32_t *__restrict__ blk_list, int blk_first, int n_blk, int n_row_tiles, int n_col_tiles, int K, int d,
    int64_t ws_rows, PlaneSel sel, float alpha, bool a_blocked) {
  constexpr int WN = BN / 2;            // wavefront patch: 128 rows x WN columns
  constexpr int MB = 4;                 // 32-row MFMA blocks per wavefront
  constexpr int NB = WN / 32;           // 32-column MFMA blocks per wavefront
  constexpr int A_BYTES = BM * BK * 2, B_BYTES = BN * BK * 2, STAGE = A_BYTES + B_BYTES;
  constexpr int NSTAGE = 3;
  __shared__ __attribute__((aligned(128))) char smem[NSTAGE * STAGE];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  const int l32 = lane & 31, lhalf = lane >> 5;

  // Workgroup id -> (row tile, column tile).  Consecutive workgroup ids go round-robin over the 8
  // XCDs, each with its own L2: XCD x takes the row tiles congruent to x mod 8 and walks through all
  // column tiles of one row tile before the next, so an activation tile is fetched from HBM once
  // and then served from that XCD's L2, while the (small) weight matrix stays resident in all L2s.
  int row_tile, col_tile;
  {
    constexpr int NXCD = 8;
    const int wg = blockIdx.x, xcd = wg % NXCD, j = wg / NXCD;
    const int full = (n_row_tiles / NXCD) * NXCD;       // row tiles that split evenly over the XCDs
    const int rt = (j / n_col_tiles) * NXCD + xcd;
    if (rt < full) {
      row_tile = rt;
      col_tile = j % n_col_tiles;
    } else {                                            // the tail is dealt out in plain order
      const int t = wg - full * n_col_tiles;
      row_tile = full + t / n_col_tiles;
      col_tile = t % n_col_tiles;
    }
  }
  // column tile -> (plane, offset inside the plane)
  int plane = 0, n_in_plane = 0, n0;
  if (EPI == 0) {
    const int tiles_per_plane = d / BN;
    plane = sel.id[col_tile / tiles_per_plane];
    n_in_plane = (col_tile % tiles_per_plane) * BN;
    n0 = plane * d + n_in_plane;
  } else {
    n0 = col_tile * BN;
  }
  // the 64-row blocks of this row tile (-1: absent; loads then fall back to the first block)
  int blk[RB];
#pragma unroll
  for (int r = 0; r < RB; ++r) {
    const int t = row_tile * RB + r;
    blk[r] = t < n_blk ? (blk_list ? blk_list[t] : blk_first + t) : -1;
  }

  // LDS-DMA sources.  One instruction of a wavefront fills 1 KB = four 256-byte groups = 16 tile rows;
  // lane p owns physical slot p & 15 of group p >> 4 and must fetch the chunk the swizzle maps there:
  // row = 4 * group + (slot >> 2), chunk = (slot & 3) ^ key(row).  Instruction q of wavefront w covers tile
  // rows 16 * (4 q + w) .. + 15 (A: q = 0..3, one 64-row block each; B: q < BN / 64).
  constexpr int A_Q = BM / 64, B_Q = BN / 64;
  const int rloc = 16 * wave + 4 * (lane >> 4) + ((lane & 15) >> 2);
  const int dch = (lane & 3) ^ lds_key(rloc);
  // A is k-tile blocked (64 rows x 32 k = 2048 contiguous elements, whole 128-byte lines per request) when it is the
  // activation copy Xh, row-major when it is G.
  // Every request address is a wave-uniform base (64-row block and k tile: scalar arithmetic) plus a fixed 32-bit
  // lane offset in bytes, which is the scalar-base form of the request instruction: no vector address
  // arithmetic per k tile.  (Lane offsets are below 64 rows x K elements.)
  const char *abase[A_Q];
#pragma unroll
  for (int q = 0; q < A_Q; ++q) {
    const int b = blk[q] >= 0 ? blk[q] : blk[0];
    abase[q] = (const char *)(A + (int64_t)b * kRowAlign * K);
  }
  uint32_t alane = (uint32_t)(a_blocked ? rloc * 32 + dch * 8 : rloc * K + dch * 8) * 2u;
  const int a_kstep = (a_blocked ? 64 * BK : BK) * 2;                 // bytes per k tile
  // W is packed fragment by fragment (device_common.h): the two fragments of a 32-column block and k tile are 2 KB together.
  // Instruction q of wavefront w brings fragment w & 1 of column block 2 q + w / 2.
  const char *Wn0 = (const char *)(W + ((int64_t)(n0 / 32) + (wave >> 1)) * 32 * K + (wave & 1) * 512);  // n0 % 64 == 0
  uint32_t blane = (uint32_t)lane * 16u;
  // Operand order.  Row-major outputs (U, Q, K planes, X) want each lane to hold 4 consecutive
  // features of one token, which is the transposed accumulator: W rows as the A operand.  The V
  // plane is stored feature-major for the attention kernel (V^T is its A operand) and wants 4
  // consecutive tokens of one feature: activations as the A operand.
  const bool feature_major = (EPI == 0) && plane == 1;
  // Accumulators.  In the projection (EPI 0) they start from the bias, which then costs no instruction per
  // output: accumulator element e of block (i, j) is feature 32 j + 16 lhalf + e of the wavefront's columns
  // in the row-major planes, and feature 32 j + l32 (all elements alike) in the feature-major plane.
  f32x16 acc[MB][NB];
  if (EPI == 0) {
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      const bf16_t *bp = bias + plane * d + n_in_plane + wn * WN + 32 * j;
      if (!feature_major) {
        const bf16x8 b0v = *(const bf16x8 *)(bp + 16 * lhalf), b1v = *(const bf16x8 *)(bp + 16 * lhalf + 8);
#pragma unroll
        for (int i = 0; i < MB; ++i)
#pragma unroll
          for (int e = 0; e < 16; ++e) acc[i][j][e] = (float)(e < 8 ? b0v[e & 7] : b1v[e & 7]);
      } else {
        const float bv = to_f32(bp[l32]);
#pragma unroll
        for (int i = 0; i < MB; ++i)
#pragma unroll
          for (int e = 0; e < 16; ++e) acc[i][j][e] = bv;
      }
    }
  } else {
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
      for (int j = 0; j < NB; ++j)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;
  }
  // fragment byte offsets inside a stage for the two 16-deep steps (32-row blocks are 2048 bytes apart);
  // the activations are read in sigma32 row order when they play A;
  // W's fragments are packed in the row order of its role
  int f0[2], g0[2];
  {
    const int ra = feature_major ? sigma32(l32) : l32;
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      f0[ks] = lds_off(wm * 128 + ra, ks * 2 + lhalf);
      g0[ks] = A_BYTES + wn * (WN * 64) + ks * 1024 + lane * 16;
    }
  }

  typedef __attribute__((address_space(1))) const void gvoid;
  typedef __attribute__((address_space(3))) void lvoid;
  auto main_loop = [&](auto fm) {
    constexpr bool FM = decltype(fm)::value;
    const int nk = K / BK;
    const int k_rot = (n0 / BN) % nk;              // tied to the output columns, not to the launch's tile numbering
    auto request = [&](int tile, int stage) {            // A_Q + B_Q DMA instructions per wavefront
      // The workgroups that share a row tile (one per column tile) run at the same time on one XCD.  Each walks k
      // from a different starting tile (rotation by its column tile), so that they touch different lines of the
      // shared activations at any moment: one of them misses L2 on a line, the others hit it later, instead of
      // all of them missing together.
      int kt_ = (tile < nk ? tile : nk - 1) + k_rot;
      kt_ = kt_ >= nk ? kt_ - nk : kt_;
      // (the empty asm keeps the widening of the lane offsets next to the requests; hoisted out of the loop the
      // compiler would go back to full 64-bit vector addresses)
      asm volatile("" : "+v"(alane), "+v"(blane));
#pragma unroll
      for (int q = 0; q < A_Q; ++q)
        __builtin_amdgcn_global_load_lds((gvoid *)(abase[q] + (int64_t)kt_ * a_kstep + alane), (lvoid *)(smem + stage * STAGE + (4 * q + wave) * 1024), 16, 0, 0);
#pragma unroll
      for (int q = 0; q < B_Q; ++q)
        __builtin_amdgcn_global_load_lds((gvoid *)(Wn0 + ((size_t)q * 64 * K + (size_t)kt_ * (32 * BK)) * 2 + blane),
                                         (lvoid *)(smem + stage * STAGE + A_BYTES + (4 * q + wave) * 1024), 16, 0, 0);
    };
#define GEMM_MFMA(S, i, j)                                                                              \
  acc[i][j] = FM ? __builtin_amdgcn_mfma_f32_32x32x16_f16(fa[S][i], fb[S][j], acc[i][j], 0, 0, 0)         \
                 : __builtin_amdgcn_mfma_f32_32x32x16_f16(fb[S][j], fa[S][i], acc[i][j], 0, 0, 0)
    request(0, 0);
    request(1, 1);
    f16x8 fa[2][MB], fb[2][NB];
    // One k tile.  The stage is a compile-time constant (the loop below is unrolled over the ring), so the
    // fragment reads are a fixed lane offset plus an immediate and need no address instruction.
    auto k_step = [&](auto stage_c, const int kt) {
      constexpr int ST = decltype(stage_c)::value;
      // tile kt has landed for this wavefront once at most the requests of tile kt+1 are outstanding
      if (A_Q + B_Q == 6) asm volatile("s_waitcnt vmcnt(6)" ::: "memory");
      else asm volatile("s_waitcnt vmcnt(5)" ::: "memory");
      __builtin_amdgcn_s_barrier();
      request(kt + 2, (ST + 2) % NSTAGE);
      const char *sp = smem + ST * STAGE;
#pragma unroll
      for (int i = 0; i < MB; ++i) fa[0][i] = *(const f16x8 *)(sp + f0[0] + i * 2048);
#pragma unroll
      for (int j = 0; j < NB; ++j) fb[0][j] = *(const f16x8 *)(sp + g0[0] + j * 2048);
      __builtin_amdgcn_sched_barrier(0);
      GEMM_MFMA(0, 0, 0);
      GEMM_MFMA(0, 1, 0);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = 0; i < MB; ++i) fa[1][i] = *(const f16x8 *)(sp + f0[1] + i * 2048);
#pragma unroll
      for (int j = 0; j < NB; ++j) fb[1][j] = *(const f16x8 *)(sp + g0[1] + j * 2048);
      __builtin_amdgcn_sched_barrier(0);
      GEMM_MFMA(0, 2, 0);
      GEMM_MFMA(0, 3, 0);
#pragma unroll
      for (int j = 1; j < NB; ++j)
#pragma unroll
        for (int i = 0; i < MB; ++i) GEMM_MFMA(0, i, j);
#pragma unroll
      for (int j = 0; j < NB; ++j)
#pragma unroll
        for (int i = 0; i < MB; ++i) GEMM_MFMA(1, i, j);
      __builtin_amdgcn_sched_barrier(0);
    };
    static_assert(NSTAGE == 3, "the k loop is unrolled over a ring of three stages");
    for (int kt = 0; kt < nk; kt += NSTAGE) {
      k_step(std::integral_constant<int, 0>{}, kt);
      if (kt + 1 < nk) k_step(std::integral_constant<int, 1>{}, kt + 1);
      if (kt + 2 < nk) k_step(std::integral_constant<int, 2>{}, kt + 2);
    }
#undef GEMM_MFMA
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");     // the clamped tail requests must not outlive the workgroup's LDS
  };
  if (feature_major) main_loop(std::true_type{});
  else main_loop(std::false_type{});

  // Epilogue.  With the sigma32 row order accumulator element e of a 32x32 block sits at (A-operand
  // tile row 16*lhalf + e, B-operand tile row l32).
  const int b0 = wm ? blk[2] : blk[0], b1 = wm ? blk[3] : blk[1];    // the two 64-row blocks of this wavefront's 128 rows
  if (EPI == 0) {
    // Only two lanes share an output row in the accumulator layout, so direct stores would reach the
    // L2 as 32-byte pieces, and the write path is then bound by the number of requests.  The
    // wavefront's patch goes through LDS instead (the operand ring is free by now; each wavefront
    // owns a private slice of it, chunks XOR-swizzled by row so that writes and reads are conflict free) and leaves as 16 bytes per lane with
    // whole 128-byte lines per output row.
    __builtin_amdgcn_s_barrier();                     // every wavefront has finished reading the ring
    char *pb = smem + wave * (128 * WN * 2);
    half_t *P = (half_t *)(plane == 0 ? planes.u : plane == 1 ? planes.v : plane == 2 ? planes.q : planes.k);
    if (!feature_major) {
      // patch[128 tokens][WN features]; lane holds token 32i + l32, features 32j + 16*lhalf + 0..15
      // (the bias is already in the accumulators).  Q leaves this kernel multiplied by alpha / 2: the
      // attention kernel works on halved logits; the other planes are stored plain.
      constexpr int CPR = WN / 8;                     // 16-byte chunks per patch row
      auto to_patch = [&](auto scaled) {
        const float sc = alpha * 0.5f;
#pragma unroll
        for (int j = 0; j < NB; ++j) {
#pragma unroll
          for (int i = 0; i < MB; ++i) {
            const int row = 32 * i + l32;
#pragma unroll
            for (int g = 0; g < 2; ++g) {
              f16x8 o;
#pragma unroll
              for (int q = 0; q < 8; ++q) {
                const float w = silu_fast(acc[i][j][8 * g + q]);
                o[q] = to_f16_sat(decltype(scaled)::value ? w * sc : w);
              }
              const int c = 4 * j + 2 * lhalf + g;
              *(f16x8 *)(pb + row * (WN * 2) + ((c ^ patch_key<CPR>(row)) << 4)) = o;
            }
          }
        }
      };
      if (plane == 2) to_patch(std::true_type{});
      else to_patch(std::false_type{});
      constexpr int RPI = 64 / CPR;                   // patch rows per store instruction
      const int rl = lane / CPR, c = lane % CPR;
      // Store instruction `it` takes patch rows it * RPI + rl.  No address arithmetic per instruction: the
      // patch address is a fixed lane offset plus an immediate (rows RPI apart share their swizzle key, except
      // that with 8 chunks per row every other instruction flips bit 2 of it), and the global address is a
      // scalar base (64-row block, row group, column: wave-uniform) plus the fixed lane offset of (rl, c).
      static_assert(CPR == 8 || CPR == 4, "patch rows of 128 or 64 bytes");
      constexpr int FLIP = CPR == 8 ? 64 : 0;
      const int lds0 = rl * (WN * 2) + ((c ^ patch_key<CPR>(rl)) << 4);
      uint32_t goff = (uint32_t)(rl * d + c * 8) * 2u;
      const char *gcol = (const char *)(P + n_in_plane + wn * WN);
      // the two 64-row blocks of the patch in turn: all reads of a block first, then its stores
      constexpr int NI = 64 / RPI;                    // store instructions per 64-row block
#pragma unroll
      for (int hb = 0; hb < 2; ++hb) {
        const int rblk = hb ? b1 : b0;
        if (rblk < 0) continue;
        const char *gblk = gcol + (int64_t)rblk * kRowAlign * d * 2;
        f16x8 v[NI];
#pragma unroll
        for (int k = 0; k < NI; ++k) {
          const int it = hb * NI + k;
          v[k] = *(const f16x8 *)(pb + it * RPI * (WN * 2) + (lds0 ^ ((it & 1) ? FLIP : 0)));
        }
        asm volatile("" : "+v"(goff));   // keeps the widening of the offset next to the stores (scalar base + offset form)
#pragma unroll
        for (int k = 0; k < NI; ++k) store_once<NT>(v[k], (f16x8 *)(gblk + (int64_t)(k * RPI) * d * 2 + goff));
      }
    } else {
      // patch[WN features][128 tokens]; lane holds feature 32j + l32, tokens 32i + 16*lhalf + 0..15
#pragma unroll
      for (int j = 0; j < NB; ++j) {
        const int fr = 32 * j + l32;
#pragma unroll
        for (int i = 0; i < MB; ++i) {
#pragma unroll
          for (int g = 0; g < 2; ++g) {
            f16x8 o;
#pragma unroll
            for (int q = 0; q < 8; ++q) o[q] = to_f16_sat(silu_fast(acc[i][j][8 * g + q]));
            const int c = 4 * i + 2 * lhalf + g;
            *(f16x8 *)(pb + fr * 256 + (((c ^ fr) & 15) << 4)) = o;
          }
        }
      }
      const int rl = lane >> 4, c = lane & 15;
      const int rblk = c >= 8 ? b1 : b0;
      // Store instruction `it` takes feature rows 4 it + rl.  As above: the patch address is a fixed lane offset
      // XOR a constant (the swizzle key of row 4 it + rl is that of rl XOR 4 it) plus an immediate, the global
      // address a scalar base (feature row group) plus a fixed lane offset (row rl, token block and chunk of c).
      const int lds0 = rl * 256 + ((c ^ rl) << 4);
      uint32_t goff = (uint32_t)((int64_t)rl * ws_rows + (int64_t)(rblk < 0 ? 0 : rblk) * kRowAlign + (c & 7) * 8) * 2u;
      const char *gfeat = (const char *)(P + (int64_t)(n_in_plane + wn * WN) * ws_rows);
      if (rblk >= 0) {
        constexpr int NI = 8;                           // reads in flight before their stores
#pragma unroll
        for (int i0 = 0; i0 < WN / 4; i0 += NI) {
          f16x8 v[NI];
#pragma unroll
          for (int k = 0; k < NI; ++k) {
            const int it = i0 + k;
            v[k] = *(const f16x8 *)(pb + it * 1024 + (lds0 ^ (((4 * it) & 15) << 4)));
          }
          asm volatile("" : "+v"(goff));
#pragma unroll
          for (int k = 0; k < NI; ++k) store_once<NT>(v[k], (f16x8 *)(gfeat + (int64_t)(4 * (i0 + k)) * ws_rows * 2 + goff));
        }
      }
    }
  } else {
#pragma unroll
    for (int i = 0; i < MB; ++i) {
      const int rblk = i >= 2 ? b1 : b0;              // 32-row block i lies inside one 64-row block
      if (rblk < 0) continue;
      const int64_t m = (int64_t)rblk * kRowAlign + (i & 1) * 32 + l32;
#pragma unroll
      for (int j = 0; j < NB; ++j) {
        const int nn = n0 + wn * WN + j * 32 + 16 * lhalf;
#pragma unroll
        for (int g = 0; g < 2; ++g) {
          const bf16x8 bv = *(const bf16x8 *)(bias + nn + 8 * g);
          const f16x8 h8 = *(const f16x8 *)(Xh + blocked_index(m, nn + 8 * g, d));
          f16x8 l8;
#pragma unroll
          for (int q = 0; q < 8; ++q) l8[q] = (half_t)0.f;
          if (!lo_is_zero) l8 = *(const f16x8 *)(Xl + m * d + nn + 8 * g);
          f16x8 o, ol;
#pragma unroll
          for (int q = 0; q < 8; ++q) {
            const float x = ((float)h8[q] + (float)l8[q]) + (acc[i][j][8 * g + q] + (float)bv[q]);
            o[q] = to_f16_sat(x);
            ol[q] = to_f16_sat(x - (float)o[q]);
          }
          *(f16x8 *)(Xl + m * d + nn + 8 * g) = ol;
          *(f16x8 *)(Xh + blocked_index(m, nn + 8 * g, d)) = o;
        }
      }
    }
  }
}


// K1 on small tiles: 64 rows x 128 columns (CW = 4) or 256 (CW = 8) per workgroup.  The 64-row block of X sits whole in LDS (its k-tile blocked copy is one
// contiguous piece, brought by LDS-DMA in one go: the memory latency is paid once and not once per k tile of a short ring), W's
// fragments come straight from L2 into a register ring eight (CW = 8: four) k tiles deep, and the k loop, unrolled, has no barrier.  Wavefront
// w of CW owns columns 32 w .. 32 w + 31 of the tile, both 32-row halves.  A tile is halves of 64 columns, each within one
// plane.  Every output is the same chain of matrix instructions over the same k order as in the large tile (k starts at the
// column tile's rotation), so the two agree bit for bit.
// It serves launches that leave the chip idle at 256-row tiles, where the latency of a lone workgroup is what counts, and narrow
// models, whose large tile has six k tiles or fewer to hide its start and its epilogue behind; see launch_uvqk_bf16.
// NK = d / 32.
template <int NK, bool NT, int CW>
__global__ __launch_bounds__(64 * CW, CW == 8 ? 4 : 1) void gemm_small_kernel(const half_t *__restrict__ A, const half_t *__restrict__ W, const bf16_t *__restrict__ bias,
                                                         PlanePtrs planes, const int32_t *__restrict__ blk_list, int blk_first, int n_blk, int n_col_tiles,
                                                         int64_t ws_rows, PlaneSel sel, float alpha, const int32_t *__restrict__ uq_list, int n_uq) {
  constexpr int nk = NK, d = NK * BK, rot_cols = d % 128 == 0 ? 128 : 64;
  extern __shared__ __attribute__((aligned(256))) char lds[];   // [k / 32][64 rows][32 k], swizzled; the output patches afterwards
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, lhalf = lane >> 5;
  // XCD x takes the row blocks congruent to x mod 8 (see the large tile)
  int row_blk, col_tile;
  bool second;
  {
    constexpr int NXCD = 8;
    int wg = blockIdx.x;
    const int n_first = (int)gridDim.x - n_uq * n_col_tiles;
    second = wg >= n_first;
    if (second) {                                                // the second part of the launch: U and Q of the blocks in uq_list
      wg -= n_first;
      blk_list = uq_list;
      n_blk = n_uq;
    }
    const int xcd = wg % NXCD, j = wg / NXCD;
    const int full = (n_blk / NXCD) * NXCD;
    const int rt = (j / n_col_tiles) * NXCD + xcd;
    if (rt < full) {
      row_blk = rt;
      col_tile = j % n_col_tiles;
    } else {
      const int t = wg - full * n_col_tiles;
      row_blk = full + t / n_col_tiles;
      col_tile = t % n_col_tiles;
    }
  }
  const int blk = blk_list ? blk_list[row_blk] : blk_first + row_blk;
  // X block -> LDS.  Instruction q of a wavefront fills tile rows 16 wave .. + 15 of k tile q (the swizzle of the large tile).
  typedef __attribute__((address_space(1))) const void gvoid;
  typedef __attribute__((address_space(3))) void lvoid;
  {
    const int rloc = 16 * (wave & 3) + 4 * (lane >> 4) + ((lane & 15) >> 2);
    const int dch = (lane & 3) ^ lds_key(rloc);
    const char *src = (const char *)(A + (int64_t)blk * kRowAlign * d);
    uint32_t off = (uint32_t)(rloc * 32 + dch * 8) * 2u;
    asm volatile("" : "+v"(off));
#pragma unroll
    for (int i = 0; i < 4 * NK / CW; ++i) {
      const int q = CW / 4 * i + (wave >> 2);
      __builtin_amdgcn_global_load_lds((gvoid *)(src + q * 4096 + off), (lvoid *)(lds + q * 4096 + (wave & 3) * 1024), 16, 0, 0);
    }
  }
  // this wavefront's 32 columns
  const int cols_per_plane = d / 64;                            // halves of 64 columns per plane
  const int half = CW / 2 * col_tile + (wave >> 1);             // index over the selected planes
  const int plane = second ? 2 * (half / cols_per_plane) : sel.id[half / cols_per_plane];
  const int n_half = (half % cols_per_plane) * 64;              // first column of the half inside its plane
  const int n_col = n_half + (wave & 1) * 32;
  const int n0 = plane * d + n_col;
  const bool feature_major = plane == 1;
  const int k_rot = ((plane * d + n_half) / rot_cols) % nk;
  f32x16 acc[2];
  {
    const bf16_t *bp = bias + plane * d + n_col;
    if (!feature_major) {
      const bf16x8 b0v = *(const bf16x8 *)(bp + 16 * lhalf), b1v = *(const bf16x8 *)(bp + 16 * lhalf + 8);
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[i][e] = (float)(e < 8 ? b0v[e & 7] : b1v[e & 7]);
    } else {
      const float bv = to_f32(bp[l32]);
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[i][e] = bv;
    }
  }
  constexpr int PD = NK < 8 ? NK : CW == 8 ? 4 : 8;             // k tiles of W in flight
  auto main_loop = [&](auto fm) {
    constexpr bool FM = decltype(fm)::value;
    const char *wb = (const char *)(W + (int64_t)(n0 / 32) * 32 * d);
    uint32_t woff = (uint32_t)lane * 16u;
    const int aoff[2] = {lds_off(FM ? sigma32(l32) : l32, lhalf), lds_off(FM ? sigma32(l32) : l32, 2 + lhalf)};
    auto kt_of = [&](int i) { const int k = i + k_rot; return k >= nk ? k - nk : k; };
    f16x8 fw[PD][2], fa[2][2][2];
    auto load_w = [&](int i) {
      asm volatile("" : "+v"(woff));
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) fw[i % PD][ks] = *(const f16x8 *)(wb + (kt_of(i) * 2 + ks) * 1024 + woff);
    };
    auto read_a = [&](int i) {
      const char *t = lds + kt_of(i) * 4096;
#pragma unroll
      for (int ks = 0; ks < 2; ++ks)
#pragma unroll
        for (int r = 0; r < 2; ++r) fa[i & 1][ks][r] = *(const f16x8 *)(t + aoff[ks] + r * 2048);
    };
#pragma unroll
    for (int p = 0; p < PD; ++p) load_w(p);
    // X has landed (it was requested ahead of W's fragments, and all of those are out: the wait counts them)
    __builtin_amdgcn_sched_barrier(0);
    static_assert((PD == 8 || CW == 4 || PD == 4) && NK * 4 % CW == 0, "the waits below count the fragments requested behind X");
    if (PD == 8) asm volatile("s_waitcnt vmcnt(16)" ::: "memory");
    else if (CW == 8) asm volatile("s_waitcnt vmcnt(8)" ::: "memory");
    else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
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
          acc[r] = FM ? __builtin_amdgcn_mfma_f32_32x32x16_f16(fa[i & 1][ks][r], fw[i % PD][ks], acc[r], 0, 0, 0)
                      : __builtin_amdgcn_mfma_f32_32x32x16_f16(fw[i % PD][ks], fa[i & 1][ks][r], acc[r], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
      if (i + PD < NK) load_w(i + PD);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  if (feature_major) main_loop(std::true_type{});
  else main_loop(std::false_type{});
  // Epilogue: SiLU, then through an 8 KB patch per half so that whole 128-byte lines leave (see the large tile).
  __syncthreads();                                              // everybody has read X
  char *pb = lds + (wave >> 1) * 8192;
  const float sc = plane == 2 ? alpha * 0.5f : 1.0f;
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int g = 0; g < 2; ++g) {
      f16x8 o;
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        const float w = silu_fast(acc[i][8 * g + q]);
        o[q] = to_f16_sat(plane == 2 ? w * sc : w);
      }
      const int row = feature_major ? (wave & 1) * 32 + l32 : 32 * i + l32;
      const int c = feature_major ? 4 * i + 2 * lhalf + g : 4 * (wave & 1) + 2 * lhalf + g;
      *(f16x8 *)(pb + row * 128 + ((c ^ patch_key<8>(row)) << 4)) = o;
    }
  __syncthreads();
  half_t *P = (half_t *)(plane == 0 ? planes.u : plane == 1 ? planes.v : plane == 2 ? planes.q : planes.k);
  const int ht = tid & 127, c = ht & 7;
#pragma unroll
  for (int it = 0; it < 4; ++it) {
    const int r = (ht >> 3) + 16 * it;
    const f16x8 v = *(const f16x8 *)(pb + r * 128 + ((c ^ patch_key<8>(r)) << 4));
    half_t *dst = feature_major ? P + (int64_t)(n_half + r) * ws_rows + (int64_t)blk * kRowAlign + c * 8
                                : P + ((int64_t)blk * kRowAlign + r) * d + n_half + c * 8;
    store_once<NT>(v, (f16x8 *)dst);
  }
}

}  // namespace

// The small tile stores past the caches only from this size of a plane on, not from kStreamBytes: it runs the narrow models, whose attention
// kernel is short and still finds part of such planes in the caches.  From 64 MB on attention is the faster for stores past them.  Microseconds per forward of 4 layers, requests of 64 + 64, through / past the caches:
//   d = 64: 32 MB 748 / 768, 48 MB 1150 / 1134, 64 MB 1558 / 1461, 128 MB 3103 / 2990
//   d = 128: 48 MB 794 / 833, 64 MB 1101 / 1084, 128 MB 2189 / 2094;  d = 192: 48 MB 846 / 888, 72 MB 1281 / 1249, 192 MB 3274 / 3203
// (Attention at d = 64, 64 MB: 105.5 / 95.6 us per launch.)  The wider models leave the small tile long before.
constexpr int64_t kSmallStreamBytes = 64 << 20;
template <int NK, bool NT = false, int CW = 4>
static void launch_small(const void *Xh, const void *W1h, const void *b1, PlanePtrs planes, const int32_t *blk_list, int blk_first, int n_blk, const PlaneSel &sel,
                         const int32_t *uq_list, int n_uq, const Shape &sh, hipStream_t s) {
  const int col_tiles = sel.n * (sh.d / 64) / (CW / 2);
  const int lds = 4096 * (NK < CW ? CW : NK);                  // the X block, at least the output patches
  gemm_small_kernel<NK, NT, CW><<<(n_blk + n_uq) * col_tiles, 64 * CW, lds, s>>>((const half_t *)Xh, (const half_t *)W1h, (const bf16_t *)b1, planes, blk_list, blk_first, n_blk,
                                                           col_tiles, sh.ws_rows, sel, sh.alpha, uq_list, n_uq);
}

// Up to this many 64-row blocks a launch runs on the small tiles.  The wider the model, the fewer workgroups of the small tile fit a
// compute unit (its X block is 128 d bytes of LDS) and the more its W traffic, once per 64 rows, weighs against the large
// tile's, once per 256.  Microseconds per launch, small against large, four planes:
//   d = 512: 16 blocks 11.2 / 18.5, 48: 16.7 / 19.8, 96: 25.6 / 26.4, 128: 31.6 / 29.3 (small tiles of 128 columns; of 256: below)
//   d = 384: 16: 10.1 / 16.3, 128: 21.5 / 23.4, 384: 48 / 52, 512: 61 / 60
//   d = 256: 16: 8.6 / 13.6, 256: 21.8 / 23.6, 1024: 62 / 63, 2048: 122 / 116
//   d = 192: 16: 7.9 / 10.1, 256: 16.9 / 19.7, 2048: 84 / 91, 8192: 340 / 345 (the large tile is 64 columns wide there)
//   d = 128: 256: 14.6 / 17.3, 2048: 47 / 50, 8192: 173 / 175, 10240: 229 / 209, 16384: 352 / 343
//   d = 64: 512: 12.9 / 14.8, 2048: 22.2 / 25.3, 8192: 64 / 81, 16384: 143 / 182
// d = 384 and 512 from these blocks on with eight wavefronts, 64 rows x 256 columns, which halve the traffic of X, once per column tile, where there are enough tiles all the same.
// Forwards of 8 layers (us), 128 columns wide (or the large tile, from 97 and 385 blocks on) / 256:
//   d = 512: 16: 212 / 217, 18: 236 / 230, 45: 349 / 350, 63: 463 / 452, 90: 385 / 367, 150: 575 / 534, 250: 738 / 727, 310: 988 / 956, 350: 1064 / 1022, 400: 1177 / 1125, 480: 1349 / 1302
//     (64 + 64 from 310 on, 640: 1772 / 1734, 1000: 2597 / 2671; 512 + 128: 380: 1102 / 1086, 640: 1786 / 1778; 2048 + 512: 560: 2095 / 2121).  The line of d = 512 lies where the first
//     form of call stops to gain: prefill and scores of 4 layers, 1000 + 64, by blocks of the history pass: 288: 752 / 751, 352: 828 / 831, 368: 834 / 850, 448: 909 / 925
//   d = 384: 100: 330 / 351, 180: 485 / 493, 210: 526 / 524, 300: 724 / 721, 450: 926 / 901, 800: 1542 / 1529, 1000: 1772 / 1836
// (Stores past the caches slow the wide tile down: d = 512, 400 blocks 1065 -> 1091; d = 384, 800: 1529 -> 1567.)
// Between, d = 512: up to 32 blocks the wide tiles are one for each compute unit, and up to 47 a second one for less than half of them (45 blocks: 13.9 / 14.8 us per launch).
constexpr int kWideFrom512 = 17, kWideOneEach512 = 32, kWideAgainFrom512 = 48, kWideFrom384 = 210;
static bool wide_512(int n_blk) { return n_blk >= kWideFrom512 && (n_blk <= kWideOneEach512 || n_blk >= kWideAgainFrom512); }
static int small_tile_blocks(int d) {
  switch (d) {
    case 64: case 192: return 1 << 30;
    case 128: return 8192;
    case 256: return 1024;
    case 384: return 800;
    case 512: return 352;
    default: return 0;                                          // no instance
  }
}

void launch_uvqk_bf16(const void *Xh, const void *W1h, const void *b1, PlanePtrs planes, const int32_t *blk_list,
                      int n_blk, int blk_first, int plane_mask, const int32_t *uq_list, int n_uq, const Shape &sh, hipStream_t s) {
  if (n_blk <= 0 || !(plane_mask & 0xF)) return;
  PlaneSel sel{};
  for (int p = 0; p < 4; ++p)
    if (plane_mask & (1 << p)) sel.id[sel.n++] = p;
  const int row_tiles = (n_blk + RB - 1) / RB;
  const int bn = sh.d % 128 == 0 ? 128 : 64;
  const int64_t bytes = (int64_t)n_blk * kRowAlign * sh.d * 2;       // of a plane
  const bool nt = bytes > kStreamBytes;
  if (n_blk <= small_tile_blocks(sh.d) && sel.n * (sh.d / 64) % 2 == 0) {   // (whole tiles of 128 columns: every pair of planes has them)
    const bool snt = bytes >= kSmallStreamBytes;
#define K1_SMALL(...) launch_small<__VA_ARGS__>(Xh, W1h, b1, planes, blk_list, blk_first, n_blk, sel, uq_list, n_uq, sh, s)
    switch (sh.d) {
      case 64: if (snt) K1_SMALL(2, true); else K1_SMALL(2); break;
      case 128: if (snt) K1_SMALL(4, true); else K1_SMALL(4); break;
      case 192: if (snt) K1_SMALL(6, true); else K1_SMALL(6); break;
      case 256: K1_SMALL(8); break;
      case 384: if (n_blk >= kWideFrom384 && sel.n % 2 == 0) K1_SMALL(12, false, 8); else K1_SMALL(12); break;
      default: if (wide_512(n_blk)) K1_SMALL(16, false, 8); else K1_SMALL(16); break;
    }
#undef K1_SMALL
    return;
  }
  if (n_uq > 0) launch_uvqk_bf16(Xh, W1h, b1, planes, uq_list, n_uq, 0, 0x5, nullptr, 0, sh, s);
  const int col_tiles = sel.n * (sh.d / bn);
#define K1_CASE(BNV, NTV) gemm_mfma_kernel<BNV, 0, NTV><<<row_tiles * col_tiles, 256, 0, s>>>((const half_t *)Xh, (const half_t *)W1h, (const bf16_t *)b1, planes, nullptr, \
    nullptr, 0, blk_list, blk_first, n_blk, row_tiles, col_tiles, sh.d, sh.d, sh.ws_rows, sel, sh.alpha, true)
  if (bn == 128) { if (nt) K1_CASE(128, true); else K1_CASE(128, false); }
  else { if (nt) K1_CASE(64, true); else K1_CASE(64, false); }
#undef K1_CASE
}

void launch_outproj_bf16(const void *G, const void *W2h, const void *b2, void *Xh, void *Xl, bool lo_is_zero, const int32_t *blk_list,
                         int n_blk, int blk_first, const Shape &sh, hipStream_t s) {
  if (n_blk <= 0) return;
  PlaneSel sel{};
  const int row_tiles = (n_blk + RB - 1) / RB;
  if (sh.d % 128 == 0) {
    const int col_tiles = sh.d / 128;
    gemm_mfma_kernel<128, 1, false><<<row_tiles * col_tiles, 256, 0, s>>>((const half_t *)G, (const half_t *)W2h, (const bf16_t *)b2, PlanePtrs{}, (half_t *)Xl,
                                                                   (half_t *)Xh, lo_is_zero ? 1 : 0, blk_list, blk_first, n_blk, row_tiles, col_tiles,
                                                                   sh.d, sh.d, sh.ws_rows, sel, 1.0f, false);
  } else {
    const int col_tiles = sh.d / 64;
    gemm_mfma_kernel<64, 1, false><<<row_tiles * col_tiles, 256, 0, s>>>((const half_t *)G, (const half_t *)W2h, (const bf16_t *)b2, PlanePtrs{}, (half_t *)Xl,
                                                                  (half_t *)Xh, lo_is_zero ? 1 : 0, blk_list, blk_first, n_blk, row_tiles, col_tiles,
                                                                  sh.d, sh.d, sh.ws_rows, sel, 1.0f, false);
  }
}

}  // namespace flame
