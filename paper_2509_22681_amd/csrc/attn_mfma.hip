// Jagged masked pointwise-SiLU attention with relative-position bias, fp16 MFMA (fp32 accumulation), gfx950.
//
// For every query row r of a request and every head:
//     O_r = sum over allowed keys c of silu(<Q_r, K_c> + bias[p_r - p_c]) V_c
// Q arrives multiplied by alpha/2 and the bias table by 1/2, so the kernel sees halved logits s = x/2
// (both factors are powers of two for the usual alpha: no rounding).  History rows look at keys 0..r,
// candidate rows look at the whole history and at themselves: the customised mask of Section 3.2
// that lets all candidates of a request be scored in one pass.  No score matrix is materialised:
// like a flash-attention tile loop, but the pointwise SiLU needs neither running maximum nor
// rescaling.
//
// Work decomposition: one workgroup = (query tile of 128 rows, head); 4 wavefronts of 32 query rows
// (one 32-row MFMA block each: about 150 registers per lane and 38 KB of LDS per workgroup, so three
// workgroups = three wavefronts per SIMD fit a CU; the kernel is bound by MFMA + VALU issue, and a third
// wavefront per SIMD fills part of the issue slots that two leave empty: measured 1.46x from one to two,
// 1.04x from two to three, the latter net of twice the K/V tile traffic of 256-row query tiles).  Keys
// are walked in tiles of 64.  A tile (K rows and V^T rows) is brought into one of two LDS stages by LDS-DMA loads
// (global_load_lds: no staging registers, no LDS store instructions), requested one tile ahead right after the
// barrier that opens the current tile (three tiles' time of a wavefront alone, as three share a SIMD: a third
// stage with requests two tiles ahead is no faster).  LDS rows are unpadded (a DMA instruction fills 1 KB of consecutive LDS) and 16-byte chunks are
// XOR-swizzled so that 16 consecutive lanes of a fragment read fall into 16 different slots of the 256
// bytes the LDS serves per clock.
//
// Register-level formulation: the products are computed transposed,
//     S^T[kv][q] = K Q^T      (A operand = K rows, B operand = Q rows)
//     O^T[d][q] += V^T P^T    (A operand = V^T rows, B operand = P^T)
// so that the accumulator of the first product, where a lane holds one query column and 16 key
// rows, already has the register layout of the second product's B operand.  The only thing to
// arrange is which key goes to which MFMA row: feeding key row pi(m) = m with bits 2 and 3 swapped
// into MFMA row m makes accumulator elements 8s..8s+7 of a lane hold keys 16s+8*(lane/32)+0..7, which
// is exactly the k order of a 16-deep B operand.  V is stored feature-major by the projection
// kernel, so V^T tiles are plain row loads.
//
// SiLU: the weights of a wavefront's 32x64 block are made by the cheapest of three routes that its largest |x| (masked positions included) allows: polynomials whose correction term runs
// in packed fp16 up to 2 and 4, the exact exp2/rcp form in fp32 beyond.  Vector instructions per block, with the test: 105, 137 and 217, beside 16 MFMAs.  Error of a weight, largest and
// root mean square over the range (the fp16 rounding of the weight included): 1.4e-3 and 2.4e-4 up to 2, 4.8e-3 and 8.2e-4 up to 4.
// (A form s + s^2 for |x| <= 1/4 and a bracket of two coefficients up to 1 save half and a seventh of the instructions, but are further off where their ranges end.)
// The mask is applied on boundary tiles only.
//
// Bias: a lane's eight consecutive entries (by decreasing distance, fp32) per accumulator half-block are read from LDS
// straight into the accumulator registers, so the bias add costs LDS bandwidth but no VALU instruction (on this
// chip VALU and MFMA work of one SIMD largely serialise, so every VALU instruction saved counts).  The rows of a
// wavefront start at all offsets; a ring of 256 entries in four copies, one entry apart from each other, makes every
// lane's reads aligned 16-byte ones (beside a window per stage read by dwords, forwards: 16 x (8192 + 512), 8 heads, 2 layers
// 2310 -> 2283 us, 40 x (2500 + 300), 4 layers 2894 -> 2875, softmax 3047 -> 2978; softmax with heads of 32 3571 -> 3590: that
// instance keeps the window and three stages).  A tile adds 64 entries.
#include <type_traits>

#include "device_common.h"
#include "kernels.h"

namespace flame {

namespace {

constexpr int KH = 64;              // keys per block (one pass of the register-level loop); an LDS tile has KP of them, one per wavefront of a group

// SiLU for |x| <= 2: the polynomial of device_common.h, silu(x) = x/2 + x^2 (a1 + a3 x^2 + a5 x^4).  On the halved
// logit s = x/2, with t = s^2:
//   silu(x) = s + q,   q = t (4 a1 + 16 a3 t + 64 a5 t^2).
// t and the bracket are evaluated in packed fp16 (one multiply and two fused multiply-adds per pair of
// weights); the last step is a mixed-precision fused multiply-add per weight, fp16 t times fp16 bracket
// plus the fp32 logit itself, rounded to fp16 once, like the weight of the exact route.
constexpr float kPolyT2 = 1.0f;                                  // bound on t = s^2  (|x| <= 2)
// Second segment, |x| <= 4 (t <= 4): silu(x) = s + t (B0 + B1 t + B2 t^2 + B3 t^3 + B4 t^4), minimax-weighted fit of
// (silu(2 s) - s) / t on 0 <= t <= 4 (error of silu below 5.4e-4).
constexpr float kMidT2 = 4.0f;
__device__ constexpr float kMidB[5] = {0.9926417973f, -0.3010154918f, 0.0835130618f, -0.0141349725f, 0.0010234216f};
__device__ __forceinline__ int pi32(int m) {  // swap bits 2 and 3
  return (m & ~12) | ((m & 4) << 1) | ((m & 8) >> 1);
}

// eight attention weights -> fp16 B-operand fragment (v_cvt_pk_f16_f32, round to nearest even).
// A weight beyond the fp16 range becomes inf; the output store saturates, so nothing non-finite is
// ever written to the workspace.
__device__ __forceinline__ f16x8 pack8(const float *v) {
  f16x8 r;
#pragma unroll
  for (int i = 0; i < 8; ++i) r[i] = (half_t)v[i];
  return r;
}

// SOFTMAX = false: the weights are silu(logit), pointwise.  SOFTMAX = true: the weights of a query row are
// softmax over its allowed keys of logit / tau (tau per layer and head); the kernel keeps a running maximum and
// sum per row and rescales its output accumulators when the maximum moves (one pass over the keys).  The logit
// in the accumulators is halved, so the exponent fed to the base-2 exponential is accumulator * tscale_h[head]
// with tscale = 2 log2(e) / tau.  The 64 keys of a block of one query sit in two lanes (lane and lane ^ 32),
// which exchange their maxima with one half-swap; their partial sums are only added at the end.
//
// KP = wavefronts per group of 32 query rows.  KP = 1 is the throughput configuration described at the top: 4 wavefronts, key tiles
// of 64, three workgroups per CU.  KP > 1 is the latency configuration, for batches too small to fill the chip, where a workgroup
// sits alone on its CU and its run time is the chain of key tiles of its longest row.  There a row's keys are summed in four
// partial outputs, 64-key block i going to partial output i % 4, which are added in a fixed order at the end; the sums are
// grouped differently than with KP = 1, so the two configurations agree to rounding, not bit for bit.  Two shapes with the same bits:
//   KP = 4: 64 query rows, 8 wavefronts and 4 feeders, key tiles of 256 in two LDS stages; each of a group's FOUR wavefronts takes one 64-key quarter
//     of every tile (two wavefronts per SIMD, so one's MFMAs run under the other's VALU work).  The chain is a quarter as
//     many steps, and a request of a few thousand rows has enough query tiles for every CU.  One request of 2573 + 217, 8 heads:
//     22 us per launch (32 with query tiles of 128 and two wavefronts per group on key tiles of 128), 20 with the feeders: four wavefronts that do nothing but make the tiles'
//     64 requests of 1 KB, 1000 cycles of the compute unit's address path per tile, which the others else wait out ahead of their arithmetic; 19 with the bias window in four
//     copies as above (20 requests of 256 bytes).
//   KP = 2: 128 query rows, 8 wavefronts, key tiles of 128 in four LDS stages; each of a group's two wavefronts takes one 64-key half of every
//     tile, into one of two accumulator sets by the tile's parity.  For latency handles that are given enough rows to
//     fill the chip all the same: half the K and V traffic per query row (the rule and both sides' times are at kLatencyWideTiles).
// SEQ: the throughput configuration in launches that leave most of the chip idle, where a wavefront alone runs through all keys of its 32 rows
// at 1750 cycles per 64 of them (760 for the weights, 370 each for the two products, the rest bias and requests).  The key tiles of KP = 4, but the four wavefronts of a
// group only make the weights, each of its 64 keys, and leave them in LDS (over the tile's K, which everybody has read; behind the stages with heads of 32);
// one wavefront per feature block then adds V^T P^T up over the tile in the order of the keys.  That is the one-wavefront order, block by block of 64 keys on the same SiLU route, so the
// bits are the same.  An item of 128 rows is two workgroups of 64.  One request of 1024 + 256, 8 heads, 16 layers: 17.5 -> 13 us per launch, forward 642 -> 556 us; with the feeders 12.8 -> 11.7 us.
// (Pointwise weights only: a running maximum would have to pass from wavefront to wavefront.)
template <int DH, bool SOFTMAX, int KP, bool NT, bool SEQ = false>
__global__ __launch_bounds__(KP == 4 ? 768 : KP > 1 ? 512 : 256, KP > 1 ? 1 : 3) void attn_mfma_kernel(PlanePtrs planes, const float *__restrict__ bias_lh,
                                                           const float *__restrict__ tscale_h,
                                                           half_t *__restrict__ O, const AttnItem *__restrict__ items,
                                                           int H, int d, int D, int64_t ws_rows) {
  constexpr bool KSPLIT = KP > 1;
  static_assert(!SEQ || (KP == 4 && !SOFTMAX), "the key-ordered split is the KP = 4 one, pointwise");
  constexpr int NP = KP == 2 ? 2 : 1;  // partial outputs per wavefront
  constexpr int NW = KSPLIT ? 8 : 4;   // wavefronts per workgroup that compute
  constexpr bool FEEDERS = KP == 4;    // four more that make the requests
  constexpr int QG = NW / KP;          // groups
  constexpr int QT = 32 * QG;          // query rows per workgroup (one 32-row MFMA block per group)
  static_assert(QT == (KP == 4 ? kAttnQTileLatency : KP == 2 ? kAttnQTileLatencyWide : kAttnQTileBf16), "the planner's query tiles");
  static_assert(KP == 1 || KP * NP == 4, "the latency configuration sums in four partial outputs");
  constexpr bool BRING = KP == 1 && (DH == 64 || !SOFTMAX);   // bias: a ring over all tiles in four copies, beside the stages, instead of a window in each
  constexpr int NSTAGE = KP == 2 ? 4 : KP == 4 || BRING ? 2 : 3;  // LDS stages (ring)
  constexpr int KT = KH * KP;          // keys per LDS stage
  constexpr int BW = QT + KT;          // bias window per key tile: slot u holds bias[q_first + QT-1 - k0 - u]
  static_assert(BW <= 64 * NW, "one 64-slot window request per wavefront");
  constexpr int KS = DH / 16;          // k-steps of the Q K^T product
  constexpr int DB = DH / 32;          // 32-row blocks of O^T
  constexpr int KCH = DH / 8;          // 16-byte chunks per K row (8 or 4)
  constexpr int KSH = KCH == 8 ? 1 : 2;            // K rows per 256 bytes = 1 << KSH
  constexpr int VCH = KT / 8;          // 16-byte chunks per V^T row (32, 16 or 8)
  constexpr int VSH = VCH == 8 ? 1 : 0;            // V^T rows per 256 bytes = 1 << VSH (a row of 16 chunks is 256 bytes, one of 32 chunks 512)
  constexpr int VKEY = VCH == 8 ? 7 : 15;          // swizzle key: XORed into the chunk index inside 256 bytes
  constexpr int K_BYTES = KT * DH * 2;             // K tile [KT keys][DH]
  constexpr int V_BYTES = DH * KT * 2;             // V^T tile [DH][KT keys]
  constexpr int BCOPY = (256 + 64) * 4 + 64;       // bytes of a copy: 256 slots, the first 64 again behind them, and a quarter of the banks to the next copy
  constexpr int WCOPY = BW * 4 + 64;               // FEEDERS: the window in four copies too, BW slots and a quarter of the banks each
  constexpr int W_BYTES = BRING ? 0 : FEEDERS ? 4 * WCOPY : NW * 256;    // bias window: 64 slots per wavefront (BW <= 64 NW of them are used)
  constexpr int STAGE = K_BYTES + V_BYTES + W_BYTES;
  constexpr bool P_OVER_K = SEQ && K_BYTES >= NW * 4096;   // where the weights of a tile go: over its K, or behind the stages
  static_assert(K_BYTES % 1024 == 0 && V_BYTES % 1024 == 0 && STAGE % 256 == 0, "stage parts start on 256-byte boundaries");
  static_assert(!FEEDERS || (W_BYTES == 4 * 1344 && BW % 64 == 0), "key_split_lds_bytes");
  static_assert(QT * DH * 2 <= NSTAGE * STAGE, "output patches fit in the tile buffers");
  // the stages; the output patches of the wavefronts reuse them once the key loop is over.  The latency
  // configuration needs more than the 64 KB a static array may have and takes its stages from dynamic LDS.
  extern __shared__ __attribute__((aligned(256))) char lds_dynamic[];
  __shared__ __attribute__((aligned(256))) char lds_static[KSPLIT ? 256 : NSTAGE * STAGE + (BRING ? 4 * BCOPY : 0)];
  char *const lds = KSPLIT ? lds_dynamic : lds_static;

  const int head = blockIdx.x % H;
  AttnItem it = items[blockIdx.x / H >> (SEQ ? 1 : 0)];
  if constexpr (SEQ) {                 // an item of 128 rows is two workgroups, the one with more keys first
    const int off = (blockIdx.x / H & 1) ? 0 : QT;
    if (off >= it.n_q) return;
    it.q_row += off;
    it.n_q = min(QT, it.n_q - off);
    if (!it.is_cand) {
      it.q_pos += off;
      it.n_kv = it.q_pos + it.n_q;
    }
  }
  const int tid = threadIdx.x, lane = tid & 63;
  // wavefront index as a scalar: every branch on it is then a uniform (scalar) branch
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, lhalf = lane >> 5;

  const half_t *Vt = (const half_t *)planes.v + (int64_t)head * DH * ws_rows;   // [DH][ws_rows]
  const half_t *Qp = (const half_t *)planes.q + head * DH;                      // [row][d]
  const half_t *Kp = (const half_t *)planes.k + head * DH;
  const float *bias = bias_lh + (int64_t)head * D;

  // this wavefront's 32 query rows and (latency configuration) its 64 keys of every key tile
  const int q_group = KSPLIT ? wave / KP : wave;
  const int k_part = KSPLIT ? wave % KP : 0;
  const int q_local0 = q_group * 32;
  const bool wave_active = q_local0 < it.n_q;
  const int my_q_local = q_local0 + l32;
  const bool row_valid = my_q_local < it.n_q;
  f16x8 fq[KS];                        // Q fragments (B operand of S^T): row = my query, k = 16*s + 8*lhalf + 0..7
  int n_vis;
  int64_t q_row_clamped;
  {
    const int64_t row = it.q_row + (row_valid ? my_q_local : it.n_q - 1);   // clamped for loads
    const int q_index = it.is_cand ? it.L : it.q_pos + my_q_local;
    n_vis = visible_history(it.is_cand, q_index, it.L);
    q_row_clamped = row;
  }
  // SEQ: which wavefront of a group adds up which feature block (one per SIMD; -1: none)
  const int sum_b = SEQ && k_part - 2 * q_group >= 0 && k_part - 2 * q_group < DB ? k_part - 2 * q_group : -1;
  const int wave_vis_min = it.is_cand ? it.L : it.q_pos + q_local0 + 1;
  const int wave_vis_max = it.is_cand ? it.L : it.q_pos + q_local0 + 32;

  constexpr int ODB = SEQ ? 1 : DB;    // feature blocks that a wavefront adds up
  f32x16 oacc[NP][ODB];
#pragma unroll
  for (int p = 0; p < NP; ++p)
#pragma unroll
    for (int b = 0; b < ODB; ++b)
#pragma unroll
      for (int e = 0; e < 16; ++e) oacc[p][b][e] = 0.f;
  // softmax state of my query row, per partial output (both lanes of a pair hold the same maximum; each holds the sum over its keys)
  // Finite stand-ins for -inf, so that no inf - inf can arise: a masked key's raw logit is kNeg; the running
  // maximum starts below kNeg * tscale for any sensible temperature, so a row whose keys so far were all masked
  // holds weights exp2(0) that the first real maximum scales to zero (every row sees key 0 of tile 0 or itself).
  constexpr float kNeg = -1.0e30f;
  const float ts = SOFTMAX ? tscale_h[head] : 0.f;
  float m_run[NP], l_run[NP];
#pragma unroll
  for (int p = 0; p < NP; ++p) { m_run[p] = -3.0e38f; l_run[p] = 0.f; }

  const int n_tiles = (it.n_kv + KT - 1) / KT;
  const int q_first = it.is_cand ? it.L : it.q_pos;     // position of query row 0 of the workgroup tile

  // ---- LDS-DMA sources.  One instruction of a wavefront fills 1 KB of LDS, lane p at byte 16 p.
  // K tile: 1 KB = 64 / KCH rows; lane p owns physical chunk p % KCH of row p / KCH and fetches the logical
  // chunk the swizzle maps there (chunk ^ key, key = row bits above the rows that share 256 bytes).
  // V^T tile: 1 KB = 64 / VCH feature rows of 2 KT bytes, same scheme.
  // Instruction I = wave + 4 i of either tile belongs to this wavefront.
  typedef __attribute__((address_space(1))) const void gvoid;
  typedef __attribute__((address_space(3))) void lvoid;
  // Instruction I of a tile belongs to wavefront I % NW; going from I to I + NW leaves the swizzle key
  // unchanged, so a wavefront keeps one lane pointer per tile kind (for the tile to request next) and adds
  // scalar offsets for its further instructions.  Bias window: slots 64 w .. 64 w + 63 by wavefront w.
  constexpr int NKI = K_BYTES / 1024, NVI = V_BYTES / 1024;
  static_assert(NKI % NW == 0 && NVI % NW == 0, "every wavefront issues the same number of requests per tile");
  static_assert((NW * (64 / KCH)) % (KCH << KSH) == 0 && (NW * (64 / VCH)) % ((VKEY + 1) << VSH) == 0, "swizzle keys do not depend on the instruction");
  constexpr int REQ = NKI / NW + NVI / NW + 1;       // requests per wavefront and tile
  // Addresses are a wave-uniform base (advanced per tile with scalar arithmetic) plus a 32-bit lane offset that
  // never changes: the request instruction takes them as scalar base + vector offset, and a tile costs no
  // vector address arithmetic.  (Lane offsets stay below 2^32: at most 64 rows of d, resp. DH rows of ws_rows.)
  const char *bK = (const char *)(Kp + (int64_t)it.kv_row * d);
  const char *bV = (const char *)(Vt + it.kv_row);
  const int rw = wave % NW;              // the share of the requests (a feeder has two: of wavefronts rw and rw + 4)
  uint32_t oK, oV;
  // (candidate tiles shift the window by one slot: all their rows read it at the same slots, which then start on a
  // 16-byte boundary and leave as four-float reads)
  constexpr bool BCOPIES = BRING || FEEDERS;
  const int dW0 = q_first + (QT - 1) + (!BCOPIES && it.is_cand ? 1 : 0) - (BCOPIES ? rw + lane : rw * 64 + lane);   // distance held by window slot 64 w + lane in tile 0 (copies: slot lane of copy w)
  int sW = 0;                                                 // keys the next tile to request lies behind tile 0 (scalar)
  {
    const int row = rw * (64 / KCH) + lane / KCH;
    const int c = (lane % KCH) ^ ((row >> KSH) & (KCH - 1));
    oK = (uint32_t)(row * d + c * 8) * 2u;
  }
  {
    const int row = rw * (64 / VCH) + lane / VCH;
    const int c = (lane % VCH) ^ ((row >> VSH) & VKEY);
    oV = (uint32_t)((int64_t)row * ws_rows + c * 8) * 2u;
  }
  auto request_tile = [&](int stage) {
    char *sb = lds + stage * STAGE;
    // (the empty asm keeps the widening of the offsets next to the requests: hoisted out of the loop, the
    // compiler would add full 64-bit vector addresses per request again)
    asm volatile("" : "+v"(oK), "+v"(oV));
#pragma unroll
    for (int i = 0; i < NKI / NW; ++i)
      __builtin_amdgcn_global_load_lds((gvoid *)(bK + (int64_t)(i * NW * (64 / KCH)) * d * 2 + oK), (lvoid *)(sb + (rw + NW * i) * 1024), 16, 0, 0);
#pragma unroll
    for (int i = 0; i < NVI / NW; ++i)
      __builtin_amdgcn_global_load_lds((gvoid *)(bV + (int64_t)(i * NW * (64 / VCH)) * ws_rows * 2 + oV), (lvoid *)(sb + K_BYTES + (rw + NW * i) * 1024), 16, 0, 0);
    if constexpr (BCOPIES) return;
    // every wavefront issues one window request, so that all of them have the same number of requests in
    // flight per tile (slots past the window are filled too and never read)
    uint32_t oW = (uint32_t)max(0, min(D - 1, dW0 - sW)) * 4u;
    asm volatile("" : "+v"(oW));
    __builtin_amdgcn_global_load_lds((gvoid *)((const char *)bias + oW), (lvoid *)(sb + K_BYTES + V_BYTES + rw * 256), 4, 0, 0);
  };
  // Bias ring: slots 64 b .. 64 b + 63 of the absolute index p, copy w by wavefront w; physical slot p % 256, the first 64 of them twice.
  auto request_bias = [&](int b) {
    uint32_t oW = (uint32_t)max(0, min(D - 1, dW0 - 64 * b)) * 4u;
    asm volatile("" : "+v"(oW));
    char *dst = lds + NSTAGE * STAGE + rw * BCOPY + (b & 3) * 256;
    __builtin_amdgcn_global_load_lds((gvoid *)((const char *)bias + oW), (lvoid *)dst, 4, 0, 0);
    if ((b & 3) == 0) __builtin_amdgcn_global_load_lds((gvoid *)((const char *)bias + oW), (lvoid *)(dst + 1024), 4, 0, 0);
  };
  auto next_tile = [&]() {
    bK += (int64_t)KT * d * 2;
    bV += KT * 2;
    sW += KT;
  };

  if constexpr (FEEDERS) {
    // A feeder requests the tiles, two shares of them, one tile ahead of the others and in step with them: they meet at the same barriers.
    if (wave >= NW) {
      static_assert(NSTAGE == 2 && NW == 8, "two stages, eight shares");
      const int row2 = (rw + 4) * (64 / VCH) + lane / VCH, k2 = (rw + 4) * (64 / KCH) + lane / KCH;
      uint32_t oK2 = (uint32_t)(k2 * d + ((lane % KCH) ^ ((k2 >> KSH) & (KCH - 1))) * 8) * 2u;
      uint32_t oV2 = (uint32_t)((int64_t)row2 * ws_rows + ((lane % VCH) ^ ((row2 >> VSH) & VKEY)) * 8) * 2u;
      auto request_second = [&](int stage) {
        char *sb = lds + stage * STAGE;
        asm volatile("" : "+v"(oK2), "+v"(oV2));
#pragma unroll
        for (int i = 0; i < NKI / NW; ++i)
          __builtin_amdgcn_global_load_lds((gvoid *)(bK + (int64_t)(i * NW * (64 / KCH)) * d * 2 + oK2), (lvoid *)(sb + (rw + 4 + NW * i) * 1024), 16, 0, 0);
#pragma unroll
        for (int i = 0; i < NVI / NW; ++i)
          __builtin_amdgcn_global_load_lds((gvoid *)(bV + (int64_t)(i * NW * (64 / VCH)) * ws_rows * 2 + oV2), (lvoid *)(sb + K_BYTES + (rw + 4 + NW * i) * 1024), 16, 0, 0);
#pragma unroll
        for (int j = 0; j < BW / 64; ++j) {                // copy rw of the window
          uint32_t oW = (uint32_t)max(0, min(D - 1, dW0 - 64 * j - sW)) * 4u;
          asm volatile("" : "+v"(oW));
          __builtin_amdgcn_global_load_lds((gvoid *)((const char *)bias + oW), (lvoid *)(sb + K_BYTES + V_BYTES + rw * WCOPY + j * 256), 4, 0, 0);
        }
      };
      for (int t = 0; t < n_tiles; ++t) {
        if (t == 0) {
          request_tile(0);
          request_second(0);
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();                      // tile t has landed, and everybody has left tile t - 1
        if (t + 1 < n_tiles) {
          next_tile();
          request_tile((t + 1) & 1);
          request_second((t + 1) & 1);
        }
        if constexpr (SEQ) {
          if (P_OVER_K) __builtin_amdgcn_s_barrier();      // (the one behind S^T)
          __builtin_amdgcn_s_barrier();                    // (the weights of the tile are complete)
        }
      }
      __builtin_amdgcn_s_barrier();                        // the keys are done
#pragma unroll
      for (int i = 0; i < (SEQ ? 1 : 2); ++i) __builtin_amdgcn_s_barrier();   // (those of the end)
      return;
    }
  }

  // Window slot of (my row, key 0 of the tile) is QT-1 - m + 8*lhalf with m the row's index in the
  // workgroup tile; keys further right sit at increasing slots.  Candidate rows all sit at the same distance
  // from a key (m = 0), and their window is shifted by one slot: QT + 8*lhalf, a 16-byte boundary.
  // Ring: value p of the index is p & ~3 of copy p & 3, so that a lane's four consecutive values are one aligned 16-byte read whatever its row.
  const int bias_idx = BCOPIES ? (QT - 1) - (it.is_cand ? 0 : my_q_local) + 8 * lhalf : it.is_cand ? QT + 8 * lhalf : (QT - 1) - my_q_local + 8 * lhalf;
  const int ring_copy = BRING ? NSTAGE * STAGE + (bias_idx & 3) * BCOPY : K_BYTES + V_BYTES + (bias_idx & 3) * WCOPY, ring_at = (bias_idx & ~3) * 4;
  // fragment byte offsets inside a stage.  K (A operand of S^T): MFMA row m takes key pi32(m); per 32-key
  // block j the row advances by 32 (key bits 0..4 unchanged, so the swizzle key is the same).  V^T (A
  // operand of O^T): row = feature 32 b + l32, chunk = key / 8.
  // The swizzled chunk (c ^ key) << 4 never carries into the row bits, so an address is
  // (row base | key << 4) ^ (c << 4): one XOR with a constant per fragment.
  const int krow = pi32(l32);
  const int ka0 = (krow * (DH * 2)) | (((((krow >> KSH) & (KCH - 1)) ^ lhalf) << 4));
  const int va0 = (K_BYTES + l32 * (KT * 2)) | (((((l32 >> VSH) & VKEY) ^ lhalf) << 4));

  // Two stages: requests one tile ahead, all of them landed at the barrier that opens a tile.  Three or four: two tiles ahead, and past the last tile
  // the requests repeat it (into a free stage), so that "at most REQ requests outstanding" always means "tile t has landed".
  if (BRING && n_tiles > 0) {
    request_tile(0);
#pragma unroll
    for (int b = 0; b < 3; ++b) request_bias(b);
  } else if (!FEEDERS && n_tiles > 0) {
    request_tile(0);
    if (n_tiles > 1) next_tile();
    request_tile(1);
  }
  // The query fragments are requested behind the first tiles, not ahead of them: the tiles are what the first
  // step waits for.  (Where the waits below count requests, they do so in order: with at most REQ outstanding, the query loads and
  // every tile before the newest have landed.)
#pragma unroll
  for (int s = 0; s < KS; ++s) fq[s] = *(const f16x8 *)(Qp + q_row_clamped * d + s * 16 + lhalf * 8);
  // One key tile.  The stage is a compile-time constant (the tile loop below is unrolled over the ring), so
  // every fragment address is a fixed lane offset plus an immediate and costs no instruction.
  auto tile_step = [&](auto stage_c, const int t) {
    constexpr int ST = decltype(stage_c)::value;
    constexpr int P = NP == 2 ? ST & 1 : 0;          // partial output (the ring is even there: the stage has the tile's parity)
    const char *sb = lds + ST * STAGE;
    // tile t has landed for this wavefront; past the barrier it has landed for all of them, and everybody
    // has left tile t-1, whose stage the next request overwrites
    if (FEEDERS) asm volatile("" ::: "memory");
    else if (BRING) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    else if (REQ == 5) asm volatile("s_waitcnt vmcnt(5)" ::: "memory");
    else if (REQ == 3) asm volatile("s_waitcnt vmcnt(3)" ::: "memory");
    else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    if constexpr (BRING) {
      if (t + 1 < n_tiles) {
        next_tile();
        request_tile(ST ^ 1);
        request_bias(t + 3);
      }
    } else if constexpr (!FEEDERS) {
      if (t + 2 < n_tiles) next_tile();
      request_tile((ST + 2) % NSTAGE);
    }
    __builtin_amdgcn_sched_barrier(0);   // the requests stay ahead of the tile's arithmetic
#pragma unroll 1
    for (int u = k_part; u < k_part + 1; ++u) {
    const int k0 = t * KT + u * KH;
    const bool seen = wave_active && k0 < wave_vis_max;
    if (P_OVER_K && !seen) __builtin_amdgcn_s_barrier();     // (the one behind S^T)
    if (seen) {
      const char *kb = sb + u * (KH * DH * 2);                 // K rows of this block
      const int vau = va0 ^ (u << 7);                          // V^T: chunks 8 u .. 8 u + 7 of each row
      const bool need_mask = k0 + KH > wave_vis_min;
      // key 32 j + 16 (e >> 3) + 8 lhalf + (e & 7) of this block is visible to my row iff its constant part is below vis_lim
      const int vis_lim = n_vis - k0 - 8 * lhalf;
      {
        // ---- S^T = K Q^T: blocks [j], j = 32-key half.  Fragment reads run one group
        // ahead of the MFMAs that use them (and the first V^T group is fetched behind the last K group),
        // so LDS latency hides behind matrix work instead of being paid once per group.
        f32x16 sacc[2];
        {
          // one address register, the 32 reads use immediate offsets (the empty asm keeps the compiler
          // from folding constant parts of the address into every read as a separate add)
          typedef const __attribute__((address_space(3))) float *lds_cfloat;
          typedef const __attribute__((address_space(3))) f32x4 *lds_cf4;
          lds_cfloat bp = BRING ? (lds_cfloat)(lds + ring_copy + ((ring_at + 4 * k0) & 1023)) : FEEDERS ? (lds_cfloat)(sb + ring_copy + ring_at + 4 * KH * u) : (lds_cfloat)(sb + K_BYTES + V_BYTES) + (bias_idx + u * KH);
          asm volatile("" : "+v"(bp));
          if (BCOPIES || it.is_cand) {
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
              for (int g = 0; g < 4; ++g) {
                const f32x4 v = *(lds_cf4)(bp + 32 * j + 16 * (g >> 1) + 4 * (g & 1));
#pragma unroll
                for (int q = 0; q < 4; ++q) sacc[j][4 * g + q] = v[q];
              }
          } else {
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
              for (int e = 0; e < 16; ++e) sacc[j][e] = bp[32 * j + 16 * (e >> 3) + (e & 7)];
          }
        }
        f16x8 fk[2][2], fv[2][DB];
#pragma unroll
        for (int j = 0; j < 2; ++j) fk[0][j] = *(const f16x8 *)(kb + j * (32 * DH * 2) + ka0);
#pragma unroll
        for (int s = 0; s < KS; ++s) {
          if (s + 1 < KS) {
#pragma unroll
            for (int j = 0; j < 2; ++j)
              fk[(s + 1) & 1][j] = *(const f16x8 *)(kb + j * (32 * DH * 2) + (ka0 ^ ((s + 1) << 5)));
          } else if (!SEQ) {
#pragma unroll
            for (int b = 0; b < DB; ++b) fv[0][b] = *(const f16x8 *)(sb + b * (32 * KT * 2) + vau);
          }
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int j = 0; j < 2; ++j)
            sacc[j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(fk[s & 1][j], fq[s], sacc[j], 0, 0, 0);
          __builtin_amdgcn_sched_barrier(0);
        }
        if constexpr (P_OVER_K) {
          __builtin_amdgcn_s_barrier();                      // everybody has read K: its place takes the weights
          __builtin_amdgcn_sched_barrier(0);
        }
        // ---- P^T = silu(S^T) (the bias is already in the accumulators), or the softmax numerators
        f16x8 fp[4];
        if constexpr (SOFTMAX) {
          // maximum of the raw (halved) logits first: the temperature scale is positive, so it commutes with the max.
          // Maxima and sums are taken in four independent chains (the 32 values of a lane would otherwise form one
          // chain of dependent instructions).
          if (need_mask) {
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
              for (int e = 0; e < 16; ++e) {
                sacc[j][e] = 32 * j + 16 * (e >> 3) + (e & 7) < vis_lim ? sacc[j][e] : kNeg;
              }
          }
          // maximum of the lane's 32 logits as a tree of three-input maxima, 10 + 4 + 2 instructions.  (IEEE maximum: for fmaxf on accumulator values the compiler first emits one
          // canonicalising v_max_f32 per value, 53 instructions in all.  No inline assembly here: the compiler does not put the wait that a matrix result needs ahead of one.)
          auto max3 = [](float a, float b, float c) { return __builtin_elementwise_maximum(__builtin_elementwise_maximum(a, b), c); };
          float l1[10], l2[4];
#pragma unroll
          for (int k = 0; k < 10; ++k) {
            const int e = 3 * k;   // values 0..29 in the order sacc[0][0..15], sacc[1][0..13]
            l1[k] = max3(sacc[e >> 4][e & 15], sacc[(e + 1) >> 4][(e + 1) & 15], sacc[(e + 2) >> 4][(e + 2) & 15]);
          }
#pragma unroll
          for (int k = 0; k < 3; ++k) l2[k] = max3(l1[3 * k], l1[3 * k + 1], l1[3 * k + 2]);
          l2[3] = max3(l1[9], sacc[1][14], sacc[1][15]);
          const float l3 = max3(l2[0], l2[1], l2[2]);
          const float mt = __builtin_elementwise_maximum(l3, l2[3]);
          const float m_new = fmaxf(m_run[P], pair_max(mt) * ts);
          // The accumulators are rescaled only when some row of the wavefront has a new maximum; the branch is uniform over the wavefront, and a row without one is multiplied by exactly 1,
          // so that no row's bits depend on the others.
          if (__builtin_amdgcn_ballot_w64(m_new != m_run[P]) != 0) {
            const float sc = __builtin_amdgcn_exp2f(m_run[P] - m_new);
            l_run[P] *= sc;
#pragma unroll
            for (int b = 0; b < DB; ++b)
#pragma unroll
              for (int e = 0; e < 16; ++e) oacc[P][b][e] *= sc;
            m_run[P] = m_new;
          }
          const float nm = -m_new;
          float psum[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int j = 0; j < 2; ++j) {
            float w[16];
#pragma unroll
            for (int e = 0; e < 16; ++e) w[e] = __builtin_amdgcn_exp2f(__builtin_fmaf(sacc[j][e], ts, nm));
#pragma unroll
            for (int e = 0; e < 16; ++e) psum[e & 3] += w[e];
            fp[2 * j] = pack8(w);
            fp[2 * j + 1] = pack8(w + 8);
          }
          const float ps = (psum[0] + psum[1]) + (psum[2] + psum[3]);
          l_run[P] += ps;
        } else {
          // weights -> fragments of 32 keys, masked where a row's horizon runs through the block
          auto finish = [&](int j, f16x2 (&w)[8]) {
            if (need_mask) {
#pragma unroll
              for (int i = 0; i < 8; ++i) {
                const int c = 32 * j + 16 * (i >> 2) + (2 * i & 7);
                const uint32_t b = __builtin_bit_cast(uint32_t, w[i]);
                w[i] = __builtin_bit_cast(f16x2, c + 1 < vis_lim ? b : c < vis_lim ? b & 0xffffu : 0u);
              }
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
              for (int i = 0; i < 8; ++i) fp[2 * j + h][i] = w[4 * h + i / 2][i & 1];
          };
          f16x2 th[2][8];
#pragma unroll
          for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int i = 0; i < 8; ++i) {
              const f16x2 yh = f16x2{(half_t)sacc[j][2 * i], (half_t)sacc[j][2 * i + 1]};
              th[j][i] = yh * yh;
            }
          // maximum of the 16 pairs with the packed three-input maximum (NaN-propagating): 5 + 2 + 1 instructions
          auto max3 = [](f16x2 a, f16x2 b, f16x2 c) { return __builtin_elementwise_maximum(__builtin_elementwise_maximum(a, b), c); };
          const f16x2 m0 = max3(th[0][0], th[0][1], th[0][2]), m1 = max3(th[0][3], th[0][4], th[0][5]);
          const f16x2 m2 = max3(th[0][6], th[0][7], th[1][0]), m3 = max3(th[1][1], th[1][2], th[1][3]);
          const f16x2 m4 = max3(th[1][4], th[1][5], th[1][6]);
          const f16x2 m = __builtin_elementwise_maximum(max3(m0, m1, m2), max3(m3, m4, th[1][7]));
          const half_t mx = __builtin_elementwise_maximum(m[0], m[1]);
          auto all_within = [&](float t2) { return __builtin_amdgcn_ballot_w64(!(mx <= (half_t)t2)) == 0; };     // NaN counts as beyond
          // s + t (B0 + B1 t + ...), stage by stage over eight independent pairs, so that no instruction waits for the one before
          auto polynomial = [&](auto... coefficient) {
            constexpr int N = sizeof...(coefficient);
            const half_t c[N] = {(half_t)coefficient...};
#pragma unroll
            for (int j = 0; j < 2; ++j) {
              f16x2 r[8], w[8];
#pragma unroll
              for (int i = 0; i < 8; ++i) r[i] = __builtin_elementwise_fma(f16x2{c[N - 1], c[N - 1]}, th[j][i], f16x2{c[N - 2], c[N - 2]});
#pragma unroll
              for (int n = N - 3; n >= 0; --n)
#pragma unroll
                for (int i = 0; i < 8; ++i) r[i] = __builtin_elementwise_fma(r[i], th[j][i], f16x2{c[n], c[n]});
#pragma unroll
              for (int i = 0; i < 8; ++i)
#pragma unroll
                for (int h = 0; h < 2; ++h) w[i][h] = (half_t)__builtin_fmaf((float)th[j][i][h], (float)r[i][h], sacc[j][2 * i + h]);
              finish(j, w);
            }
          };
          if (all_within(kPolyT2)) {
            polynomial(4.0f * kPolyA1, 16.0f * kPolyA3, 64.0f * kPolyA5);
          } else if (all_within(kMidT2)) {
            polynomial(kMidB[0], kMidB[1], kMidB[2], kMidB[3], kMidB[4]);
          } else {
#pragma unroll
            for (int j = 0; j < 2; ++j) {
              f16x2 w[8];
#pragma unroll
              for (int i = 0; i < 8; ++i) w[i] = f16x2{(half_t)silu_half_domain(sacc[j][2 * i]), (half_t)silu_half_domain(sacc[j][2 * i + 1])};
              finish(j, w);
            }
          }
        }
        if constexpr (SEQ) {
#pragma unroll
          for (int s2 = 0; s2 < 4; ++s2) *(f16x8 *)(lds + (P_OVER_K ? ST : NSTAGE) * STAGE + (q_group * KP + u) * 4096 + s2 * 1024 + lane * 16) = fp[s2];
        }
        // ---- O^T += V^T P^T; V^T fragments read one group ahead
        if constexpr (!SEQ)
#pragma unroll
        for (int s2 = 0; s2 < 4; ++s2) {
          if (s2 + 1 < 4) {
#pragma unroll
            for (int b = 0; b < DB; ++b)
              fv[(s2 + 1) & 1][b] = *(const f16x8 *)(sb + b * (32 * KT * 2) + (vau ^ ((s2 + 1) << 5)));
          }
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int b = 0; b < DB; ++b)
            oacc[P][b] = __builtin_amdgcn_mfma_f32_32x32x16_f16(fv[s2 & 1][b], fp[s2], oacc[P][b], 0, 0, 0);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    }
    }
    if constexpr (SEQ) {
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      __builtin_amdgcn_s_barrier();                          // the weights of the tile are complete
      __builtin_amdgcn_sched_barrier(0);
      if (sum_b >= 0 && wave_active) {
        // The tile's keys in order, 16 a product, the visible 64-key blocks of them: as one wavefront alone adds them up.  (As built, the reads three products ahead are
        // waited for at each block's branch.)
        const char *pp = lds + (P_OVER_K ? ST : NSTAGE) * STAGE + q_group * (KP * 4096) + lane * 16;
        const char *vp = sb + sum_b * (32 * KT * 2);
        f16x8 pw[4], vw[4];
        auto fetch = [&](int i) {
          pw[i & 3] = *(const f16x8 *)(pp + i * 1024);
          vw[i & 3] = *(const f16x8 *)(vp + (va0 ^ (i << 5)));
        };
        const int n_blk = min(KP, (wave_vis_max - t * KT + KH - 1) / KH);
#pragma unroll
        for (int i = 0; i < 3; ++i) fetch(i);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int b = 0; b < KP; ++b) {
          if (b < n_blk) {
#pragma unroll
            for (int s2 = 0; s2 < 4; ++s2) {
              const int i = 4 * b + s2;
              if (i + 3 < 4 * KP) fetch(i + 3);
              __builtin_amdgcn_sched_barrier(0);
              oacc[0][0] = __builtin_amdgcn_mfma_f32_32x32x16_f16(vw[i & 3], pw[i & 3], oacc[0][0], 0, 0, 0);
              __builtin_amdgcn_sched_barrier(0);
            }
          }
        }
      }
    }
  };
  for (int t = 0; t < n_tiles; t += NSTAGE) {
    tile_step(std::integral_constant<int, 0>{}, t);
    if (t + 1 < n_tiles) tile_step(std::integral_constant<int, 1>{}, t + 1);
    if constexpr (NSTAGE > 2)
      if (t + 2 < n_tiles) tile_step(std::integral_constant<int, 2>{}, t + 2);
    if constexpr (NSTAGE > 3)
      if (t + 3 < n_tiles) tile_step(std::integral_constant<int, 3>{}, t + 3);
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the repeated requests of the tail have landed
  __builtin_amdgcn_s_barrier();          // everybody has left the last tile: the stages become output patches

  // ---- candidates: the row itself is one more key, at distance 0.  The wavefront multiplies its 32
  // candidate rows against themselves and keeps the diagonal.  (Latency configuration: in the last partial output.)
  if (it.is_cand && wave_active && (SEQ ? sum_b >= 0 : k_part == KP - 1)) {
    constexpr int P = NP - 1;
    const float b0 = bias[0];
    const int64_t base_row = it.q_row + q_local0;   // multiple of 32 inside the padded workspace
    f32x16 sacc;
#pragma unroll
    for (int e = 0; e < 16; ++e) sacc[e] = b0;
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      const f16x8 fk = *(const f16x8 *)(Kp + (base_row + pi32(l32)) * d + s * 16 + lhalf * 8);
      sacc = __builtin_amdgcn_mfma_f32_32x32x16_f16(fk, fq[s], sacc, 0, 0, 0);
    }
    float p[16];
    if constexpr (SOFTMAX) {
      // the diagonal element of my query sits in one lane of the pair
      float ys = kNeg;
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int kv_local = 16 * (e >> 3) + 8 * lhalf + (e & 7);
        ys = kv_local == l32 ? sacc[e] * ts : ys;
      }
      const bool mine = ys > kNeg;
      const float m_new = fmaxf(m_run[P], pair_max(ys));
      const float sc = __builtin_amdgcn_exp2f(m_run[P] - m_new);
      const float pself = mine ? __builtin_amdgcn_exp2f(ys - m_new) : 0.f;
      m_run[P] = m_new;
      l_run[P] = l_run[P] * sc + pself;
#pragma unroll
      for (int b = 0; b < DB; ++b)
#pragma unroll
        for (int e = 0; e < 16; ++e) oacc[P][b][e] *= sc;
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int kv_local = 16 * (e >> 3) + 8 * lhalf + (e & 7);
        p[e] = (kv_local == l32 && row_valid) ? pself : 0.f;
      }
    } else {
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const int kv_local = 16 * (e >> 3) + 8 * lhalf + (e & 7);
      p[e] = (kv_local == l32 && row_valid) ? silu_half_domain(sacc[e]) : 0.f;
    }
    }
    const f16x8 fps[2] = {pack8(p), pack8(p + 8)};
#pragma unroll
    for (int s2 = 0; s2 < 2; ++s2)
#pragma unroll
      for (int b = 0; b < ODB; ++b) {
        const f16x8 fv = *(const f16x8 *)(Vt + (int64_t)(32 * (SEQ ? sum_b : b) + l32) * ws_rows + base_row + s2 * 16 + lhalf * 8);
        oacc[P][b] = __builtin_amdgcn_mfma_f32_32x32x16_f16(fv, fps[s2], oacc[P][b], 0, 0, 0);
      }
  }

  // ---- write O[q][head*DH + dd]; accumulator element e of block b: dd = 32b + 8*(e/4) + 4*lhalf + e%4.
  // Only two lanes share a query row there (16 contiguous bytes per row and store instruction, and the
  // write path is bound by the number of requests), so each wavefront transposes its 32 x DH patch
  // through LDS (16-byte chunks XOR-swizzled by row; every wavefront is past the barrier that closes the key
  // loop, nobody reads the tile buffers any more) and stores 16 bytes per lane, a whole head row of
  // 2*DH bytes per group of lanes.
  constexpr int CPR = DH / 8;                       // 16-byte chunks per patch row
  constexpr int RPI = 64 / CPR;                     // patch rows per store instruction
  char *pb = lds + q_group * (32 * DH * 2);
  auto pkey = [](int row) { return CPR == 8 ? (row >> 1) & 7 : (row >> 2) & 3; };   // spreads 16 rows over 256 bytes
  auto to_patch = [&](int b, int g, const f32x4 o) {
    f16x4 v;
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = to_f16_sat(o[i]);
    const int c = 4 * b + g;
    *(f16x4 *)(pb + l32 * (DH * 2) + ((c ^ pkey(l32)) << 4) + 8 * lhalf) = v;
  };
  const int rl = lane / CPR, c = lane % CPR;
  half_t *obase = O + (int64_t)it.q_row * d + head * DH + c * 8;
  auto store_rows = [&](int t) {
    const int row = t * RPI + rl;
    const f16x8 v = *(const f16x8 *)(pb + row * (DH * 2) + ((c ^ pkey(row)) << 4));
    if (q_local0 + row < it.n_q) store_once<NT>(v, (f16x8 *)(obase + (int64_t)(q_local0 + row) * d));
  };
  // latency configuration: factors of the four partial outputs (softmax: to the common maximum, and divided by the row's sum)
  auto part_factors = [&](const float2 (&ml)[4], float (&sc)[4]) {
    const float m_all = fmaxf(fmaxf(ml[0].x, ml[1].x), fmaxf(ml[2].x, ml[3].x));
    float l_all = 0.f;
#pragma unroll
    for (int p = 0; p < 4; ++p) {
      sc[p] = __builtin_amdgcn_exp2f(ml[p].x - m_all);
      l_all = __builtin_fmaf(ml[p].y, sc[p], l_all);
    }
    const float lt = pair_sum(l_all);
    const float inv = lt > 0.f ? 1.0f / lt : 0.f;
#pragma unroll
    for (int p = 0; p < 4; ++p) sc[p] *= inv;
  };
  // (multiply-adds written out: left to the compiler, which of two products is rounded first would differ between the kernels)
  auto add_parts = [&](const f32x4 (&v)[4], const float (&sc)[4]) {
    if constexpr (!SOFTMAX) return (v[0] + v[1]) + (v[2] + v[3]);
    f32x4 o;
#pragma unroll
    for (int i = 0; i < 4; ++i) o[i] = __builtin_fmaf(v[0][i], sc[0], v[1][i] * sc[1]) + __builtin_fmaf(v[2][i], sc[2], v[3][i] * sc[3]);
    return o;
  };
  if constexpr (SEQ) {
    if (sum_b >= 0) {
#pragma unroll
      for (int g = 0; g < 4; ++g) to_patch(sum_b, g, f32x4{oacc[0][0][4 * g], oacc[0][0][4 * g + 1], oacc[0][0][4 * g + 2], oacc[0][0][4 * g + 3]});
    }
    __syncthreads();
    if (k_part < 32 / RPI) store_rows(k_part);
  } else if constexpr (KP == 4) {
    // The four wavefronts of a row group leave their partial outputs (and their softmax states) in LDS behind the patches; each
    // adds up a quarter of the features, in the order (0 + 1) + (2 + 3), and stores a quarter of the rows.
    constexpr int PART = DB * 16 * 64 * 4;            // bytes of one wavefront's accumulators
    static_assert(QG * (32 * DH * 2) + NW * (PART + 512) <= NSTAGE * STAGE, "patches and partial outputs fit in the tile buffers");
    char *area = lds + QG * (32 * DH * 2) + q_group * KP * (PART + 512);
    char *mine = area + k_part * (PART + 512);
#pragma unroll
    for (int b = 0; b < DB; ++b)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const f32x4 v = {oacc[0][b][4 * g], oacc[0][b][4 * g + 1], oacc[0][b][4 * g + 2], oacc[0][b][4 * g + 3]};
        *(f32x4 *)(mine + ((b * 4 + g) * 64 + lane) * 16) = v;
      }
    if constexpr (SOFTMAX) *(float2 *)(mine + PART + lane * 8) = float2{m_run[0], l_run[0]};
    __syncthreads();
    float sc[4];
    if constexpr (SOFTMAX) {
      float2 ml[4];
#pragma unroll
      for (int p = 0; p < 4; ++p) ml[p] = *(const float2 *)(area + p * (PART + 512) + PART + lane * 8);
      part_factors(ml, sc);
    }
#pragma unroll
    for (int b = 0; b < DB; ++b) {
      f32x4 v[4];
#pragma unroll
      for (int p = 0; p < 4; ++p) v[p] = *(const f32x4 *)(area + p * (PART + 512) + ((b * 4 + k_part) * 64 + lane) * 16);
      to_patch(b, k_part, add_parts(v, sc));
    }
    __syncthreads();
    if (k_part < 32 / RPI) store_rows(k_part);
  } else if constexpr (KP == 2) {
    // Wavefront k of a group holds partial outputs k and k + 2.  Each leaves the half of the features that its partner adds up (groups
    // 2, 3 for k = 0, else 0, 1) in LDS, adds up its own half, in the same order as above, and stores half of the rows.
    constexpr int HALF = NP * DB * 2 * 1024;          // bytes of half the features of a wavefront's two partial outputs
    static_assert(QG * (32 * DH * 2) + NW * (HALF + NP * 512) <= NSTAGE * STAGE, "patches and partial outputs fit in the tile buffers");
    char *area = lds + QG * (32 * DH * 2) + q_group * KP * (HALF + NP * 512);
    char *mine = area + k_part * (HALF + NP * 512);
    const char *theirs = area + (k_part ^ 1) * (HALF + NP * 512);
    auto leave = [&](auto k_c) {
      constexpr int K = decltype(k_c)::value;
#pragma unroll
      for (int p = 0; p < NP; ++p)
#pragma unroll
        for (int b = 0; b < DB; ++b)
#pragma unroll
          for (int i = 0; i < 2; ++i) {
            const int g = 2 * (K ^ 1) + i;
            const f32x4 v = {oacc[p][b][4 * g], oacc[p][b][4 * g + 1], oacc[p][b][4 * g + 2], oacc[p][b][4 * g + 3]};
            *(f32x4 *)(mine + (((p * DB + b) * 2 + i) * 64 + lane) * 16) = v;
          }
    };
    if (k_part == 0) leave(std::integral_constant<int, 0>{});
    else leave(std::integral_constant<int, 1>{});
    if constexpr (SOFTMAX) {
#pragma unroll
      for (int p = 0; p < NP; ++p) *(float2 *)(mine + HALF + p * 512 + lane * 8) = float2{m_run[p], l_run[p]};
    }
    __syncthreads();
    auto finish = [&](auto k_c) {
      constexpr int K = decltype(k_c)::value;
      float sc[4];
      if constexpr (SOFTMAX) {
        float2 ml[4];
#pragma unroll
        for (int p = 0; p < NP; ++p) {
          ml[2 * p + K] = float2{m_run[p], l_run[p]};
          ml[2 * p + (K ^ 1)] = *(const float2 *)(theirs + HALF + p * 512 + lane * 8);
        }
        part_factors(ml, sc);
      }
#pragma unroll
      for (int b = 0; b < DB; ++b)
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          const int g = 2 * K + i;
          f32x4 v[4];
#pragma unroll
          for (int p = 0; p < NP; ++p) {
            v[2 * p + K] = f32x4{oacc[p][b][4 * g], oacc[p][b][4 * g + 1], oacc[p][b][4 * g + 2], oacc[p][b][4 * g + 3]};
            v[2 * p + (K ^ 1)] = *(const f32x4 *)(theirs + (((p * DB + b) * 2 + i) * 64 + lane) * 16);
          }
          to_patch(b, g, add_parts(v, sc));
        }
    };
    if (k_part == 0) finish(std::integral_constant<int, 0>{});
    else finish(std::integral_constant<int, 1>{});
    __syncthreads();
    constexpr int SPW = 32 / RPI / 2;                 // store instructions per wavefront
#pragma unroll
    for (int t = 0; t < SPW; ++t) store_rows(k_part * SPW + t);
  } else {
    if constexpr (SOFTMAX) {
      const float lt = pair_sum(l_run[0]);
      const float inv = lt > 0.f ? 1.0f / lt : 0.f;
#pragma unroll
      for (int b = 0; b < DB; ++b)
#pragma unroll
        for (int e = 0; e < 16; ++e) oacc[0][b][e] *= inv;
    }
#pragma unroll
    for (int b = 0; b < DB; ++b)
#pragma unroll
      for (int g = 0; g < 4; ++g) to_patch(b, g, f32x4{oacc[0][b][4 * g], oacc[0][b][4 * g + 1], oacc[0][b][4 * g + 2], oacc[0][b][4 * g + 3]});
#pragma unroll
    for (int t = 0; t < 32 / RPI; ++t) store_rows(t);
  }
}

}  // namespace

// The configurations that split the keys need their LDS limit raised once per kernel instance and device (a function attribute, no
// allocation): attn_setup, ahead of any launch.
template <int DH, int KP, bool SEQ = false>
constexpr int key_split_lds_bytes() {   // the stages: K, V^T and the bias window each; the weights of a tile where they do not fit over its K
  return (KP == 4 ? 2 : 4) * (2 * 64 * KP * DH * 2 + (KP == 4 ? 4 * 1344 : 8 * 256)) + (SEQ && 64 * KP * DH * 2 < 8 * 4096 ? 8 * 4096 : 0);
}

template <int DH, bool SM, int KP, bool SEQ = false>
static hipError_t key_split_setup() {
  static std::atomic<uint64_t> done{0};
  return raise_lds_limit(reinterpret_cast<const void *>(&attn_mfma_kernel<DH, SM, KP, false, SEQ>), key_split_lds_bytes<DH, KP, SEQ>(), done);
}

template <int DH, bool SM>
static hipError_t latency_setup() {
  const hipError_t e = key_split_setup<DH, SM, 4>();
  return e != hipSuccess ? e : key_split_setup<DH, SM, 2>();
}

template <int DH, bool SM, int KP>
static void launch_key_split(int grid, PlanePtrs planes, const float *bias_lh, const float *tscale_h, half_t *O,
                             const AttnItem *items, const Shape &sh, hipStream_t s) {
  attn_mfma_kernel<DH, SM, KP, false><<<grid, KP == 4 ? 768 : 512, key_split_lds_bytes<DH, KP>(), s>>>(planes, bias_lh, tscale_h, O, items, sh.H, sh.d, sh.D, sh.ws_rows);
}

hipError_t attn_setup(const Shape &sh) {
  if (!sh.latency) return sh.softmax ? hipSuccess : sh.dh == 32 ? key_split_setup<32, false, 4, true>() : key_split_setup<64, false, 4, true>();
  if (sh.softmax) return sh.dh == 32 ? latency_setup<32, true>() : latency_setup<64, true>();
  return sh.dh == 32 ? latency_setup<32, false>() : latency_setup<64, false>();
}

// Workgroups of 128 rows (tiles x heads) up to which a launch takes the key-ordered split, by the longest history of the pass.  Its workgroups have 64 rows and a
// compute unit each, so up to 128 are one round of them; beyond, it pays only where most tiles are history tiles, whose chains of keys are half as long on average, and the longest
// chain is what the other kernel takes.  Forwards of four layers, one wavefront per group / split (us):
//   1024 + 256, 8 heads: 80 workgroups 153 / 128, 160: 167 / 142, 240: 177 / 164, 320: 202 / 204; 4 heads: 80: 145 / 119, 240: 166 / 154, 320: 176 / 178; 1024 + 1024: 128: 156 / 131, 256: 182 / 182
//   2048 + 256, 8 heads: 144: 222 / 173, 288: 256 / 231, 432: 286 / 291; 3 heads: 108: 196 / 147, 216: 219 / 179, 324: 222 / 210; 8192 + 512, 2 heads: 136: 514 / 300
//   512 + 128, 8 heads: 80: 127 / 113, 120: 132 / 119, 160: 140 / 132, 200: 146 / 145; 4 heads: 160: 131 / 123, 240: 137 / 139
//   320 + 128, 2 heads: 24: 79 / 75, 128: 95 / 95; 128 + 64: 40: 69 / 71, 160: 84 / 105 (a history of one or two 256-key tiles has no chain to shorten)
// Candidate tiles alone (one layer), 4 heads: 512 + 128: 64: 48 / 46, 128: 53 / 53, 160: 59 / 65; 2048 + 128: 64: 87 / 79, 128: 140 / 136, 160: 152 / 169.
constexpr int kAttnSeqHistory = 384, kAttnSeqWorkgroups = 128;                            // from this history on; up to this many workgroups, and where history tiles prevail
constexpr int kAttnSeqLongHistory = 1024, kAttnSeqLongWorkgroups = 240, kAttnSeqLongerHistory = 2048, kAttnSeqLongerWorkgroups = 288;   // up to these
bool attn_key_ordered(int grid, int n_items, int n_cand, int longest) {
  if (longest < kAttnSeqHistory) return false;
  const int limit = longest < kAttnSeqLongHistory || 2 * n_cand > n_items ? kAttnSeqWorkgroups : longest < kAttnSeqLongerHistory ? kAttnSeqLongWorkgroups : kAttnSeqLongerWorkgroups;
  return grid <= limit;
}

void launch_attn_bf16(PlanePtrs planes, const float *bias_lh, const float *tscale_h, void *O, const AttnItem *items,
                      int n_items, int n_cand, int q_tile, int longest, const Shape &sh, hipStream_t s) {
  if (n_items <= 0) return;
  const int grid = n_items * sh.H;
  if (sh.latency) {
#define SPLIT_LAUNCH(DHV, SM, KPV) launch_key_split<DHV, SM, KPV>(grid, planes, bias_lh, tscale_h, (half_t *)O, items, sh, s)
#define SPLIT_CASE(DHV, SM) do { if (q_tile == kAttnQTileLatencyWide) SPLIT_LAUNCH(DHV, SM, 2); else SPLIT_LAUNCH(DHV, SM, 4); } while (0)
    if (sh.softmax) {
      if (sh.dh == 32) SPLIT_CASE(32, true);
      else SPLIT_CASE(64, true);
    } else {
      if (sh.dh == 32) SPLIT_CASE(32, false);
      else SPLIT_CASE(64, false);
    }
#undef SPLIT_CASE
#undef SPLIT_LAUNCH
    return;
  }
  if (!sh.softmax && attn_key_ordered(grid, n_items, n_cand, longest)) {
#define SEQ_LAUNCH(DHV) attn_mfma_kernel<DHV, false, 4, false, true><<<2 * grid, 768, key_split_lds_bytes<DHV, 4, true>(), s>>>(planes, bias_lh, tscale_h, (half_t *)O, items, sh.H, sh.d, sh.D, sh.ws_rows)
    if (sh.dh == 32) SEQ_LAUNCH(32);
    else SEQ_LAUNCH(64);
#undef SEQ_LAUNCH
    return;
  }
  const bool nt = (int64_t)n_items * kAttnQTileBf16 * sh.d * 2 > kStreamBytes;
#define ATTN_LAUNCH(DHV, SM, NTV) attn_mfma_kernel<DHV, SM, 1, NTV><<<grid, 256, 0, s>>>(planes, bias_lh, tscale_h, (half_t *)O, items, sh.H, sh.d, sh.D, sh.ws_rows)
#define ATTN_CASE(DHV, SM) do { if (nt) ATTN_LAUNCH(DHV, SM, true); else ATTN_LAUNCH(DHV, SM, false); } while (0)
  if (sh.softmax) {
    if (sh.dh == 32) ATTN_CASE(32, true);
    else ATTN_CASE(64, true);
  } else {
    if (sh.dh == 32) ATTN_CASE(32, false);
    else ATTN_CASE(64, false);
  }
#undef ATTN_CASE
#undef ATTN_LAUNCH
}

}  // namespace flame
