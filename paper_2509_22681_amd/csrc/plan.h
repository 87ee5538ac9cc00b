// Host-side planner of the jagged GR forward: integer work only, no HIP.
//
// A batch of requests (history length L_i, candidate count M_i: Sections 1 and 3.3 of the paper)
// becomes a list of segments laid out in one padded token workspace, plus the work lists the
// kernels consume.  The mask and the relative-position bucket function (Section 3.2's customised
// mask; bucket function as documented in flame_gr.h) also live here so that host tests can
// compare them bit for bit with an independent implementation.
#pragma once
#include <cstdint>
#include <string>
#include <vector>

#include "../../include/flame_gr.h"

namespace flame {

constexpr int kRowAlign = 64;  // history part and candidate part of a segment start on multiples of this
constexpr int kSpareRows = 256;  // rows at the end of every workspace that no plan places a segment in

struct Segment {
  int32_t req;        // request index in the caller's batch
  int32_t L;          // history length
  int32_t cand_begin; // first candidate (relative to the request) handled here
  int32_t M;          // number of candidates handled here
  int32_t row_start;  // first workspace row (history row 0)
  int32_t Lp;         // L rounded up to kRowAlign: candidates start at row_start + Lp
  int32_t Mp;         // M rounded up to kRowAlign
  int32_t group;      // stream group
  int64_t cost;       // model cost, 10*N*d^2 + 4*P*d
};

// One 64-row block of the workspace: where its rows come from.
struct RowBlock {
  int32_t src_row;  // first source row in history_emb (kind 0) or cand_emb (kind 1)
  int32_t n_valid;  // rows [0, n_valid) of the block are real tokens, the rest is zero padding
  int32_t kind;     // 0 history, 1 candidate
  int32_t seg;      // owning segment
};

// Query rows per attention work item.
constexpr int kAttnQTileBf16 = 128;         // MFMA path, throughput configuration
constexpr int kAttnQTileLatency = 64;       // latency configuration: four wavefronts per group of 32 rows
constexpr int kAttnQTileLatencyWide = 128;  // the same for batches that fill the chip: two wavefronts per group, the same bits
constexpr int kAttnQTileF32 = 64;           // fp32 path

// One attention work item: a tile of query rows of one segment (all heads run it).
struct AttnItem {
  int32_t q_row;    // workspace row of the first query
  int32_t n_q;      // valid query rows in the tile (<= tile height)
  int32_t kv_row;   // workspace row of the segment's history row 0
  int32_t L;        // history length of the segment
  int32_t q_pos;    // position of the first query row: its history index, or L for candidate tiles
  int32_t is_cand;  // 1: rows are candidates (see all L history keys + themselves)
  int32_t n_kv;     // number of history keys the tile can see (causal upper bound)
  int32_t pad;
};

// Attention tiles run in request order, so that the tiles of a request find its K and V in the caches; the last kTailItems of a group run
// longest first instead, whatever their request, so that a launch ends on short tiles and not on one long chain of keys.
// Per launch, request order against this: 64 users of 256 + 128, 3 heads 16.9 -> 15.1 us; a forward of 32 x (512 + 128) 259 -> 250 us.  All
// tiles longest first loses more in the caches than it gains once the batch is large: 128 production requests 61.9 -> 68.7 ms, with the last
// 384 tiles 62.0.
constexpr int kTailItems = 384;

// Latency handles: from this many workgroups of 64 query rows (tiles x heads) on a pass runs on tiles of 128 rows.  With fewer, a workgroup
// has a compute unit to itself (or shares it little) and the shorter chain of key tiles counts; with more, the chip is full and the K and V
// traffic does, which a 64-row workgroup makes twice per query row.  Microseconds per launch, tiles of 64 / 128 rows:
//   heads of 64: one request of 4096 + 2000, 8 heads (768 workgroups) 56.4 / 58.5, of 8192 + 512 (1088) 118.6 / 116.0; requests of 1024 + 256:
//     8 (1280) 35.7 / 31.3, 16 (2560) 77.5 / 56.7, 32 (5120) 152 / 110
//   heads of 32: 2573 + 217, 16 heads (720) 27.4 / 27.6, 4096 + 2000 (1536) 79.6 / 71.8; 1024 + 256: 4 (1280) 27.2 / 23.5, 16 (5120) 113 / 82
//   heads of 32, softmax, whose chain has the exponentials on top: 4096 + 300 (1104) 42.9 / 49.0, 4096 + 2000 (1536) 65.9 / 71.3, 8192 + 512 (2176)
//     132.1 / 131.1; 1024 + 256: 6 (1920) 31.4 / 27.5
// Histories of up to 128 keys are one step on either tile, so that 128 rows pay as soon as there is a workgroup for every compute unit: 4 layers,
// d = 512, 16 x (128 + 64) (384 workgroups) 155 / 144 us per forward, 4 x (128 + 128) (128) 112 / 116.
constexpr int kLatencyWideTiles = 1280;
constexpr int kLatencyWideTilesSoftmax32 = 2048;
constexpr int kLatencyWideTilesShort = 256;
constexpr int kLatencyShortHistory = 128;

struct Group {
  int32_t row_begin, row_end;          // workspace rows [begin, end) of this stream group (multiples of 64)
  int32_t blk_begin, blk_end;          // RowBlock range
  int32_t item_begin, item_end;        // AttnItem range, all layers but the last
  int32_t citem_begin, citem_end;      // AttnItem range of candidate tiles only (last layer, score stage)
  int32_t cblk_begin, cblk_end;        // range in cand_blocks (last-layer row pruning, score head, score stage)
  int32_t hitem_begin, hitem_end;      // AttnItem range of history tiles only (prefill stage)
  int32_t hblk_begin, hblk_end;        // range in hist_blocks (prefill stage)
};

struct Plan {
  std::vector<int32_t> tok_off;        // logical merged offsets, [B+1]
  std::vector<Segment> segs;           // in workspace order
  std::vector<RowBlock> blocks;        // total_rows / 64 entries
  std::vector<AttnItem> items;         // per group: request by request, the last kTailItems longest first
  std::vector<AttnItem> cand_items;    // candidate tiles only
  std::vector<int32_t> cand_blocks;    // indices of candidate RowBlocks with valid rows, per group contiguous
  std::vector<AttnItem> hist_items;    // history tiles only
  std::vector<int32_t> hist_blocks;    // indices of history RowBlocks, per group contiguous
  std::vector<Group> groups;
  int32_t q_tile = 0;                  // query rows per attention item
  int32_t longest = 0;                 // longest history
  int32_t total_rows = 0;
  int64_t total_cands = 0;
  bool split = false;                  // some request was split into several segments
};

// Validation + planning.  Returns a flame_gr_status;
// on failure `err` holds the reason.
int validate_config(const flame_gr_config &cfg, std::string &err);
// cand_capacity (optional, [B]): rows are reserved for that many candidates per request (>= the actual
// count), and layout and stream groups depend on the capacities only, not on the actual counts: the plans
// of a prefill (no candidates yet) and of the score calls that follow it then agree on every row.
int build_plan(const flame_gr_config &cfg, const int32_t *hoff, const int32_t *coff, int32_t B,
               int32_t n_groups, int64_t ws_rows, Plan &plan, std::string &err,
               const int32_t *cand_capacity = nullptr);

// bucket(delta) for delta in [0, D)
void bucket_table(int32_t n_buckets, int32_t D, int32_t *out);
int32_t bucket_of(int32_t delta, int32_t n_buckets, int32_t D);

// The mask predicate, on (row, col) token indices of a request with L history items.
inline bool allowed(int32_t r, int32_t c, int32_t L) {
  return r < L ? (c <= r) : (c < L || c == r);
}

// Workspace rows needed for a capacity (used at create).
int64_t workspace_rows(const flame_gr_config &cfg);

}  // namespace flame
