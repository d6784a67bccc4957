// Internal definitions shared by libaep's host code and its gfx950 kernels.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace aep {

// One mu-queue entry (16 bytes): the row it refers to (the token's tensor
// stays where it arrived, as the paper's token metadata refers to GPU-resident
// input tensors), the layer-local token id and top-k slot, and the gate weight.
struct QEntry {
  const void* row;
  int32_t token_slot;  // token | slot << 24
  float w;
};
static_assert(sizeof(QEntry) == 16, "QEntry must be 16 bytes");

constexpr int kTokenBits = 24;
constexpr int32_t kTokenMask = (1 << kTokenBits) - 1;

// Weights of one expert (device pointers) -- the per-layer table the FFN
// kernels read.
struct WeightDesc {
  const void* gate;
  const void* up;
  const void* down;
  const uint16_t* s_gu;    // fp8 only: [2f] bf16 scales
  const uint16_t* s_down;  // fp8 only: [d]  bf16 scales
  const void* pad;
};
static_assert(sizeof(WeightDesc) == 48, "WeightDesc layout");

// One FFN group of a drained batch, written by the plan kernel.  A group's
// rows are covered by row tiles of up to three families (bf16 / fp8 weights):
// family 0 (256 rows) over its full 256-row blocks and a remainder above 128
// rows, else one tile of family 1 (128 rows) or 2 (64 rows) over the
// remainder, from row row1 on.  f32 weights use family 0 alone, with 64-row
// tiles.  t0[s * 3 + f] is the group's first tile id in family f of FFN stage
// s (0: gate/up, 1: down).
struct GroupDesc {
  int32_t n;        // rows
  int32_t x_row0;   // first row in x_perm
  int32_t y_row0;   // first row in h and y
  int32_t t0[6];    // first tile id per (stage, family)
  int32_t nrt[3];   // row tiles per family
  int32_t row1;     // first row of the family 1 or 2 tile
  int32_t pad[3];
};
static_assert(sizeof(GroupDesc) == 64, "GroupDesc layout");

// Device error flag bits.
constexpr int32_t kErrNonFinite = 1;
constexpr int32_t kErrTokenRange = 2;
constexpr int32_t kErrSlotRange = 4;
constexpr int32_t kErrCollision = 8;

constexpr int kRouteThreads = 256;
constexpr int kRouteLanes = 8;                              // lanes per token in the router
constexpr int kRouteTokens = kRouteThreads / kRouteLanes;   // tokens per router workgroup
constexpr int kMaxRouteExperts = 64;
constexpr int kDirectPrefixBlocks = 64;  // router workgroups whose appends sum earlier counts directly
// Fragments of up to this many tokens are routed and appended by one workgroup
// in one launch: up to 1024 threads.  Against two launches, us per fragment: 8
// experts top-2, 33 / 128 tokens 3.0 / 3.3 and 4.6 / 5.1; 32 top-4 4.2 / 4.7 and
// 5.4 / 5.9; 64 top-6 6.1 / 6.9 and 6.9 / 7.2; 64 top-8 7.3 / 8.1 and 7.4 / 7.9.
constexpr int kFusedTokens = 128;
constexpr int kMaxTopK = 8;
constexpr int kMaxGroups = 1024;

// FFN tiling (bf16 / fp8 weights): tiles of kBM >> family rows x kBN columns;
// gate/up tiles cover kBN / 2 features of gate and the same of up.
constexpr int kBM = 256;
constexpr int kBN = 256;
constexpr int kBK = 64;
constexpr int kFfnLds = 160 * 1024;  // LDS of one FFN workgroup (the CU's)
// Split-K of the last, partial round of an FFN launch's tiles: up to
// kMaxSplit pieces of at least kMinSplitSteps K steps each per tile or column
// half, at most kSplitCounters of these.
constexpr int kMaxSplit = 8;
constexpr int kMinSplitSteps = 8;
constexpr int kSplitCounters = 1024;
// Words of the tile totals' array: 6 totals, then the cut of each stage's last
// round (see ffn_sched.h).
constexpr int kCutWord = 6;
constexpr int kTileWords = 8;
// Workgroups of a bf16 / fp8 FFN launch: one per CU, a multiple of 8 (the map
// from XCDs to items needs that).
inline int ffn_grid(int num_cu) { return num_cu < 8 ? 8 : (num_cu + 7) & ~7; }
// The partial sums' area of a context: 128 parts of a 256-row tile (a tile of
// n pieces needs n - 1 parts; the cut is chosen to fit).
constexpr int64_t kSplitBytes = 128 * (int64_t)kBM * kBN * 4;
// f32 path
constexpr int kBM32 = 64;
constexpr int kBN32 = 64;

// Layer-granularity pick (host): the block to drain next from per-block
// totals R[nb] under an aep_policy (defrag: R[b] + sum_{i=1..lookahead}
// R[(b + i) mod nb] * delta^i).  Ties go to the lowest block; false when every
// block is empty.  Defined with the host scheduler (sched.hip).
bool pick_block(const int64_t* R, int nb, int policy, double delta, int lookahead, int* pb);

// ---------------------------------------------------------------- launchers
// Each returns hipGetLastError() after the launch.
// Routes T tokens; blockcnt [ceil(T / kRouteTokens)][E] receives each router
// workgroup's row count per expert.  Above kDirectPrefixBlocks workgroups the
// launch then rewrites them into each workgroup's first queue slot and writes
// depth_nxt (depth_cur + this fragment's counts); below, append does both.
// done: a launch counter that must be 0 before the launch (the kernel leaves
// it 0).
hipError_t launch_route(const float* logits, int T, int E, int k, int renorm, int32_t* r_idx,
                        float* r_w, int32_t* r_rank, int32_t* blockcnt, int32_t* idx_out,
                        float* w_out, const int32_t* depth_cur, int32_t* depth_nxt, int32_t* done,
                        int32_t* err, hipStream_t s);
// Both for a fragment of at most kFusedTokens tokens, in one launch (arguments
// as below and above).
hipError_t launch_route_append(const float* logits, int T, int E, int k, int renorm, int32_t* idx_out, float* w_out,
                               const char* x, int64_t row_bytes, int32_t token_base, const int32_t* depth_cur,
                               int32_t* depth_nxt, QEntry* q, int64_t q_stride, const void** tok_row,
                               const int32_t* token_ids, int n_ids, int32_t* live, int32_t* pend, int32_t* err,
                               hipStream_t s);
// token_ids == nullptr: token t of the fragment is token_base + t.  Else its
// id is token_ids[t] (< n_ids) and it claims pool entry live[id] / pend[id].
hipError_t launch_append(const int32_t* r_idx, const float* r_w, const int32_t* r_rank,
                         const int32_t* first_slot, int T, int E, int k, const char* x,
                         int64_t row_bytes, int32_t token_base, const int32_t* depth_cur,
                         int32_t* depth_nxt, QEntry* q, int64_t q_stride, const void** tok_row,
                         const int32_t* token_ids, int n_ids, int32_t* live, int32_t* pend,
                         int32_t* err, hipStream_t s);
// Rows of several experts in one launch: rows [pre[e], pre[e+1]) to queue e
// (pre: device, E + 1 entries, exclusive prefix of the per-expert counts).
hipError_t launch_enqueue_grouped(const char* rows, int64_t row_bytes, const int32_t* token_ids,
                                  const int32_t* slots, const float* gate_w, int n, int n_tokens, int k, int E,
                                  const int32_t* pre, const int32_t* depth_cur, int32_t* depth_nxt, QEntry* q,
                                  int64_t q_stride, int32_t* err, hipStream_t s);
hipError_t launch_enqueue_rows(const char* rows, int64_t row_bytes, const int32_t* token_ids,
                               const int32_t* slots, const float* gate_w, int n, int n_tokens,
                               int k, int expert, int E, const int32_t* depth_cur,
                               int32_t* depth_nxt, QEntry* q, int64_t q_stride, int32_t* err,
                               hipStream_t s);
// tile_totals[kTileWords]: tiles per (stage, family), index stage * 3 + family
// (stage 0 gate/up, 1 down), then the cuts, not chosen yet.  nt[2]: column
// tiles per row tile of each stage.
// bm: rows of a family 0 tile; families: 3, or 1 (f32: every row in family 0).
// only_expert >= 0: drain that expert's queue alone (every other group gets
// 0 rows and keeps its queue).  depth is the current half of the layer's
// depth ping-pong, depth_other the other one; both are cleared for the
// drained experts.
// tile_group [2][tile_cap]: the group of each tile of the gate/up (row 0) and
// down (row 1) launch, tiles numbered family by family;
// tile_cap bounds either launch's tile count.
hipError_t launch_plan(int E, int S, int n_tokens, int k, int only_expert, int32_t* depth,
                       int32_t* depth_other, int32_t* counts, int32_t* offsets, GroupDesc* groups,
                       int32_t* tile_totals, const int* nt, int bm, int families, int32_t* tile_group, int64_t tile_cap, int32_t* pos, float* posw,
                       hipStream_t s);
// N bounds the routed rows (the exact count is offsets[E] on the device);
// pos == nullptr skips the (token, slot) -> row map.  A few extra workgroups
// choose how each FFN launch's last round is cut (cut.nwg == 0: none do).
struct CutArgs {
  int32_t* tile_totals;
  int nwg;              // workgroups of the FFN launches
  int kt[2];            // K steps per stage
  bool fp8;             // fp8 weights
  int64_t split_bytes;  // room for partial sums
};
hipError_t launch_gather(const QEntry* q, int64_t q_stride, const int32_t* offsets, int E,
                         int64_t N, int n_tokens, int shared, const void* const* tok_row,
                         char* xp, int64_t row_bytes, int32_t* row_token, float* row_w,
                         int32_t* pos, float* posw, int k, int32_t* err, const CutArgs& cut, hipStream_t s);
// token pool: rows [0, offsets[E]) of a batch (N bounds them) are merged into
// pool[row_token[r]]; release writes out / ready for completed ids.
hipError_t launch_pool_accumulate(int act_dtype, const void* y, int64_t N, const int32_t* offsets,
                                  int E, const int32_t* row_token, const float* row_w, float* pool,
                                  int32_t* pend, int d, hipStream_t s);
hipError_t launch_pool_release(int act_dtype, float* pool, int32_t* live, int32_t* pend, int n_ids,
                               void* out, int32_t* ready, int d, hipStream_t s);
// stage 0: gate/up (xp -> h), stage 1: down (h -> y); max_tiles bounds the
// stage's tile count (the exact count is on the device); tile_group is that
// stage's row of the plan's tile -> group map.  split_slots holds the split-K
// partial sums and split_cnt [kSplitCounters] the arrivals per split tile,
// zero before the launch and left zero (bf16 / fp8 weights).
// clk != nullptr: workgroup w < clk_n writes its elapsed (s_memtime,
// s_memrealtime) ticks to clk[2w], clk[2w + 1] (bf16 / fp8 weights only).
hipError_t launch_ffn(int stage, int act_dtype, int w_dtype, const GroupDesc* groups,
                      const WeightDesc* wtab, const int32_t* tile_totals, const int32_t* tile_group,
                      float* split_slots, int32_t* split_cnt, int max_tiles,
                      const void* xp, void* h, void* y, int d, int f, int num_cu,
                      unsigned long long* clk, int clk_n, hipStream_t s);
hipError_t launch_combine(int act_dtype, const void* y, int64_t N, int n_tokens, int S, int k,
                          const int32_t* pos, const float* posw, void* out, int d, hipStream_t s);
hipError_t launch_fp8_to_bf16(const uint8_t* codes, uint16_t* out, int64_t n, hipStream_t s);

}  // namespace aep
