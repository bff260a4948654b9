// Internal declarations shared by the translation units of libsp.so (not part of the ABI).
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include <string>
#include <vector>

#include "sp.h"

namespace sp {

constexpr int kMaxRanges = 1024;   // ancestor key ranges per row group (after merging neighbours); a sanity bound, no array depends on it
constexpr int kPrefillThreads = 256;
constexpr int kMaxDevices = 64;
// per-path accumulator of the saliency launch: fixed-point sum of log-likelihoods, scored rows, flags
struct SalSlot {
  unsigned long long sum;   // two's complement, 2^-36 units
  uint32_t count;
  uint32_t flags;           // 1: a row with lp = -inf, 2: +inf, 4: NaN
};
// what the saliency row kernel leaves of a piece of a row: maximum, sum of exp(x - maximum), the target's logit (first
// piece) and whether the row has a target
struct RowPart {
  float m, s, x_target;
  uint32_t scored;
};
// Rows are cut into pieces only while rows * pieces stays at or below this, which the scratch of any call can hold.
constexpr int64_t kSalSplitRows = 2048;
constexpr int64_t kSalDefaultRows = int64_t(1) << 16;               // what a new context's workspace is sized for
constexpr int kSalDefaultSlots = 16384;
constexpr int64_t kSalStaticRows = int64_t(1) << 16;                // limits of the no-allocation entry point
constexpr int kSalStaticSlots = 16384;
inline size_t saliency_scratch_bytes(int64_t rows, int32_t slots) {
  return 256 + sizeof(SalSlot) * size_t(slots) + sizeof(RowPart) * size_t(rows);
}
static_assert(kSalSplitRows <= kSalDefaultRows && kSalSplitRows <= kSalStaticRows, "pieces of a call fit its scratch");
constexpr size_t kSalStaticBytes = 256 + size_t(kSalStaticRows) * sizeof(RowPart) + sizeof(SalSlot) * size_t(kSalStaticSlots);

// A decode launch whose key lists are cut into pieces needs scratch, a region: partial sums of at most kDecPartRows (query
// row, piece) pairs plus {max, sum} each, and at most kDecPartCounters arrival counters (zero between launches).
constexpr int64_t kDecPartRows = 4096;
constexpr int kDecPartCounters = 1024;
// Regions that a plan has from the start (or as many as the plan destroyed last had in use, up to kDecPlanRegions), and the
// most that a plan may come to have.
constexpr int kDecFirstRegions = 4, kDecPlanRegions = 32, kDecMaxRegions = 256;
// A decode launch is small with up to this many workgroups per compute unit (build_key_table); what the descriptors of paths at
// a fixed stride may take in any case.
constexpr int kDecFewWgsPerCu = 4;
constexpr int64_t kDecPaddedDescs = 4096;
constexpr size_t kDecChunkBytes = size_t(16) << 20;
struct DecodeRegion {
  void *part;
  uint32_t *count;
  // owner: a stream (hipStreamPerThread: of one thread), or a stream within one capture
  hipStream_t stream;
  unsigned long long capture, thread;     // capture id + 1; number of the thread; else 0
  bool taken;
};

// A run of segments fused on the query side: child segments that are packed directly behind
// their parent continue the parent's causal sequence (Sec. 3.2: a chain is a classical prompt).
// Rows [tok_start, tok_start+len) see: the ancestor ranges (all keys), then own rows causally.
struct RowGroup {
  int32_t tok_start;
  int32_t len;
  int32_t range_off;   // first ancestor range (root-to-leaf order)
  int32_t n_ranges;
  int32_t anc_keys;    // total keys in the ancestor ranges
  int32_t prompt;
};

struct KeyRange {
  int32_t tok_start;
  int32_t len;
};

struct RangeDesc {
  int32_t beg, end;    // decode ranges [beg, end) of dec_ranges
  int32_t tok_start;   // copy of dec_ranges[beg] (0, 0 when beg == end)
  int32_t len;
};

// A query head and its KV head, 16 bits each: both unsigned (KV heads from 32768 on set the sign bit).
inline int32_t pack_heads(int32_t head, int32_t kv_head) { return int32_t(uint32_t(head) | uint32_t(kv_head) << 16); }

// One prefill work item: a tile of query rows of one row group, for one group of query heads.
// Self-contained (one 32-byte scalar load), so a workgroup never chases pointers between items.
struct WorkItem {
  int32_t tok_start;   // first packed token of the row group
  int32_t row0;        // first row of the tile inside the group
  int32_t n_rows;      // token rows in the tile (1 .. tile_rows)
  int32_t anc_keys;    // keys in the ancestor ranges
  int32_t range_off;   // first ancestor range
  int32_t n_ranges;
  int32_t head0;       // pack_heads(first query head handled by the workgroup, its KV head)
  int32_t r0_start;    // first token of ancestor range 0 (the only one when n_ranges == 1)
};

// Work of the wide prefill kernel: tiles of kWideWaves blocks of up to 32 rows (over the query heads of a workgroup), and items
// that name a tile and its heads.  The rows of a tile may belong to several row groups when these have the same ancestors; its
// keys are one virtual sequence [ancestors ; own run of each group], cut into ranges.  With several groups every own run
// begins at a multiple of 32 keys (a block of 32 never holds keys of two of them).  The kernel moves them in pieces of 16 bytes.
constexpr int kWideWaves = 8, kWideStageKeys = 64, kWideRanges = 16;
struct alignas(16) WideRange {
  int32_t delta;       // virtual keys from the end of the range before up to `end` are the tokens min(delta + key, last)
  int32_t end;         // the last range's has no end
  int32_t last;
  int32_t unused;
};
struct alignas(16) WideBlock {
  int32_t tok;         // first row's token
  int32_t n_rows;      // 0: none
  int32_t first;       // first row's virtual key
  int32_t base;        // first virtual key of its own run
};
struct alignas(16) WideTile {
  int32_t n_keys;
  int32_t anc;         // ancestor keys
  int32_t anc_end;     // several groups: `anc` rounded up to 32; one group, whose own run follows directly: 0
  int32_t steps;       // stages that each block is computed on, summed up (what a tile takes, for the host)
  WideBlock block[kWideWaves];
  WideRange range[kWideRanges];
};
static_assert(sizeof(WideRange) == 16 && sizeof(WideBlock) == 16 && offsetof(WideTile, block) == 16 &&
              offsetof(WideTile, range) == 16 + 16 * kWideWaves && sizeof(WideTile) == 16 * (1 + kWideWaves + kWideRanges));
struct WideItem {
  int32_t tile;
  int32_t heads;       // pack_heads(first query head, its KV head)
};

// Device-side view of a plan (plain pointers, passed by value to kernels).
struct PlanDev {
  const KeyRange *ranges;
  const WorkItem *items;
  const int32_t *wg_begin;       // [n_wg + 1] slice of the (permuted) work list per workgroup slot
  const WideTile *wide_tiles;
  const WideItem *wide_items;
  const float *tok_pos;          // [n_tokens] or nullptr
  const float *slopes;           // [n_q_heads] or nullptr
  // decode tables
  const int32_t *path_off;       // [n_prompts+1]
  // first/last+1 decode range and a copy of the first range: one 16-byte read tells a source's
  // ranges when there is only one (the usual case), without a further dependent read
  const RangeDesc *shared_desc;  // [n_prompts] the shared segments of each prompt
  const RangeDesc *path_desc;    // each path slot: [n_prompts][path_stride], or [n_slots] where path_stride is 0
  int32_t path_stride;           // most paths of any prompt, or 0 (more than 64, or too much padding, or no small launch)
  const KeyRange *dec_ranges;
  int32_t n_items;
  int32_t n_wg;
  int32_t n_tokens;
  int32_t n_prompts;
  int32_t n_q_heads, n_kv_heads, head_dim;
};

}  // namespace sp

struct sp_ctx {
  int device = 0;
  hipStream_t stream = nullptr;
  std::string err;
  int n_cu = 256;             // compute units of the device (read once)
  // saliency accumulators (zero between launches); a block that became too small is kept until
  // sp_destroy, because a captured graph may still name it
  void *sal = nullptr;        // [launch counter][sal_slots accumulators][sal_rows per-row values]
  int32_t sal_slots = 0;
  int64_t sal_rows = 0;
  std::vector<void *> retired;
  // plan upload: one pinned staging buffer, one event that tells when its last copy has left it,
  // and the device blocks of destroyed plans, kept for the next plan
  void *stage = nullptr;
  size_t stage_bytes = 0;
  hipEvent_t stage_ev = nullptr;
  bool stage_busy = false;
  std::vector<std::pair<void *, size_t>> blob_pool;
  int dec_regions = sp::kDecFirstRegions;   // decode regions that the next plan starts with
  // Memory for the partial sums of plans' first regions: chunks, cut up as plans ask (a hipMalloc of a few MB per plan would
  // double the time to make one), and the pieces of plans that are gone.  Freed with the last plan, since a captured decode
  // may be replayed until then.
  std::vector<void *> dec_chunks;
  char *dec_at = nullptr;
  size_t dec_left = 0;
  std::vector<std::pair<void *, size_t>> dec_free;
  int refs = 1;               // the context itself + every live plan made on it
  bool closed = false;        // sp_destroy was called; the struct lives on until the last plan is gone
};

struct sp_plan {
  sp_ctx *ctx = nullptr;      // nullptr: host-only plan
  int32_t n_prompts = 0, n_segments = 0, n_tokens = 0, n_slots = 0;
  int32_t n_q_heads = 0, n_kv_heads = 0, head_dim = 0;
  sp_dtype dtype = SP_F32;
  int32_t heads_per_wg = 1;   // query heads stacked in one prefill workgroup
  int32_t waves_per_wg = 4;   // waves (32-row blocks) per prefill workgroup
  int32_t tile_rows = 0;      // token rows per prefill tile
  int32_t n_tiles = 0;
  int32_t n_wg = 0;           // slots of the prefill work list (a multiple of 8): persistent workgroups, or items of a round
  int32_t max_slice = 0;      // most work items of any slot
  int32_t max_ranges = 0;
  int32_t max_dec_ranges = 0; // largest joined-cache range count bound per prompt (shared + per-path max)
  int64_t visible_pairs = 0;
  int64_t max_shared_keys = 0, max_path_keys = 0;   // most tokens of a prompt's shared part / of any path
  bool has_pos = false, has_slopes = false;
  // host copies
  std::vector<int32_t> prompt_seg_off, seg_tok_start, seg_tok_len, seg_parent, seg_path;
  std::vector<sp::RowGroup> groups;
  std::vector<sp::KeyRange> ranges;
  std::vector<sp::WorkItem> items;
  bool wide = false;                   // prefill by the wide kernel: its work list takes the place of `items`
  std::vector<sp::WideTile> wide_tiles;
  std::vector<sp::WideItem> wide_items;
  std::vector<int32_t> wg_begin;
  std::vector<int32_t> tok_group;      // token -> row group (host inspection)
  std::vector<int32_t> path_off, shared_rng_beg, shared_rng_end, path_rng_beg, path_rng_end;
  std::vector<sp::KeyRange> dec_ranges;
  std::vector<int32_t> path_max_ranges;  // per prompt: max ranges of any single path
  std::vector<float> pos, slopes;        // copies of tok_pos / alibi_slopes (empty when not given)
  // Decode scratch (sp::DecodeRegion).  A region belongs to one order of execution -- a stream, or a stream within one
  // capture -- until the plan is updated or destroyed, so that launches that may overlap never share one.  The first
  // regions' counters lie behind the tables in the plan's device block and their partial sums in the context's chunks,
  // further regions come in blocks of their own; all go the way of the tables: whoever gets the memory next has work ordered
  // behind the plan's, as sp_plan_update and sp_plan_destroy require.
  size_t dec_part_bytes = 0, dec_count_bytes = 0;     // of one region; 0: no decode of this plan is cut into pieces
  size_t dec_first = 0;                               // first regions; the others are in dec_blocks
  void *dec_scratch = nullptr;                        // the first regions' partial sums
  size_t dec_scratch_bytes = 0;
  mutable std::vector<sp::DecodeRegion> dec_regions;
  mutable std::vector<std::pair<void *, size_t>> dec_blocks;
  // device copies (one allocation)
  void *dev_blob = nullptr;
  size_t dev_blob_bytes = 0;  // capacity of the allocation
  sp::PlanDev dev{};
};

namespace sp {

// Kernel launchers (defined next to their kernels).  All return hipError_t from the launch.
struct PrefillArgs {
  const void *Q, *K, *V;
  void *O;
  int64_t q_tok_stride, q_head_stride, kv_tok_stride, kv_head_stride;
  float scale;
};
hipError_t launch_prefill_bf16(const sp_plan *plan, const PrefillArgs &a, hipStream_t s);
hipError_t launch_prefill_wide(const sp_plan *plan, const PrefillArgs &a, hipStream_t s);
hipError_t launch_prefill_f32(const sp_plan *plan, const PrefillArgs &a, hipStream_t s);

hipError_t launch_saliency(const void *logits, sp_dtype dt, int64_t n_rows, int64_t vocab, int64_t row_stride,
                           const int32_t *target, const int32_t *row_path, const float *prior,
                           int32_t n_slots, int mode, void *scratch, int32_t cap_slots, float *score, hipStream_t s);
hipError_t saliency_static_scratch(int device, void **out);

hipError_t launch_topk(const float *score, const int32_t *path_off, int32_t n_prompts, int32_t n_paths_max,
                       int32_t k, int32_t *kept, hipStream_t s);

struct DecodeArgs {
  const int32_t *kept;
  int32_t k;
  const void *Kp, *Vp;
  int64_t kv_tok_stride, kv_head_stride;
  void *Kr, *Vr;
  float *pos_resp;
  int32_t resp_capacity;
  const int32_t *resp_len;
  int32_t resp_len_add;
  const float *new_pos;
  const void *q_new, *k_new, *v_new;
  void *o_out;
  float scale;
};
// bytes of partial sums and of counters that the largest decode of the plan needs (0: none is ever cut into pieces)
void decode_scratch(const sp_plan *plan, int n_cu, size_t *part_bytes, size_t *count_bytes);
// Scratch region for a decode launch on stream s, or nullptr when there is none to be had (the launch then does without).
const DecodeRegion *decode_region(const sp_plan *plan, hipStream_t s);
hipError_t launch_decode(const sp_plan *plan, const DecodeArgs &a, hipStream_t s);

}  // namespace sp
