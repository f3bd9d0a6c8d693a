// Host-side planning for the entry points: argument validation, workspace layout and the
// per-call work lists.  Plain C++ (no HIP); the entry points in tide_api.hip stage the blob
// it builds.
#pragma once

#include <stddef.h>
#include <stdint.h>

#include <vector>

#include "tide.h"
#include "tide_common.h"

namespace tide {

// Where each region lives inside the caller's workspace (byte offsets).
struct Plan {
  int op = 0;
  int32_t num_tasks = 0;
  // upload region [0, upload_bytes): header, task table, items
  size_t tasks_off = 0;
  size_t items_off = 0;
  size_t upload_bytes = 0;
  // extend split-KV plan: per-row merge descriptors (uploaded after the items)
  bool split = false;
  size_t merge_rows_off = 0;
  // decode, at the blob's end, zeros in it.  Chunks: arrival counters per (task, kv head), used
  // when the split kernel merges (fold_merge: few splits per task) instead of a merge kernel.
  // Runs (`stream`): a flag per partial slot, set to the call's own number, so the zeros do not
  // matter where the plan is read in place and never copied.
  size_t tickets_off = 0;
  bool fold_merge = false;
  // decode with the library's own split (make_plan_decode): StreamItems, one per run
  bool stream = false;
  int32_t num_runs = 0;
  int32_t steps = 0;       // key steps per run
  int32_t last_steps = 0;  // of the last run
  int64_t row_slots = 0;  // partial row slots (each holds every query head)
  // the planner's run-time estimates (microseconds) of the plain and chosen extend plans;
  // 0 when the call was too large to consider splitting
  double est_plain_us = 0.0;
  double est_us = 0.0;
  // decode and split-extend partials (not uploaded)
  size_t part_o_off = 0;
  size_t part_ml_off = 0;
  size_t total_bytes = 0;
  int32_t num_items = 0;
  // extend: tokens per work item and waves per workgroup
  int32_t tokens_per_item = 0;
  int32_t waves = 0;
  // extend: passes over the blocks that the search for the chunk length made
  int32_t search_passes = 0;
  int32_t chunk = 0;  // decode: keys per chunk or run; split extend: most key tiles per chunk
  // decode
  int32_t max_splits = 0;
  int32_t total_rows = 0;
  std::vector<uint8_t> blob;  // bytes to upload (header + tasks + items)
};

// Shape validation shared by every entry point.
int check_dims(const tide_dims* dims);

// Validates lengths and builds the plan.  When `build_blob` is false only the sizes are
// computed (tide_workspace_size).  `bt_stride` < 0 skips the block-table capacity check.
int make_plan(int op, int32_t num_tasks, const int32_t* lens_a, const int32_t* lens_b,
              const tide_dims& dims, int32_t num_splits, int32_t bt_stride, bool build_blob,
              Plan* plan);

// Decode: runs of equal length when the library chooses the split (num_splits == 0) and the call's
// steps can be counted in 32 bits, else the chunk plan of make_plan.
int make_plan_decode(int32_t num_tasks, const int32_t* kv_lens, const tide_dims& dims,
                     int32_t num_splits, int32_t bt_stride, bool build_blob, Plan* plan);

// The runs of a decode plan as one int32 each, the task a run starts in, in place of the
// StreamItems; the task table then holds each task's first step (aux), from which the rest
// follows.  Returns the bytes of the blob up to their end.
size_t compact_runs(Plan* plan);

// Shared-prefix decode: groups are consecutive task ranges [group_start[g],
// group_start[g+1]); the first shared_lens[g] keys (a multiple of the page size, below
// every member's kv_len) live in pages every member's block table shares.
constexpr int kOpDecodeShared = 100;  // internal op code of the plan
int make_plan_shared(int32_t num_tasks, const int32_t* kv_lens, int32_t num_groups,
                     const int32_t* group_start, const int32_t* shared_lens,
                     const tide_dims& dims, int32_t num_splits, int32_t bt_stride,
                     bool build_blob, Plan* plan);

// Waves per workgroup of the extend kernel for a head size and GQA group.
int32_t extend_waves(int32_t head_dim, int32_t group);

inline size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

}  // namespace tide
