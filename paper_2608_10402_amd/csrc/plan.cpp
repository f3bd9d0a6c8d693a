// Host-side planning: validation, workspace layout and work lists (see plan.h).
#include "plan.h"

#include <math.h>
#include <stdlib.h>
#include <string.h>

#include <algorithm>
#include <numeric>

namespace tide {

int check_dims(const tide_dims* dims) {
  if (!dims) return TIDE_ERR_INVALID_ARG;
  if (dims->num_q_heads <= 0 || dims->num_kv_heads <= 0 || dims->head_dim <= 0 ||
      dims->page_size <= 0)
    return TIDE_ERR_INVALID_ARG;
  if (!(dims->sm_scale > 0.0f) || !isfinite(dims->sm_scale)) return TIDE_ERR_INVALID_ARG;
  if (dims->head_dim != 64 && dims->head_dim != 128) return TIDE_ERR_UNSUPPORTED;
  if (dims->page_size != kPage) return TIDE_ERR_UNSUPPORTED;
  if (dims->num_q_heads % dims->num_kv_heads != 0) return TIDE_ERR_UNSUPPORTED;
  if (dims->num_q_heads / dims->num_kv_heads > kMaxGroup) return TIDE_ERR_UNSUPPORTED;
  if (dims->num_kv_heads > kMaxKvHeads) return TIDE_ERR_UNSUPPORTED;
  return TIDE_OK;
}

int32_t extend_waves(int32_t head_dim, int32_t group) {
  (void)head_dim;
  (void)group;
  return 8;
}

namespace {

int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

// Automatic decode chunk.  The device holds 2048 decode waves at once (8 per CU).  When
// most (task, kv head) units are cut into several chunks, the items are nearly all full
// chunks and a launch of n items runs in about ceil(n / 2048) rounds, each about as long
// as a chunk plus a fixed cost (first loads, partial stores, a wave's start and end); a
// launch just above a multiple of 2048 items then leaves a mostly empty last round.  So
// for every round count R the planner takes the shortest chunk whose items fit in R
// rounds and keeps the R with the least R * (kDecodeRoundCost + chunk).  When that gives
// fewer than 4 chunks per unit, most items are units' shorter last chunks of scattered
// lengths; many items then balance the launch better, and the chunk is
// sum(kv) * Hkv / 4096 keys.  Chunks are multiples of the kernel step within [512, 16384].
// The rule now serves the calls whose runs would be too long (make_plan_decode).  Measured on
// MI355X against about 4096 items, call us: 32 tasks of 32k-96k keys (64 / 8 heads) 1368 ->
// 1242; 256 tasks of 1k-32k (32 / 8; 2 chunks per unit) 5% slower, so the item count rule
// stays there.
constexpr int64_t kDecodeWaveSlots = 2048;
constexpr int64_t kDecodeRoundCost = 1200;  // keys
constexpr int64_t kDecodeMinUnitChunks = 4;
constexpr int64_t kDecodeMaxRoundsTried = 8;
constexpr int64_t kDecodeMinChunk = 512;
constexpr int64_t kDecodeMaxChunk = 16384;
constexpr int64_t kDecodeTargetItems = 4096;
constexpr int64_t kStreamMaxSteps = 208;  // longest run of the equal-runs plan
constexpr int64_t kStreamMergeSteps = 40;  // see make_plan_decode, with the next three
constexpr double kStreamStepUs = 0.6;      // a step of a run, in workgroups of 4 waves
constexpr double kStreamBusyStepUs = 1.0;  // and of 8
constexpr double kStreamPartUs = 0.3;      // a part in the merge of G > 8 heads of d = 128
// Shared-prefix decode in one round of waves: chunks of at most this length.
constexpr int64_t kSharedRoundChunk = 1280;
constexpr int64_t kFoldMeanSplits = 4;  // merge inside the split kernel up to this mean

// The automatic decode chunk (see kDecodeRoundCost).  Round rule: for R rounds from the
// fewest that can hold the items, the shortest chunk (a multiple of the kernel step) whose
// items fit in R * 2048 waves, scored R * (kDecodeRoundCost + chunk); items fall as the
// chunk grows, so each R is a binary search.  R stops growing once the shortest allowed
// chunk fits, once R rounds of it already score worse than the best found, or after
// kDecodeMaxRoundsTried values (a few dozen passes over the tasks per call).  Item rule,
// when the round rule would leave fewer than 4 chunks per unit (or cannot reach 4 at
// all): sum(kv) * Hkv / 4096 keys.
int64_t decode_auto_chunk(const std::vector<TaskDesc>& tasks, int32_t hkv) {
  const int64_t units = (int64_t)tasks.size() * hkv;
  // Items for a chunk of m kernel steps: Hkv * sum over tasks of ceil(kv / (32 m)), from
  // each task's length in steps (32-bit divisions: this runs a few dozen times per call).
  std::vector<uint32_t> steps(tasks.size());
  for (size_t b = 0; b < tasks.size(); ++b)
    steps[b] = (uint32_t)ceil_div((int64_t)tasks[b].prefix + 1, kDecodeStep);
  auto items_at = [&](int64_t m) {
    int64_t n = 0;
    for (uint32_t k : steps) n += (k + (uint32_t)m - 1) / (uint32_t)m;
    return n * hkv;
  };
  auto item_rule = [&]() {
    int64_t total = 0;
    for (const TaskDesc& t : tasks) total += (int64_t)t.prefix + 1;
    int64_t c = ceil_div(total * hkv, kDecodeTargetItems);
    c = ceil_div(c, kDecodeStep) * kDecodeStep;
    return std::min<int64_t>(std::max<int64_t>(c, kDecodeMinChunk), kDecodeMaxChunk);
  };
  if (items_at(kDecodeMinChunk / kDecodeStep) < kDecodeMinUnitChunks * units) return item_rule();
  const int64_t lo_step = kDecodeMinChunk / kDecodeStep, hi_step = kDecodeMaxChunk / kDecodeStep;
  const int64_t r0 = std::max<int64_t>(1, ceil_div(items_at(kDecodeMaxChunk / kDecodeStep),
                                                   kDecodeWaveSlots));
  int64_t best = kDecodeMaxChunk, best_score = INT64_MAX;
  int64_t hi_prev = hi_step;  // R rounds' chunk also fits R + 1 rounds: the next search's top
  for (int64_t r = r0; r < r0 + kDecodeMaxRoundsTried; ++r) {
    if (r * (kDecodeRoundCost + kDecodeMinChunk) >= best_score) break;  // cannot win
    const int64_t cap = r * kDecodeWaveSlots;
    int64_t lo = lo_step, hi = hi_prev;  // in kernel steps; items_at(hi) <= cap
    if (items_at(lo) <= cap) hi = lo;
    while (hi - lo > 1) {
      const int64_t mid = (lo + hi) / 2;
      if (items_at(mid) <= cap) hi = mid;
      else lo = mid;
    }
    hi_prev = hi;
    const int64_t c = hi * kDecodeStep;
    const int64_t score = r * (kDecodeRoundCost + c);
    if (score < best_score) {
      best_score = score;
      best = c;
    }
    if (hi == lo_step) break;  // more rounds can only add cost
  }
  if (items_at(best / kDecodeStep) < kDecodeMinUnitChunks * units) return item_rule();
  return best;
}

// Per-task (prefix, extend) of the positions this call touches or attends.
int task_lengths(int op, int32_t b, const int32_t* lens_a, const int32_t* lens_b, int32_t* prefix,
                 int32_t* extend) {
  switch (op) {
    case TIDE_OP_KV_APPEND:
    case TIDE_OP_EXTEND:
      *prefix = lens_a[b];
      *extend = lens_b[b];
      if (*prefix < 0 || *extend < 0) return TIDE_ERR_INVALID_ARG;
      break;
    case TIDE_OP_FULL_PREFILL:
      *prefix = 0;
      *extend = lens_a[b];
      if (*extend < 0) return TIDE_ERR_INVALID_ARG;
      break;
    case TIDE_OP_DECODE:
      if (lens_a[b] <= 0) return TIDE_ERR_INVALID_ARG;
      *prefix = lens_a[b] - 1;
      *extend = 1;
      break;
    default:
      return TIDE_ERR_INVALID_ARG;
  }
  if ((int64_t)*prefix + *extend > INT32_MAX) return TIDE_ERR_INVALID_ARG;
  return TIDE_OK;
}

}  // namespace

// ---- extend / prefill work lists ------------------------------------------------------
//
// A work item is one block of tb = 256 / G tokens of one (task, kv head): its 256 query
// rows are the block's (token, head) pairs, and one 8-wave workgroup, which fills a CU,
// walks the key tiles (64 keys) the block sees.  Two plans are considered:
//   plain  every item walks all its tiles and writes its rows;
//   split  a block that spans many tiles is cut into chunks of about T tiles that run on
//          different CUs and write unnormalised fp32 partials, which a second kernel
//          merges (the split-K scheme of flash decoding, applied to extend blocks).
// Splitting pays when a call has too few items to keep 256 CUs busy to the end, or a last
// round of items that is nearly empty.  The choice compares run-time estimates of the plain
// plan and of split plans whose chunks fill 1/4 .. 6 rounds of the CUs: the items of a kv
// head are dealt out longest first, a round of 256 / Hkv at a time, and a round lasts as long
// as its longest item; a tile costs less while CUs are idle (the card is power-limited, so
// its clock is higher then), a chunk costs the write of its partial, and a split plan the
// merge (of very many chunks, the time a row's merge takes to walk them: one task of 40,000 + 8
// tokens at 8 / 2 heads, d = 64, takes 41 us as 124 chunks a kv head and 29 as 32).  The planner
// runs on every call, so a number of rounds costs one pass over the blocks
// for its estimate and about 2 log2 of the longest block's tiles for its chunk length, and only
// the chosen plan is materialised.
namespace {

constexpr int kCus = 256;  // MI355X compute units, 32 per XCD
// Cost model, fitted to 27 calls of 1-40 tasks, 500-90,000 keys and 8-1,500 new tokens timed
// plain and with 1 .. 6 rounds of chunks (all head shapes); the plan it takes was within 5% of
// the fastest of them on 23 and within 15% on the others.  Against the plan before it (chunks
// on a fixed grid of T tiles, the last up to 1.5 T long, for the least estimated sum) on the
// same kernel, one task of 12,000 + 800 tokens went from 185 to 161 us (28 / 4 heads, d = 128);
// with the kernel's own 7% in it, one of 30,000 + 200 from 151 to 103, 3 of 12,000 + 800 from
// 551 to 440, 8 of 6,000 + 380 from 338 to 262, 2 of 8,000 + 1,500 (32 / 8) from 549 to 405.
constexpr double kCuFlopsPerUs = 4.7e6;    // MFMA rate of one CU, all CUs busy
constexpr double kIdleClockGain = 0.25;    // a tile is this much cheaper with half the CUs idle
constexpr double kItemUs = 1.0;            // first-tile latency and epilogue
constexpr double kChunkUs = 3.0;           // the same with the partial's statistics
constexpr double kChunkRowsUs = 6.6;       // write of 256 rows' partials, all CUs at once
constexpr double kMergeBytesPerUs = 6.5e6; // rate at which the merge reads the partials
constexpr double kMergePartUs = 0.26;      // the least it takes a row's merge per chunk
constexpr double kMergeLaunchUs = 4.0;     // second kernel launch
constexpr double kSplitGain = 0.96;        // split when estimated at least this much faster
constexpr int kMinChunkTiles = 4;
constexpr int kMaxChunks = 512;
// Rounds of chunks tried, in quarters.  Fewer than a round only where a block may have over
// kManyChunks chunks: there the walk of its merge is what they cost, and with fewer the estimates
// are too close to tell (5 tasks of 500 + 100 tokens took 31.8 us so and 30.6 unsplit).
constexpr int kManyChunks = 32;
constexpr int kQuarterRounds[] = {1, 2, 4, 8, 12, 16, 20, 24};
constexpr int64_t kSplitMaxItems = 2048;  // larger calls fill the chip with the plain plan

struct Block {
  int32_t task, tok0, ntok, ntiles;
};

// A block's tiles cut into chunks of at most T tiles, as few as that takes (at most
// kMaxChunks) and of equal length to one tile, so that equally long blocks of a task are cut
// at the same keys.  T == 0: the plain plan (one chunk).
inline int32_t num_chunks(int32_t ntiles, int32_t T) {
  if (T <= 0 || ntiles <= T) return 1;
  return std::min(kMaxChunks, (int32_t)(((uint32_t)ntiles + (uint32_t)T - 1) / (uint32_t)T));
}

inline int32_t chunk_begin(int32_t ntiles, int32_t n, int32_t c) {
  return n == 1 ? c * ntiles : c * (ntiles / n) + std::min(c, ntiles % n);
}

inline int32_t chunk_tiles(int32_t ntiles, int32_t n, int32_t c) {
  return n == 1 ? ntiles : ntiles / n + (c < ntiles % n ? 1 : 0);
}

// What dealing items out to XCDs takes a chunk to cost (in tiles).
inline double chunk_cost(int32_t ntiles, int32_t n, int32_t c) {
  return chunk_tiles(ntiles, n, c) + (n > 1 ? 3.0 : 0.5);
}

// Estimated run time (us) of the plan with chunk length T (0: plain).
double estimate(const std::vector<Block>& blocks, int32_t longest, const tide_dims& dims, int32_t T,
                double tile_us, int64_t* row_slots) {
  const int32_t group = dims.num_q_heads / dims.num_kv_heads;
  const int64_t round = std::max(1, kCus / dims.num_kv_heads);  // CUs of a kv head
  // the chunks of one kv head by length (in steps of 2^shift tiles, if very long)
  constexpr int kBins = 1024;
  int64_t count[kBins];
  int32_t most_rows[kBins];
  const int32_t most = T > 0 ? std::min(T, longest) : longest;
  int shift = 0;
  while (most >> shift >= kBins) ++shift;
  const int top = (kMaxChunks * (int64_t)T < longest ? longest : most) >> shift;
  const int bins = std::min(kBins, top + 1);
  std::fill_n(count, bins, 0);
  std::fill_n(most_rows, bins, 0);
  int64_t slots = 0, items = 0;
  int32_t parts = 1;  // the most chunks of a block
  for (const Block& b : blocks) {
    if (T <= 0 || b.ntiles <= T) {  // one chunk
      ++items;
      ++count[std::min(kBins - 1, b.ntiles >> shift)];
      continue;
    }
    const int32_t n = num_chunks(b.ntiles, T);
    slots += (int64_t)b.ntok * n;
    items += n;
    parts = std::max(parts, n);
    const int32_t q = b.ntiles / n, r = b.ntiles % n, rows = b.ntok * group;
    for (int up = 0; up < 2; ++up) {
      const int32_t m = up ? r : n - r, bin = std::min(kBins - 1, (q + up) >> shift);
      if (m == 0) continue;
      count[bin] += m;
      most_rows[bin] = std::max(most_rows[bin], rows);
    }
  }
  double us = 0.0;
  int64_t seen = 0, lead = 0;  // lead: place of the longest item of the next round
  for (int bin = bins - 1; bin >= 0; --bin) {
    seen += count[bin];
    for (; lead < seen; lead += round) {
      const double busy = (double)std::min(round, items - lead) / round;
      us += (double)((int64_t)bin << shift) * tile_us *
                (1.0 - kIdleClockGain * std::min(1.0, 2.0 * (1.0 - busy))) +
            (most_rows[bin] ? kChunkUs + kChunkRowsUs * most_rows[bin] / 256 : kItemUs);
    }
  }
  us *= std::max(1.0, (double)dims.num_kv_heads / kCus);
  if (slots > 0)
    us += std::max((double)slots * dims.num_q_heads * (dims.head_dim * 4.0 + 16.0) / kMergeBytesPerUs,
                   parts * kMergePartUs) +
          kMergeLaunchUs;
  *row_slots = slots;
  return us;
}

// Consecutive blocks [k0, k1) of one task (longest first), chunk c (-1: whole blocks)
// of kv head g.  Workgroups of a piece read the same K/V.
struct Piece {
  double cost;
  int32_t k0, k1, g, c;
};

// Item order.  Workgroups are dispatched round-robin over the XCDs (slot i runs on XCD
// i % 8), each with its own L2.  A column -- one (task, kv head, chunk) -- is kept on one
// XCD, its items consecutive, so workgroups that walk the same K/V run side by side and
// share it through L2 instead of re-reading HBM.  A column longer than a quarter of an
// XCD's share is cut into consecutive pieces first, so that a call with fewer units than
// XCDs still reaches every XCD; pieces then go longest first to the least loaded XCD.
// Returns, per XCD, its pieces in order.
std::vector<std::vector<Piece>> place(const std::vector<Block>& blocks,
                                      const std::vector<int32_t>& task_first,
                                      const std::vector<int32_t>& nchunks, int32_t num_kv_heads,
                                      int32_t T) {
  const int32_t ntasks = (int32_t)task_first.size() - 1;
  std::vector<Piece> cols;
  double total = 0.0, biggest = 0.0;
  for (int32_t b = 0; b < ntasks; ++b) {
    const int32_t k0 = task_first[b], k1 = task_first[b + 1];
    if (k0 == k1) continue;
    const int32_t nmax = nchunks[k0];  // chunk counts do not grow along a task's blocks
    for (int32_t c = 0; c < nmax; ++c) {
      int32_t end = k0;
      double cost = 0.0;
      while (end < k1 && nchunks[end] > c) {
        const double ci = chunk_cost(blocks[end].ntiles, nchunks[end], c);
        cost += ci;
        biggest = std::max(biggest, ci);
        ++end;
      }
      for (int32_t g = 0; g < num_kv_heads; ++g)
        cols.push_back(Piece{cost, k0, end, g, T > 0 ? c : -1});
      total += cost * num_kv_heads;
    }
  }
  const double cap = std::max(biggest, total / (kXcds * 4));
  std::vector<Piece> pieces;
  pieces.reserve(cols.size());
  for (const Piece& col : cols) {
    const int32_t c = std::max(col.c, 0);
    Piece cur{0.0, col.k0, col.k0, col.g, col.c};
    for (int32_t k = col.k0; k < col.k1; ++k) {
      const double ci = chunk_cost(blocks[k].ntiles, nchunks[k], c);
      if (cur.k1 > cur.k0 && cur.cost + ci > cap) {
        pieces.push_back(cur);
        cur = Piece{0.0, k, k, col.g, col.c};
      }
      cur.k1 = k + 1;
      cur.cost += ci;
    }
    if (cur.k1 > cur.k0) pieces.push_back(cur);
  }
  std::stable_sort(pieces.begin(), pieces.end(),
                   [](const Piece& x, const Piece& y) { return x.cost > y.cost; });
  std::vector<std::vector<Piece>> queues(kXcds);
  // In a call of a few rounds no XCD takes more items than its CUs' share of the rounds: one
  // more would be a round of its own (the same call as 264 items, 33 an XCD, took 65 us and
  // as 256 took 45).
  int64_t items = 0;
  for (const Piece& p : pieces) items += p.k1 - p.k0;
  const int64_t room = items <= kSplitMaxItems ? (items + kCus - 1) / kCus * (kCus / kXcds) : items;
  double load[kXcds] = {};
  int64_t count[kXcds] = {};
  for (Piece p : pieces) {
    while (p.k0 < p.k1) {
      int x = -1;
      for (int i = 0; i < kXcds; ++i)
        if (count[i] < room && (x < 0 || load[i] < load[x])) x = i;
      Piece part = p;
      part.k1 = (int32_t)std::min<int64_t>(p.k1, p.k0 + room - count[x]);
      part.cost = p.cost * (part.k1 - part.k0) / (p.k1 - p.k0);
      load[x] += part.cost;
      count[x] += part.k1 - part.k0;
      p.cost -= part.cost;
      p.k0 = part.k1;
      queues[x].push_back(part);
    }
  }
  return queues;
}

// Item slots in dispatch order: slot i * 8 + x is the i-th item of XCD x's queue, and an
// XCD whose queue ran out gets empty slots (ntok == 0) that return at once.  In a call of a
// few rounds an XCD's items go longest first, in steps of an eighth of the longest (items of
// about equal length keep their order, and so the K/V they share): a long item that starts
// last ends the call.  8 tasks of 6,000 + 380 tokens took 260 us so, 302 in column order.
// Larger calls keep the order of the columns throughout: full-size re-prefills were 10%
// slower with their items sorted.
template <class Item, class Make, class Tiles>
std::vector<Item> interleave(const std::vector<std::vector<Piece>>& queues, Make make, Tiles tiles) {
  std::vector<std::vector<Item>> per(kXcds);
  size_t depth = 0, total = 0;
  int32_t longest = 1;
  for (int x = 0; x < kXcds; ++x) {
    size_t n = 0;
    for (const Piece& p : queues[x]) n += p.k1 - p.k0;
    per[x].reserve(n);
    for (const Piece& p : queues[x])
      for (int32_t k = p.k0; k < p.k1; ++k) {
        per[x].push_back(make(k, p.g, std::max(p.c, 0)));
        longest = std::max(longest, tiles(k, std::max(p.c, 0)));
      }
    depth = std::max(depth, per[x].size());
    total += per[x].size();
  }
  if (total <= (size_t)kSplitMaxItems && depth > (size_t)(kCus / kXcds))
    for (int x = 0; x < kXcds; ++x) {
      std::vector<uint8_t> cls;  // length class of each item, 0 .. 8
      cls.reserve(per[x].size());
      int32_t at[10] = {};       // first place of each class, longest first
      for (const Piece& p : queues[x])
        for (int32_t k = p.k0; k < p.k1; ++k) {
          cls.push_back((uint8_t)((int64_t)tiles(k, std::max(p.c, 0)) * 8 / longest));
          ++at[8 - cls.back() + 1];
        }
      for (int i = 1; i < 10; ++i) at[i] += at[i - 1];
      std::vector<Item> sorted(per[x].size());
      for (size_t i = 0; i < cls.size(); ++i) sorted[at[8 - cls[i]]++] = per[x][i];
      per[x].swap(sorted);
    }
  std::vector<Item> items(depth * kXcds);  // value-initialised: ntok == 0
  for (int x = 0; x < kXcds; ++x)
    for (size_t i = 0; i < per[x].size(); ++i) items[i * kXcds + x] = per[x][i];
  while (!items.empty() && items.back().ntok == 0) items.pop_back();
  return items;
}

template <class Item>
void to_bytes(const std::vector<Item>& v, std::vector<uint8_t>* out) {
  out->resize(v.size() * sizeof(Item));
  if (!v.empty()) memcpy(out->data(), v.data(), out->size());
}

int plan_extend(const std::vector<TaskDesc>& tasks, const tide_dims& dims, bool build_blob,
                Plan* plan, std::vector<uint8_t>* items_bytes, std::vector<uint8_t>* merge_bytes,
                int64_t* n_items) {
  const int32_t group = dims.num_q_heads / dims.num_kv_heads;
  const int32_t waves = extend_waves(dims.head_dim, group);
  const int32_t tb = waves * 32 / group;  // tokens per item: waves*32 rows of (token, head)
  const int32_t hkv = dims.num_kv_heads;
  plan->waves = waves;
  plan->tokens_per_item = tb;
  // one workgroup-tile: 64 keys against 256 query rows, two products
  const double tile_us = 4.0 * kExtendKeyTile * (waves * 32) * dims.head_dim / kCuFlopsPerUs;

  // Blocks of each task, latest first (later blocks see more keys).
  const int32_t ntasks = (int32_t)tasks.size();
  std::vector<int32_t> task_first((size_t)ntasks + 1, 0);
  int64_t nblocks = 0;
  for (int32_t b = 0; b < ntasks; ++b) nblocks += (tasks[b].extend + tb - 1) / tb;
  if (nblocks * hkv > INT32_MAX / 4) return TIDE_ERR_INVALID_ARG;
  std::vector<Block> blocks;
  blocks.reserve((size_t)nblocks);
  for (int32_t b = 0; b < ntasks; ++b) {
    task_first[b] = (int32_t)blocks.size();
    const int32_t p = tasks[b].prefix, e = tasks[b].extend;
    for (int32_t k = (e + tb - 1) / tb - 1; k >= 0; --k) {
      Block bl;
      bl.task = b;
      bl.tok0 = k * tb;
      bl.ntok = std::min(tb, e - k * tb);
      bl.ntiles = (int32_t)(((int64_t)p + bl.tok0 + bl.ntok + kExtendKeyTile - 1) / kExtendKeyTile);
      blocks.push_back(bl);
    }
  }
  task_first[ntasks] = (int32_t)blocks.size();
  const int64_t plain_items = nblocks * hkv;

  // TIDE_EXTEND_SPLIT=0 keeps the plain plan, =1 takes the best split plan whenever one
  // exists (both for tests and tuning); otherwise the estimate decides.
  const char* env = getenv("TIDE_EXTEND_SPLIT");
  const int mode = (env && env[0] == '0') ? 0 : (env && env[0] == '1') ? 1 : -1;
  int32_t T = 0;
  if (mode != 0 && plain_items > 0 && plain_items <= kSplitMaxItems) {
    int64_t slots = 0, tiles = 0;
    int32_t longest = 0;
    for (const Block& b : blocks) {
      tiles += b.ntiles;
      longest = std::max(longest, b.ntiles);
    }
    const double plain_us =
        estimate(blocks, longest, dims, 0, tile_us, &slots);
    plan->est_plain_us = plan->est_us = plain_us;
    double best_us = mode == 1 ? INFINITY : plain_us * kSplitGain;
    // T for each number of rounds: the shortest chunks that are no more than the CUs take
    int32_t last = -1;
    int worse = 0;
    for (const int quarters : kQuarterRounds) {
      if (longest <= kMinChunkTiles) break;
      if (quarters < 4 && longest <= kManyChunks * kMinChunkTiles) continue;
      if ((double)tiles * hkv / kCus * tile_us * (1.0 - kIdleClockGain) + quarters / 4 * kChunkUs >=
          best_us)
        break;  // more rounds cannot win
      const int64_t room = (int64_t)quarters * kCus / 4 / hkv;
      if ((int64_t)blocks.size() > room) continue;
      auto fits = [&](int32_t t) {
        ++plan->search_passes;
        int64_t n = 0;
        for (const Block& b : blocks) n += num_chunks(b.ntiles, t);
        return n <= room;
      };
      // (steps that double, then a bisection: a scan took 440 us of planning on one long task
      // among many short ones, this takes 100)
      int32_t lo = (int32_t)std::max<int64_t>(kMinChunkTiles, ceil_div(tiles, room)) - 1, hi = lo + 1;
      while (hi < longest && !fits(hi)) {
        const int32_t next = (int32_t)std::min<int64_t>(longest, hi + 2 * (int64_t)(hi - lo));
        lo = hi;
        hi = next;
      }
      hi = std::min(hi, longest);  // (T = longest: one chunk a block, which fits)
      while (hi - lo > 1) {
        const int32_t mid = lo + (hi - lo) / 2;
        if (fits(mid)) hi = mid;
        else lo = mid;
      }
      if (hi == last) continue;
      last = hi;
      const double us = estimate(blocks, longest, dims, hi, tile_us, &slots);
      if (slots > 0 && slots <= INT32_MAX / 2 && us < best_us) {
        best_us = plan->est_us = us;
        T = hi;
        worse = 0;
      } else if (T > 0 && ++worse == 2) {
        break;
      }
    }
  }

  std::vector<int32_t> nchunks(blocks.size());
  for (size_t k = 0; k < blocks.size(); ++k) nchunks[k] = num_chunks(blocks[k].ntiles, T);
  const std::vector<std::vector<Piece>> queues = place(blocks, task_first, nchunks, hkv, T);
  plan->split = T > 0;
  plan->chunk = T;
  if (T == 0) {
    const std::vector<ExtendItem> items = interleave<ExtendItem>(
        queues, [&](int32_t k, int32_t g, int32_t) {
          return ExtendItem{blocks[k].task, g, blocks[k].tok0, blocks[k].ntok};
        },
        [&](int32_t k, int32_t) { return blocks[k].ntiles; });
    *n_items = (int64_t)items.size();
    if (build_blob) to_bytes(items, items_bytes);
    return TIDE_OK;
  }

  // partial row slots of the split blocks
  std::vector<int32_t> pbase(blocks.size(), 0);
  int64_t slots = 0;
  for (size_t k = 0; k < blocks.size(); ++k)
    if (nchunks[k] > 1) {
      pbase[k] = (int32_t)slots;
      slots += (int64_t)blocks[k].ntok * nchunks[k];
    }
  plan->row_slots = slots;
  const std::vector<ExtendChunkItem> items = interleave<ExtendChunkItem>(
      queues, [&](int32_t k, int32_t g, int32_t c) {
        const int32_t n = nchunks[k];
        ExtendChunkItem it;
        it.task = blocks[k].task;
        it.kv_head = g;
        it.tok0 = blocks[k].tok0;
        it.ntok = blocks[k].ntok;
        it.t_begin = chunk_begin(blocks[k].ntiles, n, c);
        it.t_end = chunk_begin(blocks[k].ntiles, n, c + 1);
        it.split = n > 1 ? c : -1;
        it.pbase = pbase[k];
        return it;
      },
      [&](int32_t k, int32_t c) { return chunk_tiles(blocks[k].ntiles, nchunks[k], c); });
  *n_items = (int64_t)items.size();
  if (build_blob) {
    to_bytes(items, items_bytes);
    std::vector<MergeRow> rows((size_t)plan->total_rows, MergeRow{0, 0, 0, 0});
    for (size_t k = 0; k < blocks.size(); ++k) {
      if (nchunks[k] < 2) continue;
      const int32_t r0 = tasks[blocks[k].task].row_start + blocks[k].tok0;
      for (int32_t tk = 0; tk < blocks[k].ntok; ++tk)
        rows[r0 + tk] = MergeRow{pbase[k] + tk, blocks[k].ntok, nchunks[k], 0};
    }
    to_bytes(rows, merge_bytes);
  }
  return TIDE_OK;
}

}  // namespace

int make_plan(int op, int32_t num_tasks, const int32_t* lens_a, const int32_t* lens_b,
              const tide_dims& dims, int32_t num_splits, int32_t bt_stride, bool build_blob,
              Plan* plan) {
  if (!plan) return TIDE_ERR_INVALID_ARG;
  if (op != TIDE_OP_KV_APPEND && op != TIDE_OP_EXTEND && op != TIDE_OP_DECODE &&
      op != TIDE_OP_FULL_PREFILL)
    return TIDE_ERR_INVALID_ARG;
  if (num_tasks < 0) return TIDE_ERR_INVALID_ARG;
  if (num_tasks > 0 && !lens_a) return TIDE_ERR_INVALID_ARG;
  if (num_tasks > 0 && (op == TIDE_OP_KV_APPEND || op == TIDE_OP_EXTEND) && !lens_b)
    return TIDE_ERR_INVALID_ARG;
  if (op == TIDE_OP_DECODE && num_splits < 0) return TIDE_ERR_INVALID_ARG;
  int rc = check_dims(&dims);
  if (rc != TIDE_OK) return rc;

  *plan = Plan();
  plan->op = op;
  plan->num_tasks = num_tasks;

  std::vector<TaskDesc> tasks((size_t)num_tasks);
  int64_t rows = 0;
  int64_t max_len = 0;
  for (int32_t b = 0; b < num_tasks; ++b) {
    int32_t p = 0, e = 0;
    rc = task_lengths(op, b, lens_a, lens_b, &p, &e);
    if (rc != TIDE_OK) return rc;
    tasks[b].row_start = (int32_t)(op == TIDE_OP_DECODE ? b : rows);
    tasks[b].prefix = p;
    tasks[b].extend = e;
    tasks[b].aux = 0;
    rows += (op == TIDE_OP_DECODE) ? 1 : e;
    if (rows > INT32_MAX) return TIDE_ERR_INVALID_ARG;
    max_len = std::max<int64_t>(max_len, (int64_t)p + e);
    if (bt_stride >= 0 && ceil_div((int64_t)p + e, kPage) > bt_stride) return TIDE_ERR_CAPACITY;
  }
  plan->total_rows = (int32_t)rows;

  // ---- work items -------------------------------------------------------------------
  std::vector<uint8_t> items_bytes, merge_bytes;
  int64_t n_items = 0;
  if (op == TIDE_OP_KV_APPEND) {
    std::vector<AppendItem> items;
    for (int32_t b = 0; b < num_tasks; ++b) {
      const int32_t p = tasks[b].prefix, e = tasks[b].extend;
      if (e == 0) continue;
      for (int64_t lp = p / kPage; lp <= (int64_t)(p + e - 1) / kPage; ++lp) {
        AppendItem it;
        it.task = b;
        it.lpage = (int32_t)lp;
        it.pos_begin = (int32_t)std::max<int64_t>(p, lp * kPage);
        it.pos_end = (int32_t)std::min<int64_t>((int64_t)p + e, (lp + 1) * kPage);
        items.push_back(it);
      }
    }
    n_items = (int64_t)items.size();
    if (build_blob) {
      items_bytes.resize(items.size() * sizeof(AppendItem));
      if (!items.empty()) memcpy(items_bytes.data(), items.data(), items_bytes.size());
    }
  } else if (op == TIDE_OP_EXTEND || op == TIDE_OP_FULL_PREFILL) {
    rc = plan_extend(tasks, dims, build_blob, plan, &items_bytes, &merge_bytes, &n_items);
    if (rc != TIDE_OK) return rc;
  } else {  // decode
    int64_t chunk = 0;
    if (num_splits > 0) {
      for (int32_t b = 0; b < num_tasks; ++b)
        chunk = std::max<int64_t>(chunk, ceil_div(tasks[b].prefix + 1, num_splits));
      chunk = std::max<int64_t>(kDecodeStep, ceil_div(chunk, kDecodeStep) * kDecodeStep);
    } else {
      chunk = decode_auto_chunk(tasks, dims.num_kv_heads);
    }
    int32_t max_splits = 0;
    std::vector<DecodeItem> items;
    for (int32_t b = 0; b < num_tasks; ++b) {
      const int64_t kv = (int64_t)tasks[b].prefix + 1;
      const int32_t s = (int32_t)ceil_div(kv, chunk);
      tasks[b].aux = s;
      max_splits = std::max(max_splits, s);
      for (int32_t sp = 0; sp < s; ++sp)
        for (int32_t g = 0; g < dims.num_kv_heads; ++g) {
          DecodeItem it;
          it.task = b;
          it.kv_head = g;
          it.split = sp;
          it.k_begin = (int32_t)(sp * chunk);
          items.push_back(it);
        }
    }
    // Longest first: the shorter last chunks of the tasks then run at the end of the
    // launch, while the CUs that free up early still find work (the result does not
    // depend on the order: each split writes its own partial slot).
    {
      auto keys = [&](const DecodeItem& x) {
        return std::min<int64_t>(chunk, (int64_t)tasks[x.task].prefix + 1 - x.k_begin);
      };
      std::vector<DecodeItem> tail;  // every task's last, shorter chunk
      size_t nfull = 0;
      for (const DecodeItem& it : items) {
        if (keys(it) == chunk) items[nfull++] = it;
        else tail.push_back(it);
      }
      std::stable_sort(tail.begin(), tail.end(),
                       [&](const DecodeItem& x, const DecodeItem& y) { return keys(x) > keys(y); });
      std::copy(tail.begin(), tail.end(), items.begin() + nfull);
    }
    plan->chunk = (int32_t)chunk;
    plan->max_splits = max_splits;
    n_items = (int64_t)items.size();
    // The split kernel merges a (task, kv head) in its last split when tasks have few
    // splits on average; with many, the merge tail at the end of the launch (each merge
    // one wave, latency-bound) costs more than a merge kernel (measured on MI355X: at 2.5
    // splits per task the fold saves the merge kernel's 10 us; at 16 it adds 40-57 us).
    // (and the partial rows of one (task, kv head) must fit a 32-bit buffer range)
    plan->fold_merge = n_items <= (int64_t)kFoldMeanSplits * num_tasks * dims.num_kv_heads &&
                       (int64_t)(dims.num_q_heads / dims.num_kv_heads) * max_splits *
                               dims.head_dim * 4 <= INT32_MAX;
    if (build_blob) {
      items_bytes.resize(items.size() * sizeof(DecodeItem));
      if (!items.empty()) memcpy(items_bytes.data(), items.data(), items_bytes.size());
    }
  }
  if (n_items > INT32_MAX / 4) return TIDE_ERR_INVALID_ARG;
  plan->num_items = (int32_t)n_items;
  const size_t item_size = plan->split ? sizeof(ExtendChunkItem) : 16;

  // ---- layout -------------------------------------------------------------------------
  size_t off = sizeof(WsHeader);
  plan->tasks_off = off;
  off = align_up(off + tasks.size() * sizeof(TaskDesc), kWsAlign);
  plan->items_off = off;
  off = align_up(off + (size_t)n_items * item_size, kWsAlign);
  if (plan->split) {
    plan->merge_rows_off = off;
    off = align_up(off + (size_t)plan->total_rows * sizeof(MergeRow), kWsAlign);
  }
  if (op == TIDE_OP_DECODE) {  // left zero in the blob: every call starts the counts at 0
    plan->tickets_off = off;
    off = align_up(off + (size_t)num_tasks * dims.num_kv_heads * sizeof(int32_t), kWsAlign);
  }
  plan->upload_bytes = off;
  if (plan->split) {
    const size_t slots = (size_t)plan->row_slots * dims.num_q_heads;
    plan->part_o_off = off;
    off = align_up(off + slots * dims.head_dim * sizeof(float), kWsAlign);
    plan->part_ml_off = off;
    off = align_up(off + slots * 4 * sizeof(float), kWsAlign);
  }
  if (op == TIDE_OP_DECODE) {
    const size_t slots = (size_t)num_tasks * dims.num_q_heads * (size_t)plan->max_splits;
    plan->part_o_off = off;
    off = align_up(off + slots * dims.head_dim * sizeof(float), kWsAlign);
    plan->part_ml_off = off;
    off = align_up(off + slots * 4 * sizeof(float), kWsAlign);
  }
  plan->total_bytes = off;

  if (build_blob) {
    plan->blob.assign(plan->upload_bytes, 0);
    if (!tasks.empty())
      memcpy(plan->blob.data() + plan->tasks_off, tasks.data(), tasks.size() * sizeof(TaskDesc));
    if (!items_bytes.empty())
      memcpy(plan->blob.data() + plan->items_off, items_bytes.data(), items_bytes.size());
    if (plan->split && !merge_bytes.empty())
      memcpy(plan->blob.data() + plan->merge_rows_off, merge_bytes.data(), merge_bytes.size());
  }
  return TIDE_OK;
}

// Decode cut into equal runs of key steps (attn_decode_stream.hip): the fewest steps a run with
// which runs x kv heads fit the waves the device holds at once.  Calls of longer runs than
// kStreamMaxSteps keep the chunks of make_plan: there the start and end of a wave no longer
// matter, and chunks, whose waves all read whole tasks in step, draw slightly more from the
// memory.  Measured on MI355X (call us, chunks against runs): 190 steps 1013 / 957, 187 steps
// 945 / 928, 225 steps (256 tasks of 1k-32k, 32 / 8 heads) 1140 / 1141, 246 steps (32 of
// 32k-96k, 64 / 8 heads) 1214 / 1248.
// With few kv heads a task has many runs, and the one wave that merges its parts (a batch of loads
// after the other, 0.25 us a part) outlasts short runs (0.6 us a step): the sum of both is least
// where steps^2 is in proportion to the task's length.  One task of 60,000 keys (1875 steps), 32 /
// 2 heads, d = 64: 2 steps a run 46.2 us, 3 35.5, 4 31.7, 6 27.5, 8 28.9, 16 29.3 (chunks 28.0);
// 30,000 keys, 8 / 2 heads: 1 step 24.1, 2 17.5, 4 16.3, 6 18.4, 12 19.7 (chunks 24.1).
// Over 8 query heads a kv head of d = 128 take the merging wave two passes of twice the loads, and
// there the steps are those for which a run's steps and the parts of the longest task cost least
// (8 waves of a workgroup share a CU and so a step costs more, but make one part): 16 / 1 heads, one
// task of 30,000 keys 40.6 us with the rule above (4 steps) and 31.9 so (10), 9,000 27.2 (2) and
// 21.4 (6), 2 of 90,000 62.3 (9) and 59.9 (12); no slower than 2% on 27 other calls.
int make_plan_decode(int32_t num_tasks, const int32_t* kv_lens, const tide_dims& dims,
                     int32_t num_splits, int32_t bt_stride, bool build_blob, Plan* plan) {
  if (!plan || num_tasks < 0 || num_splits < 0) return TIDE_ERR_INVALID_ARG;
  if (num_splits > 0 || num_tasks == 0 || !kv_lens)
    return make_plan(TIDE_OP_DECODE, num_tasks, kv_lens, nullptr, dims, num_splits, bt_stride,
                     build_blob, plan);
  const int rc = check_dims(&dims);
  if (rc != TIDE_OK) return rc;
  int64_t total = 0, longest = 0;  // steps of all tasks (one kv head) and of one
  for (int32_t b = 0; b < num_tasks; ++b) {
    if (kv_lens[b] <= 0) return TIDE_ERR_INVALID_ARG;
    if (bt_stride >= 0 && ceil_div(kv_lens[b], kPage) > bt_stride) return TIDE_ERR_CAPACITY;
    const int64_t st = ceil_div(kv_lens[b], kDecodeStep);
    total += st;
    longest = std::max(longest, st);
  }
  const int32_t hkv = dims.num_kv_heads;
  int64_t steps = ceil_div(total, std::max<int64_t>(1, kDecodeWaveSlots / hkv));
  const int32_t group = dims.num_q_heads / hkv;
  if (group > 8 && dims.head_dim > 64) {
    int64_t best = steps;
    double best_us = INFINITY;
    for (int64_t s = steps; s <= kStreamMaxSteps && s * kStreamStepUs < best_us; ++s) {
      const int32_t waves = stream_waves(ceil_div(total, s) * hkv);
      const double us = s * (waves > 4 ? kStreamBusyStepUs : kStreamStepUs) +
                        ceil_div(ceil_div(longest, s), waves) * kStreamPartUs;
      if (us < best_us) best_us = us, best = s;
    }
    steps = best;
  } else {
    while (kStreamMergeSteps * (steps + 1) * (steps + 1) <= longest) ++steps;
  }
  if (steps > kStreamMaxSteps)
    return make_plan(TIDE_OP_DECODE, num_tasks, kv_lens, nullptr, dims, num_splits, bt_stride,
                     build_blob, plan);
  *plan = Plan();
  plan->op = TIDE_OP_DECODE;
  plan->num_tasks = num_tasks;
  plan->total_rows = num_tasks;
  plan->stream = true;
  plan->fold_merge = true;
  plan->steps = (int32_t)steps;
  plan->num_runs = (int32_t)ceil_div(total, plan->steps);
  plan->last_steps = (int32_t)(total - (int64_t)(plan->num_runs - 1) * plan->steps);
  plan->num_items = plan->num_runs * hkv;
  plan->chunk = plan->steps * kDecodeStep;
  plan->max_splits = (int32_t)std::min<int64_t>(longest, ceil_div(longest - 1, plan->steps) + 1);

  size_t off = sizeof(WsHeader);
  plan->tasks_off = off;
  off = align_up(off + (size_t)num_tasks * sizeof(TaskDesc), kWsAlign);
  plan->items_off = off;
  off = align_up(off + (size_t)plan->num_runs * sizeof(StreamItem), kWsAlign);
  const StreamSlots per_head = {plan->num_runs, num_tasks, stream_waves(plan->num_items)};
  plan->tickets_off = off;  // the parts' flags, zero in the blob
  off = align_up(off + (size_t)per_head.count() * hkv * sizeof(uint64_t), kWsAlign);
  plan->upload_bytes = off;
  const size_t slots = (size_t)per_head.count() * dims.num_q_heads;
  plan->part_o_off = off;
  off = align_up(off + slots * dims.head_dim * sizeof(float), kWsAlign);
  plan->part_ml_off = off;
  off = align_up(off + slots * 4 * sizeof(float), kWsAlign);
  plan->total_bytes = off;
  if (!build_blob) return TIDE_OK;

  plan->blob.assign(plan->upload_bytes, 0);
  TaskDesc* tasks = reinterpret_cast<TaskDesc*>(plan->blob.data() + plan->tasks_off);
  StreamItem* items = reinterpret_cast<StreamItem*>(plan->blob.data() + plan->items_off);
  int64_t at = 0, run = 0;  // first step of the task, next run to place
  for (int32_t b = 0; b < num_tasks; ++b) {
    tasks[b] = TaskDesc{b, kv_lens[b] - 1, 1, 0};
    const int64_t end = at + ceil_div(kv_lens[b], kDecodeStep);
    for (; run * plan->steps < end; ++run)
      items[run] = StreamItem{b, (int32_t)(run * plan->steps - at), kv_lens[b], 0};
    at = end;
  }
  return TIDE_OK;
}

size_t compact_runs(Plan* plan) {
  TaskDesc* tasks = reinterpret_cast<TaskDesc*>(plan->blob.data() + plan->tasks_off);
  uint8_t* to = plan->blob.data() + plan->items_off;
  const StreamItem* items = reinterpret_cast<const StreamItem*>(to);
  int32_t at = 0;
  for (int32_t b = 0; b < plan->num_tasks; ++b) {
    tasks[b].aux = at;
    at += (tasks[b].prefix + kDecodeStep) / kDecodeStep;
  }
  for (int32_t r = 0; r < plan->num_runs; ++r) {  // (never past the record it reads)
    const int32_t task = items[r].task;
    memcpy(to + r * sizeof(int32_t), &task, sizeof(int32_t));
  }
  return plan->items_off + plan->num_runs * sizeof(int32_t);
}

int make_plan_shared(int32_t num_tasks, const int32_t* kv_lens, int32_t num_groups,
                     const int32_t* group_start, const int32_t* shared_lens,
                     const tide_dims& dims, int32_t num_splits, int32_t bt_stride,
                     bool build_blob, Plan* plan) {
  if (!plan) return TIDE_ERR_INVALID_ARG;
  int rc = check_dims(&dims);
  if (rc != TIDE_OK) return rc;
  if (num_tasks < 0 || num_splits < 0 || num_groups < 0) return TIDE_ERR_INVALID_ARG;
  *plan = Plan();
  plan->op = kOpDecodeShared;
  plan->num_tasks = num_tasks;
  if (num_tasks > 0) {
    if (!kv_lens || !group_start || !shared_lens || num_groups < 1) return TIDE_ERR_INVALID_ARG;
    if (group_start[0] != 0 || group_start[num_groups] != num_tasks) return TIDE_ERR_INVALID_ARG;
  }
  const int32_t group = dims.num_q_heads / dims.num_kv_heads;
  const int32_t per_item = std::max<int32_t>(1, 16 / group);  // trajectories per prefix item

  std::vector<TaskDesc> tasks((size_t)num_tasks);
  std::vector<int32_t> shared_of((size_t)num_tasks, 0);
  for (int32_t g = 0; g < (num_tasks > 0 ? num_groups : 0); ++g) {
    const int32_t s0 = group_start[g], s1 = group_start[g + 1];
    const int32_t sh = shared_lens[g];
    if (s1 <= s0 || s1 > num_tasks) return TIDE_ERR_INVALID_ARG;
    if (sh < 0 || sh % kPage != 0) return TIDE_ERR_INVALID_ARG;
    for (int32_t b = s0; b < s1; ++b) {
      if (kv_lens[b] <= 0 || sh > kv_lens[b] - 1) return TIDE_ERR_INVALID_ARG;
      if (bt_stride >= 0 && ceil_div(kv_lens[b], kPage) > bt_stride) return TIDE_ERR_CAPACITY;
      tasks[b] = TaskDesc{b, kv_lens[b] - 1, 1, 0};
      shared_of[b] = sh;
    }
  }
  plan->total_rows = num_tasks;

  int64_t chunk = 0;
  if (num_splits > 0) {
    for (int32_t b = 0; b < num_tasks; ++b)
      chunk = std::max<int64_t>(chunk, ceil_div(kv_lens[b], num_splits));
    chunk = std::max<int64_t>(kDecodeStep, ceil_div(chunk, kDecodeStep) * kDecodeStep);
  } else {
    // One round of waves, if chunks of at most kSharedRoundChunk keys can be that few: the
    // shortest that are.  Otherwise the item rule of decode, counting a shared prefix once per
    // item group.  Measured on MI355X (call us, item rule against one round of the chunk named):
    // 32 tasks in groups of 4, prompts of 2k-6k and 2k-16k keys of their own (32 / 8 heads) 167 /
    // 154 at 992; 64 in groups of 8, 4k-6k and 0.5k-4k (8 / 8) 122 / 102 at 672; 80 in groups of
    // 4, 4k-8k and 0.3k-4k (32 / 8) 173 / 165 at 1056.  Longer ones gain less for the shape's
    // raggedness: 181 / 177 at 1344, 212 / 210 at 1504, 156 / 160 at 1536 (64 / 8, 80 tasks).
    auto items_at = [&](int64_t c) {
      int64_t n = 0;
      for (int32_t g = 0; g < (num_tasks > 0 ? num_groups : 0); ++g)
        n += ceil_div(group_start[g + 1] - group_start[g], per_item) * ceil_div(shared_lens[g], c);
      for (int32_t b = 0; b < num_tasks; ++b) n += ceil_div((int64_t)kv_lens[b] - shared_of[b], c);
      return n * dims.num_kv_heads;
    };
    if (items_at(kSharedRoundChunk) <= kDecodeWaveSlots) {
      int64_t lo = kDecodeMinChunk / kDecodeStep, hi = kSharedRoundChunk / kDecodeStep;
      if (items_at(kDecodeMinChunk) <= kDecodeWaveSlots) hi = lo;
      while (hi - lo > 1) {
        const int64_t mid = (lo + hi) / 2;
        if (items_at(mid * kDecodeStep) <= kDecodeWaveSlots) hi = mid;
        else lo = mid;
      }
      chunk = hi * kDecodeStep;
    } else {
      int64_t total = 0;
      for (int32_t g = 0; g < (num_tasks > 0 ? num_groups : 0); ++g) {
        const int32_t n = group_start[g + 1] - group_start[g];
        total += ceil_div(n, per_item) * (int64_t)shared_lens[g];
      }
      for (int32_t b = 0; b < num_tasks; ++b) total += (int64_t)kv_lens[b] - shared_of[b];
      total *= dims.num_kv_heads;
      chunk = ceil_div(total, kDecodeTargetItems);
      chunk = ceil_div(chunk, kDecodeStep) * kDecodeStep;
      chunk = std::min<int64_t>(std::max<int64_t>(chunk, kDecodeMinChunk), kDecodeMaxChunk);
    }
  }

  std::vector<SharedDecodeItem> items;
  int32_t max_splits = 0;
  for (int32_t g = 0; g < (num_tasks > 0 ? num_groups : 0); ++g) {
    const int32_t s0 = group_start[g], s1 = group_start[g + 1], sh = shared_lens[g];
    const int32_t np = (int32_t)ceil_div(sh, chunk);
    // The items of one (kv head, chunk) -- one per run of per_item trajectories -- read the
    // same prefix keys.  They are consecutive, so they share a workgroup of the decode
    // kernel (four or eight waves by launch size, one item each, on one CU) or a
    // neighbouring one, and the later reads hit that XCD's L2.
    for (int32_t h = 0; h < dims.num_kv_heads; ++h)
      for (int32_t j = 0; j < np; ++j)
        for (int32_t f = s0; f < s1; f += per_item) {
          SharedDecodeItem it = {};
          it.first_task = f;
          it.ntasks = std::min(per_item, s1 - f);
          it.kv_head = h;
          it.split = j;
          it.k_begin = (int32_t)(j * chunk);
          it.k_end = (int32_t)std::min<int64_t>(sh, (j + 1) * chunk);
          items.push_back(it);
        }
    for (int32_t b = s0; b < s1; ++b) {
      const int32_t ns = (int32_t)ceil_div((int64_t)kv_lens[b] - sh, chunk);
      tasks[b].aux = np + ns;
      max_splits = std::max(max_splits, np + ns);
      for (int32_t h = 0; h < dims.num_kv_heads; ++h)
        for (int32_t i = 0; i < ns; ++i) {
          SharedDecodeItem it = {};
          it.first_task = b;
          it.ntasks = 1;
          it.kv_head = h;
          it.split = np + i;
          it.k_begin = (int32_t)(sh + i * chunk);
          it.k_end = (int32_t)std::min<int64_t>(kv_lens[b], sh + (i + 1) * chunk);
          items.push_back(it);
        }
    }
  }
  // Longest first, as for plain decode.  The sort is stable and the items of one prompt
  // chunk have equal lengths and are adjacent, so they stay adjacent.
  std::stable_sort(items.begin(), items.end(),
                   [](const SharedDecodeItem& x, const SharedDecodeItem& y) {
                     return x.k_end - x.k_begin > y.k_end - y.k_begin;
                   });
  if ((int64_t)items.size() > INT32_MAX / 4) return TIDE_ERR_INVALID_ARG;
  plan->chunk = (int32_t)chunk;
  plan->max_splits = max_splits;
  plan->num_items = (int32_t)items.size();

  size_t off = sizeof(WsHeader);
  plan->tasks_off = off;
  off = align_up(off + tasks.size() * sizeof(TaskDesc), kWsAlign);
  plan->items_off = off;
  off = align_up(off + items.size() * sizeof(SharedDecodeItem), kWsAlign);
  plan->upload_bytes = off;
  const size_t slots = (size_t)num_tasks * dims.num_q_heads * (size_t)max_splits;
  plan->part_o_off = off;
  off = align_up(off + slots * dims.head_dim * sizeof(float), kWsAlign);
  plan->part_ml_off = off;
  off = align_up(off + slots * 4 * sizeof(float), kWsAlign);
  plan->total_bytes = off;
  if (build_blob) {
    plan->blob.assign(plan->upload_bytes, 0);
    if (!tasks.empty())
      memcpy(plan->blob.data() + plan->tasks_off, tasks.data(), tasks.size() * sizeof(TaskDesc));
    if (!items.empty())
      memcpy(plan->blob.data() + plan->items_off, items.data(), items.size() * sizeof(SharedDecodeItem));
  }
  return TIDE_OK;
}

}  // namespace tide
