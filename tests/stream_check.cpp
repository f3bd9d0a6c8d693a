// Host-side check of the decode plan of equal runs of steps (make_plan_decode), compiled with
// g++ by test_decode_stream.py; no GPU involved.  Each stdin line is a call, "hq hkv d ntasks
// kv_0 ..": the checker walks every run as the kernel's waves do (all kv heads alike) and
// verifies that
//   * the runs tile the tasks' steps in order, and each record names its run's first step;
//   * every cut task's parts, as each of its waves derives them, agree; the slots written
//     are distinct, in bounds, the ones the merge reads, and in key order; and as many parts
//     are flagged as the merge waits for;
//   * the workspace regions lie in order, the flags zero in the upload;
//   * the compact form of the runs (compact_runs) names the same ones.
#include <stdio.h>

#include <algorithm>
#include <iostream>
#include <map>
#include <sstream>
#include <string>
#include <vector>

#include "plan.h"

using namespace tide;

static int fail(const char* what, long a = 0, long b = 0) {
  printf("FAIL %s %ld %ld\n", what, a, b);
  return 1;
}

struct Seen {
  StreamUnit u;
  std::map<int, int> slots;  // slot -> first step of the part
  int arrivals = 0, covered = 0;
};

static int check(const tide_dims& dims, const std::vector<int32_t>& kv) {
  const int n = (int)kv.size(), hkv = dims.num_kv_heads, G = dims.num_q_heads / hkv;
  Plan plan, sized;
  if (make_plan_decode(n, kv.data(), dims, 0, -1, true, &plan) != TIDE_OK) return fail("plan");
  if (make_plan_decode(n, kv.data(), dims, 0, -1, false, &sized) != TIDE_OK ||
      sized.total_bytes != plan.total_bytes || sized.num_items != plan.num_items)
    return fail("size-only plan differs");
  if (!plan.stream) {  // long runs take the chunk plan, which plan_check.cpp checks
    printf("ok chunks\n");
    return 0;
  }
  if (plan.num_runs < 1 || plan.num_items != plan.num_runs * hkv ||
      plan.num_items > std::max(2048, hkv))
    return fail("waves", plan.num_items);
  const size_t R = plan.num_runs;
  const int per = stream_waves(plan.num_items);
  const StreamSlots sl = {plan.num_runs, n, per};
  const size_t slots = sl.count();
  std::map<int, int> used;  // slot -> task
  if (plan.items_off < plan.tasks_off + n * sizeof(TaskDesc) ||
      plan.tickets_off < plan.items_off + R * sizeof(StreamItem) ||
      plan.upload_bytes < plan.tickets_off + 8 * slots * hkv || plan.blob.size() != plan.upload_bytes ||
      plan.part_o_off < plan.upload_bytes ||
      plan.part_ml_off < plan.part_o_off + slots * hkv * G * dims.head_dim * 4 ||
      plan.total_bytes < plan.part_ml_off + slots * hkv * G * 16)
    return fail("layout");
  for (size_t i = plan.tickets_off; i < plan.upload_bytes; ++i)
    if (plan.blob[i]) return fail("flag not zero", (long)i);
  const TaskDesc* tasks = (const TaskDesc*)(plan.blob.data() + plan.tasks_off);
  const StreamItem* items = (const StreamItem*)(plan.blob.data() + plan.items_off);
  std::map<int, Seen> cut;
  int task = 0, step = 0;  // where the next run must begin
  for (int g = 0; g < (int)R / per + 1; ++g) {
    Seen* open[16] = {};  // what each run of the workgroup leaves unfinished
    int open_task[16], open_begin[16];
    for (int x = 0; x < per && g * per + x < (int)R; ++x) {
      const int r = g * per + x, count = r == (int)R - 1 ? plan.last_steps : plan.steps;
      if (count < 1 || count > plan.steps) return fail("run length", r, count);
      const StreamItem it = items[r];
      if (it.task != task || it.step != step || it.kv_len != kv[task]) return fail("record", r);
      int begin = step;
      for (int s = 0; s < count; ++s) {
        if (task >= n) return fail("run past the call", r);
        if (tasks[task].prefix + tasks[task].extend != kv[task] || tasks[task].row_start != task)
          return fail("task row", task);
        const int steps = (kv[task] + 31) / 32;
        const bool ends = ++step == steps, stops = s == count - 1;
        if (!ends && !stops) continue;
        if (begin > 0 || !ends) {  // a part of a cut task
          const StreamUnit u = stream_unit(r, begin, step - begin, steps, plan.steps);
          Seen& c = cut[task];
          if (c.covered == 0) c.u = u;
          if (c.u.w0 != u.w0 || c.u.n != u.n || c.u.ends_inside != u.ends_inside)
            return fail("runs disagree", task, r);
          if (r < u.w0 || r >= u.w0 + u.n || c.covered != begin) return fail("part order", task, r);
          c.covered = step;
          if (ends && step - begin < plan.steps) {
            if (!u.ends_inside || r != u.w0 + u.n - 1) return fail("end", task, r);
            const int slot = sl.ended(r, task);
            if (!used.insert({slot, task}).second) return fail("slot twice", slot);
            c.slots[slot] = begin;
            ++c.arrivals;
          } else {
            open[x] = &c;
            open_task[x] = task;
            open_begin[x] = begin;
          }
        }
        begin = 0;
        if (ends) step = 0, ++task;
      }
    }
    for (int x = 0; x < per; ++x) {  // the workgroup's combined parts
      if (!open[x] || (x > 0 && open[x - 1] && open_task[x - 1] == open_task[x])) continue;
      const int slot = sl.open(g * per + x, open_task[x]);
      if (!used.insert({slot, open_task[x]}).second) return fail("slot twice", slot);
      open[x]->slots[slot] = open_begin[x];
      ++open[x]->arrivals;
    }
  }
  if (task != n || step) return fail("steps left over", task, step);
  for (auto& kvp : cut) {
    Seen& c = kvp.second;
    if (c.covered != (kv[kvp.first] + 31) / 32) return fail("task not covered", kvp.first);
    const int np = stream_parts(c.u, per);
    if (np != c.arrivals || np != (int)c.slots.size()) return fail("arrivals", np, c.arrivals);
    int last = -1;
    for (int e = 0; e < np; ++e) {
      const auto f = c.slots.find(stream_slot(c.u, sl, kvp.first, e));
      if (f == c.slots.end() || f->first < 0 || f->first >= (int)slots) return fail("slot", e);
      if (f->second <= last) return fail("part order in the merge", e);
      last = f->second;
    }
  }
  // the compact form names the same runs
  const std::vector<StreamItem> full(items, items + R);
  const size_t bytes = compact_runs(&plan);
  if (bytes != plan.items_off + R * 4 || bytes > plan.blob.size()) return fail("compact bytes", (long)bytes);
  for (size_t r = 0; r < R; ++r) {
    const int32_t t = reinterpret_cast<const int32_t*>(plan.blob.data() + plan.items_off)[r];
    if (t != full[r].task || (int)r * plan.steps - tasks[t].aux != full[r].step ||
        tasks[t].prefix + tasks[t].extend != full[r].kv_len)
      return fail("compact run", (long)r);
  }
  printf("ok %d %d %zu\n", plan.num_items, plan.steps, cut.size());
  return 0;
}

int main() {
  std::string line;
  int bad = 0;
  while (std::getline(std::cin, line)) {
    std::istringstream in(line);
    int hq, hkv, d, n;
    if (!(in >> hq >> hkv >> d >> n)) continue;
    tide_dims dims = {hq, hkv, d, 16, 0.1f};
    std::vector<int32_t> kv(n);
    for (auto& x : kv) in >> x;
    bad |= check(dims, kv);
  }
  return bad;
}
