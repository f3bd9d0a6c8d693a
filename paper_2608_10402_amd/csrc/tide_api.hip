// The extern "C" entry points declared in include/tide.h: validation and planning on the
// host (plan.cpp), the work lists staged in a pinned ring, where a small call's kernel reads
// them and from where a copy kernel moves a larger one's into the caller's workspace (under
// graph capture they go there as kernel arguments), then the kernel launches, all on the
// caller's stream.
#include <hip/hip_runtime.h>
#include <stdlib.h>
#include <string.h>

#include <sched.h>

#include <algorithm>
#include <atomic>
#include <chrono>
#include <mutex>
#include <new>
#include <random>
#include <vector>

#include "kernels.h"
#include "plan.h"
#include "tide.h"

namespace tide {
namespace {

typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));

constexpr int kStagingSlots = 16;
// Slots start large and grow by powers of two, so that steady-state calls never
// reallocate: freeing and allocating pinned memory is slow and can stall the device.
constexpr size_t kStagingMin = 2u << 20;

// Pinned, device-mapped host buffers the work lists are staged in.  The call's own kernel
// reads a slot in place, or a kernel on the caller's stream copies it into the workspace (no
// DMA-engine copy, so no hand-off between engines on every call).  A slot is reused only once
// it has been read: each workgroup of its reader, after all its reads have returned, writes
// the slot's use count into its own flag in coherent host memory, and the host checks the
// flags before it overwrites the slot.  (A completion event recorded behind each copy did
// the same, but delayed the call's next kernel by several microseconds.)
struct StagingSlot {
  void* host = nullptr;
  const void* dev = nullptr;  // the same memory as seen from the device
  size_t cap = 0;
  uint32_t* flags = nullptr;  // one per reading workgroup, coherent host memory
  uint32_t* flags_dev = nullptr;
  uint32_t seq = 0;           // uses of the slot so far
  uint32_t nblocks = 0;       // workgroups of the last reader
  bool pending = false;
};

constexpr int kCopyBytesPerBlock = 256 * 16;

// 16 bytes per thread from the staging slot (host memory) into the workspace; then the
// workgroup's flag.  Every thread's load has returned once it has issued its store (the
// store needs the data), so after the barrier the workgroup has read all it will read.
__global__ __launch_bounds__(256) void stage_copy_kernel(u32x4_t* dst, const u32x4_t* src,
                                                         size_t n16, uint32_t* done, uint32_t seq) {
  const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (i < n16) dst[i] = src[i];
  __syncthreads();
  if (threadIdx.x == 0)
    __hip_atomic_store(done + blockIdx.x, seq, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// The same from the kernel's own arguments, which a captured graph holds a copy of.
constexpr uint32_t kPutWords = 240;  // 16 bytes each; a kernel's arguments hold up to 4 KB
struct PutArgs {
  u32x4_t* dst;
  uint32_t n16;
  u32x4_t data[kPutWords];
};

__global__ __launch_bounds__(256) void put_kernel(PutArgs a) {
  if (threadIdx.x < a.n16) a.dst[threadIdx.x] = a.data[threadIdx.x];
}

__global__ __launch_bounds__(256) void zero_kernel(u32x4_t* dst, uint32_t n16) {
  const uint32_t i = blockIdx.x * 256 + threadIdx.x;
  if (i < n16) dst[i] = u32x4_t{0u, 0u, 0u, 0u};
}

// Moves the plan into the workspace for a call under graph capture: as kernel arguments, 3,840
// bytes a launch, so that a replay needs nothing of the library's or the host's memory (a
// staging slot would hold a later call's plan by then).  The zeros a decode plan ends with are
// one launch.  A replay runs 3 such launches for 8 tasks' decode, 17 for 64 agents' extend.
int put_plan(const Plan& plan, void* workspace, hipStream_t stream) {
  const size_t need = plan.blob.size();  // a multiple of kWsAlign
  const size_t filled = plan.tickets_off ? plan.tickets_off : need;
  uint8_t* ws = static_cast<uint8_t*>(workspace);
  PutArgs a;
  for (size_t off = 0; off < filled; off += sizeof(a.data)) {
    const size_t bytes = std::min(sizeof(a.data), filled - off);
    a.dst = reinterpret_cast<u32x4_t*>(ws + off);
    a.n16 = (uint32_t)(bytes / 16);
    memcpy(a.data, plan.blob.data() + off, bytes);
    hipLaunchKernelGGL(put_kernel, dim3(1), dim3(256), 0, stream, a);
    if (hipGetLastError() != hipSuccess) return TIDE_ERR_HIP;
  }
  if (need > filled) {
    const uint32_t n16 = (uint32_t)((need - filled) / 16);
    hipLaunchKernelGGL(zero_kernel, dim3((n16 + 255) / 256), dim3(256), 0, stream,
                       reinterpret_cast<u32x4_t*>(ws + filled), n16);
    if (hipGetLastError() != hipSuccess) return TIDE_ERR_HIP;
  }
  return TIDE_OK;
}

// Waits until every workgroup of the slot's last reader has set its flag.  Normally it
// finished long ago; if not, this waits like a synchronisation on it would, and
// after a few seconds (TIDE_STAGING_WAIT_US microseconds, if set; tests set 0 to take
// this path) falls back to a device synchronisation (which reports a failed device)
// before giving up.
int wait_slot(StagingSlot& s) {
  auto done = [&] {
    for (uint32_t b = 0; b < s.nblocks; ++b)
      if (__atomic_load_n(s.flags + b, __ATOMIC_ACQUIRE) != s.seq) return false;
    return true;
  };
  if (done()) {
    s.pending = false;
    return TIDE_OK;
  }
  const char* env = getenv("TIDE_STAGING_WAIT_US");
  const long long limit_us = env ? atoll(env) : 5000000LL;
  const auto t0 = std::chrono::steady_clock::now();
  while (!done()) {
    if (std::chrono::steady_clock::now() - t0 >= std::chrono::microseconds(limit_us)) {
      if (hipDeviceSynchronize() != hipSuccess || !done()) return TIDE_ERR_HIP;
      break;
    }
    sched_yield();
  }
  s.pending = false;
  return TIDE_OK;
}

struct DeviceStaging {
  StagingSlot slots[kStagingSlots];
  int next = 0;
};

std::mutex g_mutex;
std::vector<DeviceStaging*> g_staging;  // indexed by device ordinal

// Device scratch of tide_decode_attn_noalloc: the work list and split partials of one
// call, for callers that cannot allocate.  In host code `scratch` names a host-side
// stand-in, never the device array: the device address is taken once per device with
// hipGetSymbolAddress (with that device current) and only that address is used.
static __device__ __align__(256) uint8_t scratch[TIDE_NOALLOC_SCRATCH_BYTES];

std::mutex g_scratch_mutex;
std::vector<void*> g_scratch_ptr;  // device address of `scratch`, indexed by device ordinal

int scratch_address(void** out) {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0) return TIDE_ERR_HIP;
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if ((int)g_scratch_ptr.size() <= dev) g_scratch_ptr.resize(dev + 1, nullptr);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return TIDE_ERR_HIP;
    g_scratch_ptr[dev] = p;
  }
  *out = g_scratch_ptr[dev];
  return TIDE_OK;
}

bool debug_checks() {
  const char* e = getenv("TIDE_DEBUG_CHECKS");
  return e && e[0] == '1';
}

// Where a call's kernel finds its plan.
struct Staged {
  const uint8_t* plan = nullptr;  // the workspace, or a staging slot
  PlanReads reads = {nullptr, 0};
  StagingSlot* slot = nullptr;    // set with reads.done
  // the ring's, held with a slot until its reader is launched: until then another call that
  // came round to the slot would wait for flags that no kernel is there to set
  std::unique_lock<std::mutex> lock;
};

// A plan that at most this many workgroups read, once each, is read where it was staged: a
// record costs each a read of host memory (about 2 us), which is less than the copy kernel,
// its launch and the gap behind it (3-5 us on the GPU and 3 on the host): a four-task decode
// step went from 16.0 to 13.5 us, the smallest append + extend from 31 to 25.  Each workgroup
// pays for its own read, so the gain ends where an extend's workgroups come in rounds of the
// CUs: copied and in place, us a call (28 / 4 heads, d = 128), extends of 64 workgroups 18.5 and
// 16.5, 256 23.5 and 20.9, 512 38.3 and 38.9, 1,024 69.5 and 79, 2,000 134 and 145; appends of 512
// 20.8 and 18.3, 1,024 21.4 and 18.4; decodes (up to 256 workgroups at 4 kv heads) 2 us less.
constexpr uint32_t kInPlaceGroups = 512;
static_assert(kStagingMin / kCopyBytesPerBlock >= kInPlaceGroups, "every slot has a flag for each");

bool capturing(hipStream_t stream) {
  hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(stream, &st) != hipSuccess) {
    (void)hipGetLastError();
    return true;
  }
  return st != hipStreamCaptureStatusNone;
}

// Stages the plan.  readers: the workgroups of the one kernel that reads it, if it may be read
// in place (0: not).  Under debug checks the kernel needs the zeroed header, which keeps the
// copy into the workspace; under capture no staging slot is used.
int upload(const Plan& plan, void* workspace, hipStream_t stream, uint32_t readers, Staged* out) {
  if (capturing(stream)) {
    out->plan = static_cast<const uint8_t*>(workspace);
    return put_plan(plan, workspace, stream);
  }
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0) return TIDE_ERR_HIP;
  std::unique_lock<std::mutex> lock(g_mutex);
  if ((int)g_staging.size() <= dev) g_staging.resize(dev + 1, nullptr);
  if (!g_staging[dev]) g_staging[dev] = new DeviceStaging();
  DeviceStaging& ds = *g_staging[dev];
  StagingSlot& s = ds.slots[ds.next];
  ds.next = (ds.next + 1) % kStagingSlots;
  if (s.pending) {
    const int rc = wait_slot(s);
    if (rc != TIDE_OK) return rc;
  }
  const size_t need = plan.blob.size();  // a multiple of kWsAlign
  if (s.cap < need) {
    if (s.host) (void)hipHostFree(s.host);
    if (s.flags) (void)hipHostFree(s.flags);
    s = StagingSlot();
    size_t cap = kStagingMin;
    while (cap < need) cap *= 2;
    const size_t nflags = cap / kCopyBytesPerBlock + 1;
    void* dev_ptr = nullptr;
    void* flags_dev = nullptr;
    if (hipHostMalloc(&s.host, cap, hipHostMallocMapped | hipHostMallocCoherent) != hipSuccess ||
        hipHostGetDevicePointer(&dev_ptr, s.host, 0) != hipSuccess ||
        hipHostMalloc(reinterpret_cast<void**>(&s.flags), nflags * sizeof(uint32_t),
                      hipHostMallocMapped | hipHostMallocCoherent) != hipSuccess ||
        hipHostGetDevicePointer(&flags_dev, s.flags, 0) != hipSuccess) {
      if (s.host) (void)hipHostFree(s.host);
      if (s.flags) (void)hipHostFree(s.flags);
      s = StagingSlot();
      return TIDE_ERR_HIP;
    }
    memset(s.flags, 0, nflags * sizeof(uint32_t));
    s.dev = dev_ptr;
    s.flags_dev = static_cast<uint32_t*>(flags_dev);
    s.cap = cap;
  }
  s.seq = s.seq + 1 == 0 ? 1 : s.seq + 1;  // never 0, the flags' initial value
  if (readers > 0 && readers <= kInPlaceGroups && !debug_checks()) {
    // (the flags a decode plan ends with need no zeros)
    memcpy(s.host, plan.blob.data(), plan.stream ? plan.tickets_off : need);
    s.nblocks = readers;
    s.pending = true;
    out->plan = static_cast<const uint8_t*>(s.dev);
    out->reads = PlanReads{s.flags_dev, s.seq};
    out->slot = &s;
    out->lock = std::move(lock);
    return TIDE_OK;
  }
  memcpy(s.host, plan.blob.data(), need);
  const size_t n16 = need / 16;
  const uint32_t nblocks = (uint32_t)((n16 + 255) / 256);
  hipLaunchKernelGGL(stage_copy_kernel, dim3(nblocks), dim3(256), 0, stream,
                     static_cast<u32x4_t*>(workspace), static_cast<const u32x4_t*>(s.dev), n16,
                     s.flags_dev, s.seq);
  if (hipGetLastError() != hipSuccess) return TIDE_ERR_HIP;
  s.nblocks = nblocks;
  s.pending = true;
  out->plan = static_cast<const uint8_t*>(workspace);
  return TIDE_OK;
}

int finish(hipError_t launch_status, Staged& st, void* workspace, hipStream_t stream) {
  if (st.slot && launch_status != hipSuccess) st.slot->pending = false;  // nothing will read it
  if (st.lock.owns_lock()) st.lock.unlock();
  if (launch_status != hipSuccess) return TIDE_ERR_HIP;
  if (!debug_checks()) return TIDE_OK;
  if (hipStreamSynchronize(stream) != hipSuccess) return TIDE_ERR_HIP;
  int32_t flags = 0;
  if (hipMemcpy(&flags, workspace, sizeof(flags), hipMemcpyDeviceToHost) != hipSuccess)
    return TIDE_ERR_HIP;
  return (flags & 1) ? TIDE_ERR_PAGE_RANGE : TIDE_OK;
}

template <class T>
const T* at(const void* ws, size_t off) {
  return reinterpret_cast<const T*>(static_cast<const uint8_t*>(ws) + off);
}

template <class T>
T* at_mut(void* ws, size_t off) {
  return reinterpret_cast<T*>(static_cast<uint8_t*>(ws) + off);
}

// A number no other call of the process has, and no chance contents of a workspace: the count
// starts at a random 64-bit number.
uint64_t next_call() {
  static std::atomic<uint64_t> count([] {
    std::random_device r;
    return ((uint64_t)r() << 32) ^ r();
  }());
  uint64_t c;
  do c = count.fetch_add(1, std::memory_order_relaxed);
  while (c == 0);  // what a copied plan zeroes the flags to
  return c;
}

// Shared path of tide_extend_attn and tide_full_prefill_attn.
// With k_new / v_new (tide_extend_append_attn) the new tokens' K/V are appended by the
// attention kernel itself.
int run_extend(int op, const void* q, const void* k_pool, const void* v_pool, int64_t num_pages,
               const int32_t* block_table, int32_t bt_stride, int32_t num_tasks,
               const int32_t* lens_a, const int32_t* lens_b, const tide_dims* dims, void* out,
               float* lse, void* workspace, size_t workspace_bytes, void* stream,
               const void* k_new = nullptr, const void* v_new = nullptr, bool fused = false) {
  int rc = check_dims(dims);
  if (rc != TIDE_OK) return rc;
  if (num_tasks < 0) return TIDE_ERR_INVALID_ARG;
  if (num_tasks == 0) return TIDE_OK;
  if (num_pages <= 0 || bt_stride <= 0) return TIDE_ERR_INVALID_ARG;
  Plan plan;
  rc = make_plan(op, num_tasks, lens_a, lens_b, *dims, 0, bt_stride, true, &plan);
  if (rc != TIDE_OK) return rc;
  if (plan.num_items == 0) return TIDE_OK;
  if (!q || !k_pool || !v_pool || !block_table || !out || !workspace) return TIDE_ERR_INVALID_ARG;
  if (fused && (!k_new || !v_new)) return TIDE_ERR_INVALID_ARG;
  if (workspace_bytes < plan.total_bytes) return TIDE_ERR_CAPACITY;
  hipStream_t s = static_cast<hipStream_t>(stream);
  Staged st;
  rc = upload(plan, workspace, s, plan.split ? 0 : (uint32_t)plan.num_items, &st);
  if (rc != TIDE_OK) return rc;
  ExtendArgs a;
  a.reads = st.reads;
  a.k_new = fused ? static_cast<const uint16_t*>(k_new) : nullptr;
  a.v_new = fused ? static_cast<const uint16_t*>(v_new) : nullptr;
  a.q = static_cast<const uint16_t*>(q);
  a.k_pool = static_cast<const uint16_t*>(k_pool);
  a.v_pool = static_cast<const uint16_t*>(v_pool);
  a.block_table = block_table;
  a.num_pages = num_pages;
  a.bt_stride = bt_stride;
  a.num_q_heads = dims->num_q_heads;
  a.num_kv_heads = dims->num_kv_heads;
  a.group = dims->num_q_heads / dims->num_kv_heads;
  a.scale_log2 = dims->sm_scale * 1.44269504088896340736f;
  a.num_items = plan.num_items;
  a.tasks = at<TaskDesc>(st.plan, plan.tasks_off);
  a.items = plan.split ? nullptr : at<ExtendItem>(st.plan, plan.items_off);
  a.out = static_cast<uint16_t*>(out);
  a.lse = lse;
  a.error_flags = at_mut<int32_t>(workspace, 0);
  a.chunk_items = plan.split ? at<ExtendChunkItem>(workspace, plan.items_off) : nullptr;
  a.merge_rows = plan.split ? at<MergeRow>(workspace, plan.merge_rows_off) : nullptr;
  a.part_o = plan.split ? at_mut<float>(workspace, plan.part_o_off) : nullptr;
  a.part_ml = plan.split ? at_mut<float>(workspace, plan.part_ml_off) : nullptr;
  a.total_rows = plan.total_rows;
  return finish(launch_extend(a, dims->head_dim, plan.waves, s), st, workspace, s);
}

// Shared path of tide_decode_attn, tide_decode_append_attn (fused: k_new / v_new) and
// tide_decode_attn_noalloc (in_scratch: the call runs in the static device scratch, its
// work list is copied there with hipMemcpyAsync from the plan's host buffer, or put there by
// kernels under capture, and nothing is allocated).
int run_decode(const void* q, const void* k_new, const void* v_new, const void* k_pool,
               const void* v_pool, int64_t num_pages, const int32_t* block_table,
               int32_t bt_stride, int32_t num_tasks, const int32_t* kv_lens,
               const tide_dims* dims, int32_t num_splits, void* out, float* lse,
               void* workspace, size_t workspace_bytes, bool fused, bool in_scratch,
               void* stream) {
  int rc = check_dims(dims);
  if (rc != TIDE_OK) return rc;
  if (num_tasks < 0 || num_splits < 0) return TIDE_ERR_INVALID_ARG;
  if (num_tasks == 0) return TIDE_OK;
  if (num_pages <= 0 || bt_stride <= 0) return TIDE_ERR_INVALID_ARG;
  Plan plan;
  rc = make_plan_decode(num_tasks, kv_lens, *dims, num_splits, bt_stride, true, &plan);
  if (rc != TIDE_OK) return rc;
  if (!q || !k_pool || !v_pool || !block_table || !out) return TIDE_ERR_INVALID_ARG;
  if (fused && (!k_new || !v_new)) return TIDE_ERR_INVALID_ARG;
  hipStream_t s = static_cast<hipStream_t>(stream);
  Staged st;
  if (in_scratch) {
    if (plan.total_bytes > (size_t)TIDE_NOALLOC_SCRATCH_BYTES) return TIDE_ERR_CAPACITY;
    rc = scratch_address(&workspace);
    if (rc != TIDE_OK) return rc;
    // the blob starts with the zeroed header, so this also clears the error flags; a captured
    // copy would read the plan's host buffer at every replay, long after it is freed.  A copy
    // from pageable memory takes 9 us up to 16 KB and 18 beyond, so the runs go as 4 bytes each
    // (64 tasks of 2,000 keys, 8 / 2 heads, d = 64: 22 KB and 33 us a call, now 5 KB and 19.5;
    // as chunks 24), and the flags not at all.
    const size_t bytes = plan.stream ? compact_runs(&plan) : plan.blob.size();
    if (capturing(s)) {
      rc = put_plan(plan, workspace, s);
      if (rc != TIDE_OK) return rc;
    } else if (hipMemcpyAsync(workspace, plan.blob.data(), bytes, hipMemcpyHostToDevice, s) !=
               hipSuccess) {
      return TIDE_ERR_HIP;
    }
    st.plan = static_cast<const uint8_t*>(workspace);
  } else {
    if (!workspace) return TIDE_ERR_INVALID_ARG;
    if (workspace_bytes < plan.total_bytes) return TIDE_ERR_CAPACITY;
    // a wave reads the task table again where its run crosses into the next task, so a call
    // with more tasks than runs keeps the copy
    const uint32_t readers = plan.stream && num_tasks <= plan.num_runs
                                 ? stream_groups(plan.num_runs, dims->num_kv_heads)
                                 : 0;
    rc = upload(plan, workspace, s, readers, &st);
    if (rc != TIDE_OK) return rc;
  }
  if (plan.stream) {
    StreamArgs a;
    a.q = static_cast<const uint16_t*>(q);
    a.k_pool = static_cast<const uint16_t*>(k_pool);
    a.v_pool = static_cast<const uint16_t*>(v_pool);
    a.block_table = block_table;
    a.num_pages = num_pages;
    a.bt_stride = bt_stride;
    a.num_q_heads = dims->num_q_heads;
    a.num_kv_heads = dims->num_kv_heads;
    a.group = dims->num_q_heads / dims->num_kv_heads;
    a.scale_log2 = dims->sm_scale * 1.44269504088896340736f;
    a.num_runs = plan.num_runs;
    a.num_tasks = num_tasks;
    a.steps = plan.steps;
    a.last_steps = plan.last_steps;
    a.tasks = at<TaskDesc>(st.plan, plan.tasks_off);
    a.items = at<StreamItem>(st.plan, plan.items_off);
    a.item_bytes = in_scratch ? sizeof(int32_t) : sizeof(StreamItem);
    a.reads = st.reads;
    a.part_o = at_mut<float>(workspace, plan.part_o_off);
    a.part_ml = at_mut<float>(workspace, plan.part_ml_off);
    a.flags = at_mut<uint64_t>(workspace, plan.tickets_off);
    a.call = next_call();
    a.out = static_cast<uint16_t*>(out);
    a.lse = lse;
    a.error_flags = at_mut<int32_t>(workspace, 0);
    a.k_new = static_cast<const uint16_t*>(k_new);
    a.v_new = static_cast<const uint16_t*>(v_new);
    return finish(launch_decode_stream(a, dims->head_dim, s), st, workspace, s);
  }
  DecodeArgs a;
  a.q = static_cast<const uint16_t*>(q);
  a.k_pool = static_cast<const uint16_t*>(k_pool);
  a.v_pool = static_cast<const uint16_t*>(v_pool);
  a.block_table = block_table;
  a.num_pages = num_pages;
  a.bt_stride = bt_stride;
  a.num_q_heads = dims->num_q_heads;
  a.num_kv_heads = dims->num_kv_heads;
  a.group = dims->num_q_heads / dims->num_kv_heads;
  a.scale_log2 = dims->sm_scale * 1.44269504088896340736f;
  a.num_tasks = num_tasks;
  a.num_items = plan.num_items;
  a.chunk = plan.chunk;
  a.max_splits = plan.max_splits;
  a.tasks = at<TaskDesc>(workspace, plan.tasks_off);
  a.items = at<DecodeItem>(workspace, plan.items_off);
  a.part_o = at_mut<float>(workspace, plan.part_o_off);
  a.part_ml = at_mut<float>(workspace, plan.part_ml_off);
  a.out = static_cast<uint16_t*>(out);
  a.lse = lse;
  a.error_flags = at_mut<int32_t>(workspace, 0);
  a.k_new = static_cast<const uint16_t*>(k_new);
  a.v_new = static_cast<const uint16_t*>(v_new);
  a.tickets = plan.fold_merge ? at_mut<int32_t>(workspace, plan.tickets_off) : nullptr;
  return finish(launch_decode(a, dims->head_dim, false, s), st, workspace, s);
}

}  // namespace
}  // namespace tide

using namespace tide;

extern "C" {

TIDE_API int tide_workspace_size(int op, int32_t num_tasks, const int32_t* lens_a,
                                 const int32_t* lens_b, const tide_dims* dims,
                                 int32_t num_splits, size_t* bytes_out) {
  try {
    if (!bytes_out) return TIDE_ERR_INVALID_ARG;
    int rc = check_dims(dims);
    if (rc != TIDE_OK) return rc;
    Plan plan;
    rc = op == TIDE_OP_DECODE
             ? make_plan_decode(num_tasks, lens_a, *dims, num_splits, -1, false, &plan)
             : make_plan(op, num_tasks, lens_a, lens_b, *dims, num_splits, -1, false, &plan);
    if (rc != TIDE_OK) return rc;
    *bytes_out = plan.total_bytes;
    return TIDE_OK;
  } catch (...) {
    return TIDE_ERR_HIP;
  }
}

TIDE_API int tide_plan_info_get(int op, int32_t num_tasks, const int32_t* lens_a,
                               const int32_t* lens_b, const tide_dims* dims, int32_t num_splits,
                               tide_plan_info* out) {
  try {
    if (!out) return TIDE_ERR_INVALID_ARG;
    int rc = check_dims(dims);
    if (rc != TIDE_OK) return rc;
    Plan plan;
    rc = op == TIDE_OP_DECODE
             ? make_plan_decode(num_tasks, lens_a, *dims, num_splits, -1, false, &plan)
             : make_plan(op, num_tasks, lens_a, lens_b, *dims, num_splits, -1, false, &plan);
    if (rc != TIDE_OK) return rc;
    *out = tide_plan_info{};
    out->num_items = plan.num_items;
    out->workspace_bytes = plan.total_bytes;
    if (op == TIDE_OP_DECODE) {
      out->waves_per_group =
          plan.stream ? stream_waves(plan.num_items) : decode_waves(plan.num_items);
      out->max_splits = plan.max_splits;
      out->merge_in_kernel = plan.fold_merge ? 1 : 0;
      out->run_steps = plan.steps;
    } else if (op == TIDE_OP_KV_APPEND) {
      out->waves_per_group = append_waves();
    } else {
      out->waves_per_group = plan.waves;
      out->split = plan.split ? 1 : 0;
    }
    return TIDE_OK;
  } catch (...) {
    return TIDE_ERR_HIP;
  }
}

TIDE_API int tide_kv_append(const void* k_new, const void* v_new, void* k_pool, void* v_pool,
                            int64_t num_pages, const int32_t* block_table, int32_t bt_stride,
                            int32_t num_tasks, const int32_t* prefix_lens,
                            const int32_t* extend_lens, const tide_dims* dims, void* workspace,
                            size_t workspace_bytes, void* stream) {
  try {
    int rc = check_dims(dims);
    if (rc != TIDE_OK) return rc;
    if (num_tasks < 0) return TIDE_ERR_INVALID_ARG;
    if (num_tasks == 0) return TIDE_OK;
    if (num_pages <= 0 || bt_stride <= 0) return TIDE_ERR_INVALID_ARG;
    Plan plan;
    rc = make_plan(TIDE_OP_KV_APPEND, num_tasks, prefix_lens, extend_lens, *dims, 0, bt_stride,
                   true, &plan);
    if (rc != TIDE_OK) return rc;
    if (plan.num_items == 0) return TIDE_OK;
    if (!k_new || !v_new || !k_pool || !v_pool || !block_table || !workspace)
      return TIDE_ERR_INVALID_ARG;
    if (workspace_bytes < plan.total_bytes) return TIDE_ERR_CAPACITY;
    hipStream_t s = static_cast<hipStream_t>(stream);
    Staged st;
    const int64_t groups = (int64_t)plan.num_items * append_groups(dims->num_kv_heads);
    rc = upload(plan, workspace, s, groups <= kInPlaceGroups ? (uint32_t)groups : 0, &st);
    if (rc != TIDE_OK) return rc;
    AppendArgs a;
    a.reads = st.reads;
    a.k_new = static_cast<const uint16_t*>(k_new);
    a.v_new = static_cast<const uint16_t*>(v_new);
    a.k_pool = static_cast<uint16_t*>(k_pool);
    a.v_pool = static_cast<uint16_t*>(v_pool);
    a.block_table = block_table;
    a.num_pages = num_pages;
    a.bt_stride = bt_stride;
    a.num_kv_heads = dims->num_kv_heads;
    a.head_dim = dims->head_dim;
    a.num_items = plan.num_items;
    a.tasks = at<TaskDesc>(st.plan, plan.tasks_off);
    a.items = at<AppendItem>(st.plan, plan.items_off);
    a.error_flags = at_mut<int32_t>(workspace, 0);
    return finish(launch_kv_append(a, s), st, workspace, s);
  } catch (...) {
    return TIDE_ERR_HIP;
  }
}

TIDE_API int tide_extend_attn(const void* q, const void* k_pool, const void* v_pool,
                              int64_t num_pages, const int32_t* block_table, int32_t bt_stride,
                              int32_t num_tasks, const int32_t* prefix_lens,
                              const int32_t* extend_lens, const tide_dims* dims, void* out,
                              float* lse, void* workspace, size_t workspace_bytes, void* stream) {
  try {
    return run_extend(TIDE_OP_EXTEND, q, k_pool, v_pool, num_pages, block_table, bt_stride,
                      num_tasks, prefix_lens, extend_lens, dims, out, lse, workspace,
                      workspace_bytes, stream);
  } catch (...) {
    return TIDE_ERR_HIP;
  }
}

TIDE_API int tide_extend_append_attn(const void* q, const void* k_new, const void* v_new,
                                     void* k_pool, void* v_pool, int64_t num_pages,
                                     const int32_t* block_table, int32_t bt_stride,
                                     int32_t num_tasks, const int32_t* prefix_lens,
                                     const int32_t* extend_lens, const tide_dims* dims, void* out,
                                     float* lse, void* workspace, size_t workspace_bytes,
                                     void* stream) {
  try {
    return run_extend(TIDE_OP_EXTEND, q, k_pool, v_pool, num_pages, block_table, bt_stride,
                      num_tasks, prefix_lens, extend_lens, dims, out, lse, workspace,
                      workspace_bytes, stream, k_new, v_new, true);
  } catch (...) {
    return TIDE_ERR_HIP;
  }
}

TIDE_API int tide_full_prefill_attn(const void* q, const void* k_pool, const void* v_pool,
                                    int64_t num_pages, const int32_t* block_table,
                                    int32_t bt_stride, int32_t num_tasks, const int32_t* seq_lens,
                                    const tide_dims* dims, void* out, float* lse,
                                    void* workspace, size_t workspace_bytes, void* stream) {
  try {
    return run_extend(TIDE_OP_FULL_PREFILL, q, k_pool, v_pool, num_pages, block_table,
                      bt_stride, num_tasks, seq_lens, nullptr, dims, out, lse, workspace,
                      workspace_bytes, stream);
  } catch (...) {
    return TIDE_ERR_HIP;
  }
}

TIDE_API int tide_decode_attn(const void* q, const void* k_pool, const void* v_pool,
                              int64_t num_pages, const int32_t* block_table, int32_t bt_stride,
                              int32_t num_tasks, const int32_t* kv_lens, const tide_dims* dims,
                              int32_t num_splits, void* out, float* lse, void* workspace,
                              size_t workspace_bytes, void* stream) {
  try {
    return run_decode(q, nullptr, nullptr, k_pool, v_pool, num_pages, block_table, bt_stride,
                      num_tasks, kv_lens, dims, num_splits, out, lse, workspace, workspace_bytes,
                      false, false, stream);
  } catch (...) {
    return TIDE_ERR_HIP;
  }
}

TIDE_API int tide_decode_append_attn(const void* q, const void* k_new, const void* v_new,
                                     void* k_pool, void* v_pool, int64_t num_pages,
                                     const int32_t* block_table, int32_t bt_stride,
                                     int32_t num_tasks, const int32_t* kv_lens,
                                     const tide_dims* dims, int32_t num_splits, void* out,
                                     float* lse, void* workspace, size_t workspace_bytes,
                                     void* stream) {
  try {
    return run_decode(q, k_new, v_new, k_pool, v_pool, num_pages, block_table, bt_stride,
                      num_tasks, kv_lens, dims, num_splits, out, lse, workspace, workspace_bytes,
                      true, false, stream);
  } catch (...) {
    return TIDE_ERR_HIP;
  }
}

TIDE_API int tide_decode_attn_noalloc(const void* q, const void* k_pool, const void* v_pool,
                                      int64_t num_pages, const int32_t* block_table,
                                      int32_t bt_stride, int32_t num_tasks,
                                      const int32_t* kv_lens, const tide_dims* dims,
                                      int32_t num_splits, void* out, float* lse, void* stream) {
  try {
    return run_decode(q, nullptr, nullptr, k_pool, v_pool, num_pages, block_table, bt_stride,
                      num_tasks, kv_lens, dims, num_splits, out, lse, nullptr, 0, false, true,
                      stream);
  } catch (...) {
    return TIDE_ERR_HIP;
  }
}

TIDE_API int tide_workspace_size_shared(int32_t num_tasks, const int32_t* kv_lens,
                                        int32_t num_groups, const int32_t* group_start,
                                        const int32_t* shared_lens, const tide_dims* dims,
                                        int32_t num_splits, size_t* bytes_out) {
  try {
    if (!bytes_out) return TIDE_ERR_INVALID_ARG;
    int rc = check_dims(dims);
    if (rc != TIDE_OK) return rc;
    Plan plan;
    rc = make_plan_shared(num_tasks, kv_lens, num_groups, group_start, shared_lens, *dims,
                          num_splits, -1, false, &plan);
    if (rc != TIDE_OK) return rc;
    *bytes_out = plan.total_bytes;
    return TIDE_OK;
  } catch (...) {
    return TIDE_ERR_HIP;
  }
}

TIDE_API int tide_decode_attn_shared(const void* q, const void* k_pool, const void* v_pool,
                                     int64_t num_pages, const int32_t* block_table,
                                     int32_t bt_stride, int32_t num_tasks, const int32_t* kv_lens,
                                     int32_t num_groups, const int32_t* group_start,
                                     const int32_t* shared_lens, const tide_dims* dims,
                                     int32_t num_splits, void* out, float* lse, void* workspace,
                                     size_t workspace_bytes, void* stream) {
  try {
    int rc = check_dims(dims);
    if (rc != TIDE_OK) return rc;
    if (num_tasks < 0 || num_splits < 0) return TIDE_ERR_INVALID_ARG;
    if (num_tasks == 0) return TIDE_OK;
    if (num_pages <= 0 || bt_stride <= 0) return TIDE_ERR_INVALID_ARG;
    Plan plan;
    rc = make_plan_shared(num_tasks, kv_lens, num_groups, group_start, shared_lens, *dims,
                          num_splits, bt_stride, true, &plan);
    if (rc != TIDE_OK) return rc;
    if (!q || !k_pool || !v_pool || !block_table || !out || !workspace)
      return TIDE_ERR_INVALID_ARG;
    if (workspace_bytes < plan.total_bytes) return TIDE_ERR_CAPACITY;
    hipStream_t s = static_cast<hipStream_t>(stream);
    Staged st;
    rc = upload(plan, workspace, s, 0, &st);
    if (rc != TIDE_OK) return rc;
    DecodeArgs a;
    a.q = static_cast<const uint16_t*>(q);
    a.k_pool = static_cast<const uint16_t*>(k_pool);
    a.v_pool = static_cast<const uint16_t*>(v_pool);
    a.block_table = block_table;
    a.num_pages = num_pages;
    a.bt_stride = bt_stride;
    a.num_q_heads = dims->num_q_heads;
    a.num_kv_heads = dims->num_kv_heads;
    a.group = dims->num_q_heads / dims->num_kv_heads;
    a.scale_log2 = dims->sm_scale * 1.44269504088896340736f;
    a.num_tasks = num_tasks;
    a.num_items = plan.num_items;
    a.chunk = plan.chunk;
    a.max_splits = plan.max_splits;
    a.tasks = at<TaskDesc>(workspace, plan.tasks_off);
    a.items = at<SharedDecodeItem>(workspace, plan.items_off);
    a.part_o = at_mut<float>(workspace, plan.part_o_off);
    a.part_ml = at_mut<float>(workspace, plan.part_ml_off);
    a.out = static_cast<uint16_t*>(out);
    a.lse = lse;
    a.error_flags = at_mut<int32_t>(workspace, 0);
    a.k_new = nullptr;
    a.v_new = nullptr;
    a.tickets = nullptr;
    return finish(launch_decode(a, dims->head_dim, true, s), st, workspace, s);
  } catch (...) {
    return TIDE_ERR_HIP;
  }
}

TIDE_API const char* tide_status_string(int status) {
  switch (status) {
    case TIDE_OK: return "ok";
    case TIDE_ERR_INVALID_ARG: return "invalid argument";
    case TIDE_ERR_UNSUPPORTED: return "unsupported shape";
    case TIDE_ERR_CAPACITY: return "capacity exceeded (block table or workspace too small)";
    case TIDE_ERR_HIP: return "HIP runtime error";
    case TIDE_ERR_PAGE_RANGE: return "block-table page id out of range";
    default: return "unknown status";
  }
}

TIDE_API void tide_shutdown(void) {
  std::lock_guard<std::mutex> lock(g_mutex);
  for (DeviceStaging* ds : g_staging) {
    if (!ds) continue;
    for (StagingSlot& s : ds->slots) {
      if (s.pending) (void)wait_slot(s);
      if (s.host) (void)hipHostFree(s.host);
      if (s.flags) (void)hipHostFree(s.flags);
    }
    delete ds;
  }
  g_staging.clear();
}

}  // extern "C"
