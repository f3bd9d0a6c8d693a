// Decode attention with the library's own split: equal runs of key steps per wave.
//
// Decode reads every K/V byte of the contexts once, so a call should take the time of that
// stream.  Cut into chunks of (task, kv head), a call of 1.3 or 2.5 rounds of waves leaves
// most of the chip idle in its last round, every chunk starts with an empty pipeline, and a
// context of many chunks needs a second kernel to merge them.  Here the tasks' 32-key steps
// are laid end to end and cut into equal runs, so many that runs x kv heads fill the device
// once (2048 waves, 8 per CU), and a wave takes one run of one kv head:
//   * every wave starts at once and ends at about the same time, and its loads never drain:
//     the next step is in flight while one is used, across the tasks of the run too;
//   * a task that begins and ends inside a run is finished by its wave.  A task cut by a
//     run's end leaves partials (o, m, l);
//   * the waves of a workgroup take consecutive runs, so the partials of a long context are
//     first combined in LDS, and only one per workgroup travels through memory.  Each part then
//     sets the flag of its slot to the call's own number, and a part that finds all flags of its
//     task set merges the parts, in key order; should two find them, both write the same rows
//     (`arrive`).  There is no merge kernel, and a call with fewer steps than waves runs one step
//     a wave.
// The step itself (K through LDS, V transposed in LDS, the G query heads as MFMA columns, the
// cache policy) is that of attn_decode.hip; the newest token of the fused append replaces its
// slot's row in the operands instead of being stored and waited for first.
// Measured against the chunks (MI355X, append fused, call us; 28 / 4 heads, d = 128): 8 tasks
// of 0.6k-3k keys 29.6 -> 24.6, 16 of 2k-16k 71.8 -> 53.3, 64 of 2k-16k 191 -> 183, 175 of
// 0.5k-3k 132 -> 106; 32 / 8 heads: 1024 of 64-512 keys 288 -> 218, 128 of 4k-14k 743 -> 690
// (6.7 TB/s).  All of the heads of one run in a workgroup instead of 8 runs of one head was
// slower everywhere (no partials to combine in LDS), and fewer or more waves than the device
// holds at once 2-50% slower.
#include "attn_decode.h"

namespace tide {
namespace kern {

constexpr int kStreamBig = 8, kStreamSmall = 4;  // waves per workgroup (stream_waves)

typedef const __attribute__((address_space(4))) StreamItem const_item;

// Rows of one unit being merged by a wave: lanes L j .. L j + L - 1 hold head j0 + j (64 / L
// heads a pass), each lane D / L consecutive head-dim entries.  With M the largest m seen, acc
// = sum 2^(m_s - M) o_s, l and lx the same sums of the bf16-rounded and the exact weights.
template <int D, int L>
struct RowMerge {
  static constexpr int kPer = D / L, kV = kPer / 4;
  f32x4 acc[kV];
  float mx, l, lx;
  __device__ __forceinline__ void clear() {
#pragma unroll
    for (int k = 0; k < kV; ++k) acc[k] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    mx = kNoMax;
    l = lx = 0.0f;
  }
  // makes `m` part of the running maximum
  __device__ __forceinline__ void raise(float m) {
    const float mn = fmaxf(mx, m), w = fast_exp2(mx - mn);
#pragma unroll
    for (int k = 0; k < kV; ++k) acc[k] *= w;
    l *= w;
    lx *= w;
    mx = mn;
  }
  // adds a part whose maximum is included in mx already
  __device__ __forceinline__ void add(f32x4 ml, const f32x4 (&o)[kV]) {
    const float w = fast_exp2(ml[0] - mx);
    l += w * ml[1];
    lx += w * ml[2];
#pragma unroll
    for (int k = 0; k < kV; ++k) acc[k] += w * o[k];
  }
};

template <int D, bool kAppend, int kWaves>
__global__ __launch_bounds__(kWaves * 64) __attribute__((amdgpu_waves_per_eu(2, 2)))
void decode_stream_kernel(StreamArgs a) {
  using KL = KLds<D>;
  using VL = VLds<D>;
  constexpr int kC = D / 32, kT = D / 16;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // a workgroup takes kWaves consecutive runs of one kv head (the heads of the same runs are
  // neighbours in dispatch order)
  const int R = a.num_runs, rg = blockIdx.x / a.num_kv_heads;
  const int head = blockIdx.x - rg * a.num_kv_heads;
  const int run = rg * kWaves + wave;
  // K pages of the two steps in flight, one region per wave (2 pages per step); at the end
  // the waves' partials: outputs in k_lds0, statistics in k_lds1
  __shared__ __attribute__((aligned(1024))) uint8_t k_lds0[kWaves * 2 * KL::kPageBytes];
  __shared__ __attribute__((aligned(1024))) uint8_t k_lds1[kWaves * 2 * KL::kPageBytes];
  __shared__ int open_task[kWaves];  // the task each wave leaves unfinished, or -1
  uint8_t* const ka = k_lds0 + wave * 2 * KL::kPageBytes;
  uint8_t* const kb = k_lds1 + wave * 2 * KL::kPageBytes;

  const bool live = run < R;
  const int at = live ? run : 0;
  const int n = !live ? 0 : run == R - 1 ? a.last_steps : a.steps;
  const StreamSlots slots = {R, a.num_tasks, kWaves};
  const int64_t slot0 = (int64_t)head * slots.count();  // this head's first partial slot
  const int G = a.group, Hkv = a.num_kv_heads;
  const int col = lane & 15, grp = lane >> 4;
  const bool col_ok = col < G;
  const uint8_t* kpool = reinterpret_cast<const uint8_t*>(a.k_pool);
  const uint8_t* vpool = reinterpret_cast<const uint8_t*>(a.v_pool);
  constexpr int64_t kBlk = (int64_t)kPage * D * 2;  // bytes of one (page, kv head) block

  uint32_t k_src[KL::kDma];
#pragma unroll
  for (int i = 0; i < KL::kDma; ++i) k_src[i] = KL::src_offset(i, lane);
  const uint32_t k_rd_even = KL::lds_offset(col, grp), k_rd_odd = KL::lds_offset(col, 4 + grp);
  const uint32_t v_off = (uint32_t)(16 * lane);
  constexpr int kRpl = 1024 / (2 * D);  // V rows per 1 KB load
  uint32_t v_wr[DecodeRegs<D>::kLoads];
#pragma unroll
  for (int i = 0; i < DecodeRegs<D>::kLoads; ++i)
    v_wr[i] = VL::offset(i * kRpl + lane / VL::kNG, lane % VL::kNG);
  const int gl = lane & 15, vr = 4 * grp + (gl >> 2);
  uint32_t v_rd[kT];
#pragma unroll
  for (int t = 0; t < kT; ++t)
    v_rd[t] = (uint32_t)(vr * 2 * D + 32 * (t ^ VL::vsw(vr)) + 8 * (gl & 3));

  // Position in the sequence of the tasks' steps; all wave-uniform.
  struct Cursor {
    int task, step, steps, kv_len;
  };
  auto steps_of = [](int kv_len) { return (kv_len + kDecodeStep - 1) / kDecodeStep; };
  auto next_unit = [&](Cursor& c, bool more) {  // more: there is one (it is not read otherwise)
    c.step = 0;
    ++c.task;
    if (more) {
      const const_i32* td = (const const_i32*)(a.tasks + c.task);
      c.kv_len = td[1] + td[2];  // prefix + extend
      c.steps = steps_of(c.kv_len);
    }
  };
  // (the record is loaded whole in either form: behind a branch on the form it cost 0.3 us)
  const const_item* it =
      (const const_item*)(reinterpret_cast<const uint8_t*>(a.items) + (int64_t)at * a.item_bytes);
  Cursor ld = {it->task, it->step, 0, it->kv_len};
  if (__builtin_expect(a.item_bytes != sizeof(StreamItem), 0)) {  // the task alone (compact_runs)
    const const_i32* td = (const const_i32*)(a.tasks + ld.task);
    ld.step = at * a.steps - td[3];
    ld.kv_len = td[1] + td[2];
  }
  ld.steps = steps_of(ld.kv_len);
  Cursor cu = ld;

  // Loads of the load cursor's step.  Every call issues the same loads: past the run's end
  // (and for pages past a context or with an invalid id) through zero-length buffers, which
  // return zeros without touching memory.  Page ids are scalar loads, fetched one step ahead.
  bool flag_error = false;
  int left = n;  // steps not issued yet
  int32_t pg[2];
  auto fetch_pages = [&]() {
    const const_i32* row = (const const_i32*)(a.block_table + (int64_t)(left > 0 ? ld.task : 0) * a.bt_stride);
    const int last = (ld.kv_len + kPage - 1) / kPage - 1;
    pg[0] = row[left > 0 ? 2 * ld.step : 0];
    pg[1] = row[left > 0 ? min(2 * ld.step + 1, last) : 0];
  };
  // the newest token's rows (kAppend), loaded with the step that holds its slot: lane l the K
  // granules 4 c + l / 16, and the V granule l % kNG
  struct NewRow {
    u32x4 k[kC], v;
    int page;  // its pool page, or -1
  };
  auto issue = [&](DecodeRegs<D>& r, uint8_t* kbuf, NewRow& nw) {
    const bool in = left > 0;
    const bool second = in && (2 * ld.step + 1) * kPage < ld.kv_len;
    const bool ok0 = in && pg[0] >= 0 && pg[0] < a.num_pages;
    const bool ok1 = second && pg[1] >= 0 && pg[1] < a.num_pages;
    flag_error |= (in && !ok0) || (second && !ok1);
    const int64_t b0 = ((int64_t)(ok0 ? pg[0] : 0) * Hkv + head) * kBlk;
    const int64_t b1 = ((int64_t)(ok1 ? pg[1] : 0) * Hkv + head) * kBlk;
    const int n0 = ok0 ? (int)kBlk : 0, n1 = ok1 ? (int)kBlk : 0;
    load_step<D, kStreamPolicy>(r, kbuf, block_rsrc(kpool + b0, n0), block_rsrc(kpool + b1, n1),
                                block_rsrc(vpool + b0, n0), block_rsrc(vpool + b1, n1), k_src, v_off);
    if constexpr (kAppend) {
      nw.page = -1;
      if (in && ld.step == ld.steps - 1) {
        const bool hi = ((ld.kv_len - 1) & (kDecodeStep - 1)) >= kPage;
        if (hi ? ok1 : ok0) {
          nw.page = hi ? pg[1] : pg[0];
          const int64_t row = ((int64_t)ld.task * Hkv + head) * D;
#pragma unroll
          for (int c = 0; c < kC; ++c) nw.k[c] = load_u32x4(a.k_new + row + 32 * c + 8 * grp);
          nw.v = load_u32x4(a.v_new + row + 8 * (lane % VL::kNG));
        }
      }
    }
    if (in) {
      --left;
      if (++ld.step == ld.steps) next_unit(ld, left > 0);
    }
    fetch_pages();
  };

  bf16x8 qf[kC];
  auto load_q = [&]() {
    const int64_t row = (int64_t)cu.task * a.num_q_heads + head * G + col;
#pragma unroll
    for (int c = 0; c < kC; ++c)
      qf[c] = as_bf16x8(col_ok ? load_u32x4(a.q + row * D + 32 * c + 8 * grp) : zero_u32x4());
  };
  f32x4 o[kT];
  float m_ref, l_part, l_exact;
  auto reset = [&]() {
#pragma unroll
    for (int t = 0; t < kT; ++t) o[t] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    m_ref = kNoMax;
    l_part = l_exact = 0.0f;
  };

  // One step of the compute cursor.  last: the task's last step, the only one that can hold
  // keys past the context and the newest token's slot.  Its changes to the operands are
  // branches around in-place updates; a second copy of the step would cost copies of every
  // accumulator where the two meet.
  auto compute = [&](DecodeRegs<D>& cur, const uint8_t* kbuf, NewRow& nw, bool last) {
    const int k = cu.step * kDecodeStep;
    u32x4 kk[2][kC];
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int c = 0; c < kC; ++c)
        kk[t][c] = *reinterpret_cast<const u32x4*>(kbuf + t * KL::kPageBytes + 1024 * (c >> 1) +
                                                   ((c & 1) ? k_rd_odd : k_rd_even));
    if (last) {
      if constexpr (kAppend) {
        // the newest token takes the place of its slot's row (whatever the pool holds there)
        // and goes to the pool; nothing in this call reads the slot afterwards
        if (nw.page >= 0) {
          const int slot = (cu.kv_len - 1) & (kPage - 1), half = ((cu.kv_len - 1) / kPage) & 1;
#pragma unroll
          for (int t = 0; t < 2; ++t) {
#pragma unroll
            for (int c = 0; c < kC; ++c)
              if (t == half && col == slot) kk[t][c] = nw.k[c];
#pragma unroll
            for (int i = 0; i < DecodeRegs<D>::kLoads; ++i)
              if (t == half && i * kRpl + lane / VL::kNG == slot) cur.v[t][i] = nw.v;
          }
          const int64_t at = (((int64_t)nw.page * Hkv + head) * kPage + slot) * D;
          if (col == slot) {
#pragma unroll
            for (int c = 0; c < kC; ++c)
              store_u32x4(const_cast<uint16_t*>(a.k_pool) + at + 32 * c + 8 * grp, nw.k[c]);
          }
          if (lane < VL::kNG) store_u32x4(const_cast<uint16_t*>(a.v_pool) + at + 8 * lane, nw.v);
        }
      }
      // V rows past the context must not reach the MFMA (NaN * 0 = NaN)
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int i = 0; i < DecodeRegs<D>::kLoads; ++i)
          if (k + 16 * t + i * kRpl + lane / VL::kNG >= cu.kv_len) cur.v[t][i] = zero_u32x4();
    }
    f32x4 s[2];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      s[t] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
      for (int c = 0; c < kC; ++c) s[t] = mfma16(as_bf16x8(kk[t][c]), qf[c], s[t]);
    }
    float mt = -INFINITY;
    const int keys = last ? cu.kv_len - k - 4 * grp : kDecodeStep;  // of this lane's, counted from its first
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float x = 16 * t + e < keys ? s[t][e] * a.scale_log2 : -INFINITY;
        s[t][e] = x;
        mt = fmaxf(mt, x);
      }
    mt = fmaxf(mt, xor_shfl(mt, 16));
    mt = fmaxf(mt, xor_shfl(mt, 32));
    if (__any(mt > m_ref + kRescaleSlack)) {
      const float m_new = fmaxf(m_ref, mt);
      const float alpha = fast_exp2(m_ref - m_new);
      l_part *= alpha;
      l_exact *= alpha;
#pragma unroll
      for (int t = 0; t < kT; ++t) o[t] *= alpha;
      m_ref = m_new;
    }
    u32x4 wp;
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        const float p0 = fast_exp2(s[t][2 * e] - m_ref);
        const float p1 = fast_exp2(s[t][2 * e + 1] - m_ref);
        wp[2 * t + e] = pack_bf16x2(p0, p1);
        l_part = add_bf16x2(wp[2 * t + e], l_part);
        l_exact += p0 + p1;
      }
    const bf16x8 pb = as_bf16x8(wp);
    uint8_t* vbuf = const_cast<uint8_t*>(kbuf);  // V over the K copy, which is done with
#pragma unroll
    for (int hp = 0; hp < 2; ++hp)
#pragma unroll
      for (int i = 0; i < DecodeRegs<D>::kLoads; ++i)
        *reinterpret_cast<u32x4*>(vbuf + hp * KL::kPageBytes + v_wr[i]) = cur.v[hp][i];
    u32x4 vv[kT];
#pragma unroll
    for (int t = 0; t < kT; ++t) {
      const uint2 v0 = read_tr(vbuf + v_rd[t]), v1 = read_tr(vbuf + KL::kPageBytes + v_rd[t]);
      vv[t] = u32x4{v0.x, v0.y, v1.x, v1.y};
    }
#pragma unroll
    for (int t = 0; t < kT; ++t) o[t] = mfma16(as_bf16x8(vv[t]), pb, o[t]);
  };

  auto sum_cols = [&](float v) {
    v += xor_shfl(v, 16);
    return v + xor_shfl(v, 32);
  };
  // Steps of the current unit before this wave; the unit that began earlier and ended here.
  int begin = cu.step;
  bool has_final = false, has_flush = false;
  StreamUnit flush = {0, 0, false};
  int done = 0;

  // The unit whose last step was just computed.
  auto unit_end = [&]() {
    if (begin == 0) {  // all of it in this wave: its rows are final
      const float inv = 1.0f / sum_cols(l_part), lx = sum_cols(l_exact);
      if (col_ok) {
        const int64_t row = (int64_t)cu.task * a.num_q_heads + head * G + col;
#pragma unroll
        for (int t = 0; t < kT; ++t) {
          const uint2 x = {pack_bf16x2(o[t][0] * inv, o[t][1] * inv),
                           pack_bf16x2(o[t][2] * inv, o[t][3] * inv)};
          *reinterpret_cast<uint2*>(a.out + row * D + 16 * t + 4 * grp) = x;
        }
        if (a.lse && grp == 0) a.lse[row] = (m_ref + __log2f(lx)) * kLn2;
      }
    } else if (cu.steps - begin == a.steps) {  // it took the whole run: like an unfinished one
      has_final = true;
      return;
    } else {
      has_flush = true;
      flush = stream_unit(run, begin, cu.steps - begin, cu.steps, a.steps);
      const float l = sum_cols(l_part), lx = sum_cols(l_exact);
      if (col_ok) {
        const int64_t slot = slot0 + slots.ended(run, cu.task);
        float* po = a.part_o + slot * G * D;
#pragma unroll
        for (int t = 0; t < kT; ++t)
          store_f32x4_device(po, G * D * 4, 4 * (col * D + 16 * t + 4 * grp), o[t]);
        if (grp == 0)
          store_f32x4_device(a.part_ml + slot * G * 4, G * 16, 16 * col,
                             f32x4{m_ref, l, lx, 0.0f});
      }
    }
    begin = 0;
    reset();
  };
  int flush_task = 0;
  auto process = [&](DecodeRegs<D>& r, const uint8_t* kbuf, NewRow& nw) {
    const bool last = cu.step == cu.steps - 1;
    compute(r, kbuf, nw, last);
    ++done;
    ++cu.step;
    if (last) {
      const bool was_flush = has_flush;
      unit_end();
      if (has_flush && !was_flush) flush_task = cu.task;
      if (!has_final) {
        next_unit(cu, done < n);
        if (done < n) load_q();
      }
    }
  };

  reset();
  fetch_pages();
  if (n > 0) {
    DecodeRegs<D> ra, rb;
    NewRow na, nb;
    load_q();
    // every load is issued on straight-line code (past the run's end, loads of nothing), so
    // a step's wait leaves the next step in flight; the scheduling barriers keep each
    // step's loads issued before the reads of the step before it
    issue(ra, ka, na);
    for (int i = 0;; i += 2) {
      issue(rb, kb, nb);
      __builtin_amdgcn_sched_barrier(0);
      process(ra, ka, na);
      if (i + 1 >= n) break;
      issue(ra, ka, na);
      __builtin_amdgcn_sched_barrier(0);
      process(rb, kb, nb);
      if (i + 2 >= n) break;
    }
    has_final |= cu.step > 0 && cu.step < cu.steps;
  }
  if (flag_error && lane == 0) atomicOr(a.error_flags, 1);

  // ---- parts of cut units: combined per workgroup, then across workgroups ----------------
  // All loads into LDS (the zero-length ones too) and the flushed partial's stores are done
  // before LDS takes the partials and before any arrival is counted.
  __atomic_signal_fence(__ATOMIC_SEQ_CST);
  __builtin_amdgcn_s_waitcnt(0);
  __atomic_signal_fence(__ATOMIC_SEQ_CST);
  // LDS row `col` of a wave's partial: 16-byte granule g at g ^ (col & 15)
  if (has_final) {
    const float l = sum_cols(l_part), lx = sum_cols(l_exact);
    if (col_ok) {
#pragma unroll
      for (int t = 0; t < kT; ++t)
        *reinterpret_cast<f32x4*>(ka + 4 * D * col + 16 * ((4 * t + grp) ^ col)) = o[t];
      if (grp == 0) *reinterpret_cast<f32x4*>(kb + 16 * col) = f32x4{m_ref, l, lx, 0.0f};
    }
  }
  if (lane == 0) open_task[wave] = has_final ? cu.task : -1;
  __syncthreads();
  if (a.reads.done && threadIdx.x == 0) plan_read(a.reads, blockIdx.x);

  // Merges every part of a task in key order and writes this head's rows.
  auto merge = [&](auto lanes_tag, const StreamUnit& u, int task) {
    constexpr int L = decltype(lanes_tag)::value;
    using RM = RowMerge<D, L>;
    constexpr int kB = 16 / RM::kV;  // parts loaded together
    const int sub = lane % L;
    const int np = stream_parts(u, kWaves);
    for (int j0 = 0; j0 < G; j0 += 64 / L) {
      const int j = j0 + lane / L;
      const bool ok = j < G;
      RM rm;
      rm.clear();
      for (int e0 = 0; e0 < np; e0 += kB) {
        f32x4 ml[kB], po[kB][RM::kV];
#pragma unroll
        for (int i = 0; i < kB; ++i) {
          const int e = e0 + i;
          const bool in = e < np;
          const int64_t slot = slot0 + stream_slot(u, slots, task, in ? e : 0);
          const auto rml = __builtin_amdgcn_make_buffer_rsrc(
              a.part_ml + slot * G * 4, 0, in ? G * 16 : 0, 0x00020000);
          const auto rpo = __builtin_amdgcn_make_buffer_rsrc(
              a.part_o + slot * G * D, 0, in ? G * D * 4 : 0, 0x00020000);
          ml[i] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rml, 16 * j, 0, kDeviceScope));
#pragma unroll
          for (int k = 0; k < RM::kV; ++k)
            po[i][k] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(
                                                     rpo, 4 * (j * D + RM::kPer * sub + 4 * k), 0, kDeviceScope));
        }
        float m = kNoMax;
#pragma unroll
        for (int i = 0; i < kB; ++i) {
          if (e0 + i >= np) ml[i][0] = kNoMax;
          m = fmaxf(m, ml[i][0]);
        }
        rm.raise(m);
#pragma unroll
        for (int i = 0; i < kB; ++i) rm.add(ml[i], po[i]);
      }
      if (ok) {
        const float inv = 1.0f / rm.l;
        const int64_t row = (int64_t)task * a.num_q_heads + head * G + j;
        uint16_t* orow = a.out + row * D + RM::kPer * sub;
#pragma unroll
        for (int k = 0; k < RM::kV; ++k) {
          const uint2 x = {pack_bf16x2(rm.acc[k][0] * inv, rm.acc[k][1] * inv),
                           pack_bf16x2(rm.acc[k][2] * inv, rm.acc[k][3] * inv)};
          *reinterpret_cast<uint2*>(orow + 4 * k) = x;
        }
        if (a.lse && sub == 0) a.lse[row] = (rm.mx + __log2f(rm.lx)) * kLn2;
      }
    }
  };
  // Flags the part in `slot` complete; a part that then finds all of the task's flags set merges.
  // Each flag is written (device scope, acknowledged) after the part's own stores and before
  // it looks, so the part whose flag lands last finds them all; should two find them, both
  // write the same rows.  Unlike a counter, the flags need no zeros to start from.
  auto arrive = [&](const StreamUnit& u, int task, int64_t slot) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    if (lane == 0)
      __hip_atomic_store(a.flags + slot, a.call, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    const int np = stream_parts(u, kWaves);
    for (int e = lane; e - lane < np; e += 64) {
      const int64_t other = slot0 + stream_slot(u, slots, task, min(e, np - 1));
      if (__any(__hip_atomic_load(a.flags + other, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != a.call))
        return;
    }
    asm volatile("" ::: "memory");
    if (G > 4) merge(std::integral_constant<int, 8>(), u, task);
    else merge(std::integral_constant<int, 16>(), u, task);
  };

  if (has_flush) arrive(flush, flush_task, slot0 + slots.ended(run, flush_task));
  if (!has_final) return;
  auto left_open = [&](int x) { return __builtin_amdgcn_readfirstlane(open_task[x]); };
  if (wave > 0 && left_open(wave - 1) == cu.task) return;  // the first of these waves goes on
  int len = 1;
  while (wave + len < kWaves && left_open(wave + len) == cu.task) ++len;
  const StreamUnit u = stream_unit(run, begin, cu.step - begin, cu.steps, a.steps);
  const bool whole = !u.ends_inside && u.n == len;  // the unit lies inside this workgroup
  auto combine = [&](auto lanes_tag) {
    constexpr int L = decltype(lanes_tag)::value;
    using RM = RowMerge<D, L>;
    const int sub = lane % L;
    for (int j0 = 0; j0 < G; j0 += 64 / L) {
      const int j = j0 + lane / L;
      const int jr = j < G ? j : 0;
      RM rm;
      rm.clear();
      for (int x = 0; x < len; ++x) {
        const uint8_t* xo = k_lds0 + (wave + x) * 2 * KL::kPageBytes + 4 * D * jr;
        const f32x4 ml = *reinterpret_cast<const f32x4*>(k_lds1 + (wave + x) * 2 * KL::kPageBytes + 16 * jr);
        f32x4 po[RM::kV];
#pragma unroll
        for (int k = 0; k < RM::kV; ++k)
          po[k] = *reinterpret_cast<const f32x4*>(xo + 16 * ((RM::kV * sub + k) ^ jr));
        rm.raise(ml[0]);
        rm.add(ml, po);
      }
      if (j >= G) continue;
      if (whole) {
        const float inv = 1.0f / rm.l;
        const int64_t row = (int64_t)cu.task * a.num_q_heads + head * G + j;
        uint16_t* orow = a.out + row * D + RM::kPer * sub;
#pragma unroll
        for (int k = 0; k < RM::kV; ++k) {
          const uint2 x = {pack_bf16x2(rm.acc[k][0] * inv, rm.acc[k][1] * inv),
                           pack_bf16x2(rm.acc[k][2] * inv, rm.acc[k][3] * inv)};
          *reinterpret_cast<uint2*>(orow + 4 * k) = x;
        }
        if (a.lse && sub == 0) a.lse[row] = (rm.mx + __log2f(rm.lx)) * kLn2;
      } else {
        const int64_t slot = slot0 + slots.open(run, cu.task);
        float* po = a.part_o + slot * G * D;
#pragma unroll
        for (int k = 0; k < RM::kV; ++k)
          store_f32x4_device(po, G * D * 4, 4 * (j * D + RM::kPer * sub + 4 * k), rm.acc[k]);
        if (sub == 0)
          store_f32x4_device(a.part_ml + slot * G * 4, G * 16, 16 * j,
                             f32x4{rm.mx, rm.l, rm.lx, 0.0f});
      }
    }
  };
  if (G > 4) combine(std::integral_constant<int, 8>());
  else combine(std::integral_constant<int, 16>());
  if (!whole) arrive(u, cu.task, slot0 + slots.open(run, cu.task));
}

template <int D, bool kAppend>
hipError_t launch_stream(const StreamArgs& a, hipStream_t stream) {
  const int waves = stream_waves((int64_t)a.num_runs * a.num_kv_heads);
  const int blocks = stream_groups(a.num_runs, a.num_kv_heads);
  if (waves == kStreamBig)
    hipLaunchKernelGGL((decode_stream_kernel<D, kAppend, kStreamBig>), dim3(blocks),
                       dim3(kStreamBig * 64), 0, stream, a);
  else
    hipLaunchKernelGGL((decode_stream_kernel<D, kAppend, kStreamSmall>), dim3(blocks),
                       dim3(kStreamSmall * 64), 0, stream, a);
  return hipGetLastError();
}

// Every variant is instantiated explicitly (see attn_decode.hip).
template __global__ void decode_stream_kernel<128, false, kStreamBig>(StreamArgs);
template __global__ void decode_stream_kernel<128, false, kStreamSmall>(StreamArgs);
template __global__ void decode_stream_kernel<128, true, kStreamBig>(StreamArgs);
template __global__ void decode_stream_kernel<128, true, kStreamSmall>(StreamArgs);
template __global__ void decode_stream_kernel<64, false, kStreamBig>(StreamArgs);
template __global__ void decode_stream_kernel<64, false, kStreamSmall>(StreamArgs);
template __global__ void decode_stream_kernel<64, true, kStreamBig>(StreamArgs);
template __global__ void decode_stream_kernel<64, true, kStreamSmall>(StreamArgs);

}  // namespace kern

hipError_t launch_decode_stream(const StreamArgs& a, int head_dim, hipStream_t stream) {
  const bool append = a.k_new != nullptr;
  if (head_dim == 128)
    return append ? kern::launch_stream<128, true>(a, stream) : kern::launch_stream<128, false>(a, stream);
  if (head_dim == 64)
    return append ? kern::launch_stream<64, true>(a, stream) : kern::launch_stream<64, false>(a, stream);
  return hipErrorInvalidValue;
}

}  // namespace tide
