// Device helpers for the gfx950 kernels: vector types, bf16 packing, MFMA wrappers and
// the lane-permutation that makes MFMA outputs feed the next MFMA directly.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "tide_common.h"

namespace tide {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr float kLn2 = 0.69314718055994530942f;
constexpr float kLog2e = 1.44269504088896340736f;
// Running-max sentinel: finite so that exp2(m_old - m_new) never sees (-inf) - (-inf).
constexpr float kNoMax = -1.0e30f;
// A row's reference max is only raised when the tile max exceeds it by more than this
// (base-2 units).  Unnormalised weights then stay <= 2^8, far from fp32/bf16 limits,
// and the accumulator rescale is skipped on almost every tile.
constexpr float kRescaleSlack = 8.0f;

typedef const __attribute__((address_space(4))) int32_t const_i32;

// Block-table word `idx` of a row, read through the constant address space: the table is
// read-only during a kernel, so a wave-uniform index becomes a scalar load (counted by
// lgkmcnt, so waiting for it never waits for outstanding vector loads).
__device__ __forceinline__ int32_t load_page_id(const int32_t* row, int idx) {
  return ((const_i32*)row)[idx];
}

__device__ __forceinline__ u32x4 load_u32x4(const void* p) {
  return *reinterpret_cast<const u32x4*>(p);
}

__device__ __forceinline__ void store_u32x4(void* p, u32x4 v) {
  *reinterpret_cast<u32x4*>(p) = v;
}

__device__ __forceinline__ bf16x8 as_bf16x8(u32x4 v) { return __builtin_bit_cast(bf16x8, v); }

__device__ __forceinline__ u32x4 zero_u32x4() {
  u32x4 z = {0u, 0u, 0u, 0u};
  return z;
}

// Two fp32 values -> packed bf16 pair (round to nearest even, v_cvt_pk_bf16_f32).
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
  f32x2 v = {lo, hi};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// acc + lo + hi of a packed bf16 pair (v_dot2c_f32_bf16 against (1, 1)).  Summing the
// rounded probabilities keeps the softmax denominator consistent with the bf16 weights
// the P.V product actually uses, at half a VALU instruction per probability.
__device__ __forceinline__ float add_bf16x2(uint32_t packed, float acc) {
  const bf16x2 one = __builtin_bit_cast(bf16x2, 0x3F803F80u);  // (1.0, 1.0)
  return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, packed), one, acc, false);
}

__device__ __forceinline__ float xor_shfl(float v, int mask) {
  return __shfl_xor(v, mask, 64);
}

// Tells the host that workgroup `group` has read its part of a plan in a staging slot.  One
// thread calls it, after a barrier behind which every wave has its plan values.
__device__ __forceinline__ void plan_read(const PlanReads& r, uint32_t group) {
  __hip_atomic_store(r.done + group, r.seq, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// Merge of split partials, the split-K merge of flash decoding.  D / 4 lanes combine the n
// partials of one (row, query head), so a wave takes 64 / (D / 4) of them (kMergeRows):
// partial s holds, at ml + s * ml_stride, its running max m_s (base-2 units), the sum of its
// bf16-rounded weights and their exact fp32 sum, and at po + s * po_stride its unnormalised
// output.  With M = max m_s and w_s = 2^(m_s - M) the row is sum_s w_s o_s / sum_s w_s l_s,
// written as bf16 to orow; when lse_out is non-null it receives ln(sum_s w_s l_exact_s) +
// M ln 2.  Every sum runs in split order.  n may differ between the lanes of a wave (n < 1:
// nothing to do).
//
// Each lane loads the statistics and 16 bytes of 8 partials (4, where no row of the wave has
// more) before any arithmetic, so up to 8 splits cost one memory round trip.  The merge is
// bound by the waves it keeps in flight: with one row a wave and 8 bytes a lane (104 VGPRs,
// 16 waves a CU) 22,428 rows of 8 partials took 31.0 us, now 17.5; 8,192 rows of 3-8 partials
// 12.0 us, now 6.3; 2,048 rows of 5-12 partials 7.8 us, now 4.9.
template <int D>
constexpr int kMergeRows = 64 / (D / 4);

template <int D, int kBatch>
__device__ __forceinline__ void merge_batches(const float* ml, int64_t ml_stride, const float* po,
                                               int64_t po_stride, int n, uint16_t* orow,
                                               float* lse_out) {
  const int sub = threadIdx.x & (D / 4 - 1);  // this lane's 4 head-dim entries
  f32x4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
  float mx = kNoMax, l = 0.0f, lx = 0.0f;
  for (int s0 = 0; s0 < n; s0 += kBatch) {
    f32x4 st[kBatch], src[kBatch];
#pragma unroll
    for (int i = 0; i < kBatch; ++i) {
      const int s = min(s0 + i, n - 1);  // past n: loaded again, not summed
      st[i] = *reinterpret_cast<const f32x4*>(ml + s * ml_stride);
      src[i] = *reinterpret_cast<const f32x4*>(po + s * po_stride + 4 * sub);
    }
    float m = mx;
#pragma unroll
    for (int i = 0; i < kBatch; ++i) m = fmaxf(m, st[i][0]);
    const float w = fast_exp2(mx - m);
    acc *= w;
    l *= w;
    lx *= w;
    mx = m;
#pragma unroll
    for (int i = 0; i < kBatch; ++i) {
      const float wi = s0 + i < n ? fast_exp2(st[i][0] - mx) : 0.0f;
      l += wi * st[i][1];
      lx += wi * st[i][2];
      acc += wi * src[i];
    }
  }
  if (n < 1) return;
  const float inv = 1.0f / l;
  const uint2 out = {pack_bf16x2(acc[0] * inv, acc[1] * inv), pack_bf16x2(acc[2] * inv, acc[3] * inv)};
  *reinterpret_cast<uint2*>(orow + 4 * sub) = out;
  if (lse_out && sub == 0) *lse_out = (mx + __log2f(lx)) * kLn2;
}

template <int D>
__device__ __forceinline__ void merge_partials(const float* ml, int64_t ml_stride, const float* po,
                                               int64_t po_stride, int n, uint16_t* orow,
                                               float* lse_out) {
  if (__builtin_amdgcn_ballot_w64(n > 4) == 0)
    merge_batches<D, 4>(ml, ml_stride, po, po_stride, n, orow, lse_out);
  else
    merge_batches<D, 8>(ml, ml_stride, po, po_stride, n, orow, lse_out);
}

// v_mfma_f32_32x32x16_bf16.  Lane layouts (checked on gfx950):
//   A: lane l holds row l%32, k = 8*(l/32) .. +7;  B: lane l holds column l%32, same k;
//   D: lane l register r holds row 8*(r/4) + 4*(l/32) + r%4, column l%32.
__device__ __forceinline__ f32x16 mfma32(bf16x8 a, bf16x8 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

// v_mfma_f32_16x16x32_bf16.  A: lane l row l%16, k = 8*(l/16) .. +7; B: column l%16;
//   D: lane l register r holds row 4*(l/16) + r, column l%16.
__device__ __forceinline__ f32x4 mfma16(bf16x8 a, bf16x8 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// Row permutation for the 32x32 tiles.  When the 32 rows of an S^T = K.Q^T tile are the
// keys kappa(0..31), the D registers r = 0..7 of lane l hold keys 8*(l/32) + r and
// registers 8..15 hold 16 + 8*(l/32) + (r - 8): each lane owns runs of 8 consecutive
// keys, which is exactly the B operand of the P.V product over 16 keys.  The V^T operand
// of that product is read so that its rows follow the same pattern over the head-dim
// entries, which makes each lane's outputs 8 consecutive entries (16-byte stores).
__device__ __forceinline__ int perm32(int rho) {
  const int j = rho >> 3, h = (rho >> 2) & 1, r = rho & 3;
  return 16 * (j >> 1) + 8 * h + 4 * (j & 1) + r;
}

}  // namespace tide
