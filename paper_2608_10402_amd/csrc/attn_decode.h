// attn_decode.h -- building blocks of the decode kernels (attn_decode.hip: one chunk per
// wave; attn_decode_stream.hip: a run of steps per wave): how a 32-key step's K and V pages
// are loaded, laid out in LDS and read back as MFMA operands, and the device-scope stores
// of split partials.
#pragma once

#include <type_traits>

#include "kernels.h"
#include "tide_device.h"

namespace tide {
namespace kern {

// V of one 32-key step (pages p0 = keys k..k+15 and p1 = k+16..k+31): v[h][i] is this
// lane's 16 bytes of load i of page h, which covers page bytes 1024 i .. 1024 i + 1023.
// The step's K pages sit in a per-wave LDS buffer.
template <int D>
struct DecodeRegs {
  static constexpr int kLoads = kPage * D * 2 / 1024;  // 1 KB loads per page
  u32x4 v[2][kLoads];
};

typedef __attribute__((address_space(3))) void lds_void;
typedef short i16x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) i16x4 lds_i16x4;

// V page layout in LDS, written over the step's K copy once its scores are computed: row
// r (16 of them, 2D bytes each) keeps its order, and its 32-byte blocks are XOR-swizzled
// by vsw(r), so that the 8 rows x 32 bytes a half-wave reads with ds_read_b64_tr_b16 fall
// in distinct banks, and the 16 lanes of a 16-byte write of one row too.
template <int D>
struct VLds {
  static constexpr int kNG = D / 8;  // 16-byte granules per row
  static __device__ __forceinline__ int vsw(int r) { return D == 128 ? (r & 7) : ((r >> 1) & 3); }
  // byte offset, inside a page copy, of 16-byte granule g of row r
  static __device__ __forceinline__ uint32_t offset(int r, int g) {
    return (uint32_t)(r * 2 * D + 32 * ((g >> 1) ^ vsw(r)) + 16 * (g & 1));
  }
};

// K page layout in LDS.  A page block is 16 key rows of D bf16 (2D bytes = D/8 granules
// of 16 bytes).  It is copied by 2 * (D/64) direct-to-LDS instructions; instruction
// i = a * (D/64) + h covers rows 8a..8a+7 and granules 8h..8h+7 of each, lane l taking
// row r = 8a + l/8 and granule 8h + ((l%8) ^ ((r/2)%8)), which lands at byte
// 1024 * i + 16 * l of the page's LDS copy.  Granule g of row r is therefore found at
// slot 8 * (r%8) + ((g%8) ^ ((r/2)%8)) of instruction (r/8) * (D/64) + g/8; a read of one
// granule by the 16 rows of an MFMA operand touches 16 distinct 16-byte bank groups.
template <int D>
struct KLds {
  static constexpr int kHalves = D / 64;           // 128-byte halves of a key row
  static constexpr int kDma = 2 * kHalves;         // direct-to-LDS loads per page
  static constexpr int kPageBytes = kPage * D * 2;
  static_assert(kDma * 1024 == kPageBytes, "page = whole 1 KB loads");
  // global byte offset, inside the page block, of lane `lane`'s 16 bytes in load i
  static __device__ __forceinline__ uint32_t src_offset(int i, int lane) {
    const int r = 8 * (i / kHalves) + (lane >> 3);
    const int g = 8 * (i % kHalves) + ((lane & 7) ^ ((r >> 1) & 7));
    return (uint32_t)(r * 2 * D + 16 * g);
  }
  // LDS byte offset, inside the page copy, of granule g of row r
  static __device__ __forceinline__ uint32_t lds_offset(int r, int g) {
    const int i = (r >> 3) * kHalves + (g >> 3);
    return (uint32_t)(1024 * i + 16 * (8 * (r & 7) + ((g & 7) ^ ((r >> 1) & 7))));
  }
};

// Buffer resource of one (page, kv head) block: base in SGPRs, range = the block, so each
// load is a 32-bit lane offset plus an immediate (raw buffer, gfx9 descriptor format).
__device__ __forceinline__ __amdgpu_buffer_rsrc_t block_rsrc(const uint8_t* base, int bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(base), 0, bytes, 0x00020000);
}

// Cache policy of the K/V loads.  Keys that one wave alone reads (a task's context in
// plain decode, a trajectory's own keys after a shared prompt) are streamed with the
// non-temporal hint (the nt bit, aux bit 1 on gfx950): streaming reads measured 7.1 TB/s
// on MI355X with it against 6.3 TB/s without.  A shared prompt chunk, which the waves of
// a group's other subgroups read right after, keeps the default policy so that those
// reads hit L2.
constexpr int kStreamPolicy = 2;
constexpr int kSharedPolicy = 0;

// Loads of one step.  Every instruction reads a single page block: the K pages go to
// kbuf (page t at t * kPageBytes), the V rows to registers.
template <int D, int kPolicy>
__device__ __forceinline__ void load_step(DecodeRegs<D>& r, uint8_t* kbuf,
                                          __amdgpu_buffer_rsrc_t k0, __amdgpu_buffer_rsrc_t k1,
                                          __amdgpu_buffer_rsrc_t v0, __amdgpu_buffer_rsrc_t v1,
                                          const uint32_t (&k_src)[KLds<D>::kDma],
                                          uint32_t v_off) {
  using L = KLds<D>;
#pragma unroll
  for (int i = 0; i < L::kDma; ++i) {
    __builtin_amdgcn_raw_ptr_buffer_load_lds(k0, (lds_void*)(kbuf + 1024 * i), 16, k_src[i], 0,
                                             0, kPolicy);
    __builtin_amdgcn_raw_ptr_buffer_load_lds(k1, (lds_void*)(kbuf + L::kPageBytes + 1024 * i),
                                             16, k_src[i], 0, 0, kPolicy);
  }
#pragma unroll
  for (int i = 0; i < DecodeRegs<D>::kLoads; ++i) {
    r.v[0][i] = __builtin_bit_cast(
        u32x4, __builtin_amdgcn_raw_buffer_load_b128(v0, v_off + 1024 * i, 0, kPolicy));
    r.v[1][i] = __builtin_bit_cast(
        u32x4, __builtin_amdgcn_raw_buffer_load_b128(v1, v_off + 1024 * i, 0, kPolicy));
  }
}

// Transposed read of 4 key rows x 16 head-dim entries of a V page (ds_read_b64_tr_b16).
__device__ __forceinline__ uint2 read_tr(const uint8_t* p) {
  const i16x4 v = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4*)p);
  return __builtin_bit_cast(uint2, v);
}

// Keep only the first n (0..4) bf16 elements of an 8-byte V^T piece.
__device__ __forceinline__ uint2 keep_first4(uint2 x, int n) {
  uint2 r;
  r.x = x.x & ((n > 0 ? 0x0000FFFFu : 0u) | (n > 1 ? 0xFFFF0000u : 0u));
  r.y = x.y & ((n > 2 ? 0x0000FFFFu : 0u) | (n > 3 ? 0xFFFF0000u : 0u));
  return r;
}

// Partials of plain decode travel between CUs, possibly on different XCDs, whose L2s are
// not kept coherent for ordinary accesses.  They are therefore stored and loaded with
// device-scope cache policy (SC1: the store writes through to the device's coherence
// point, the load does not take a possibly stale cached line), which makes the heavy
// cache write-back and invalidate of a device-scope fence unnecessary: a wave waits for
// its partial stores to complete before it counts its arrival, and the merging wave
// loads the partials only after its count returned.
constexpr int kDeviceScope = 16;  // buffer cache policy bit SC1

__device__ __forceinline__ void store_f32x4_device(float* base, uint32_t bytes, uint32_t off,
                                                   f32x4 v) {
  const auto rsrc = __builtin_amdgcn_make_buffer_rsrc(base, 0, bytes, 0x00020000);
  __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), rsrc, off, 0, kDeviceScope);
}

}  // namespace kern
}  // namespace tide
