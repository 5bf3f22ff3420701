// Device helpers shared by the GEMV (kernels.hip) and the batched GEMV
// (batch.hip): vector types, the instructions the decoders are built of,
// buffer descriptors, the class table's entries and the activation's pair
// order.  Not part of the public ABI.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "leech_internal.h"

namespace leech {

typedef _Float16 half2_t __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4), aligned(4)));
typedef uint32_t u32x3 __attribute__((ext_vector_type(3), aligned(4)));
typedef uint32_t u32x4a __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2a __attribute__((ext_vector_type(2)));
typedef float f32x4a __attribute__((ext_vector_type(4)));
constexpr float kTwo24 = 16777216.0f;
constexpr int kTableBytes = 1024 * 16;    // LDS class-table entries (class | gain << 9)
// Raw buffer descriptor, word 3, for the gfx9 family (32-bit elements, no
// swizzle), and the non-temporal hint of the GEMV's record and scale loads, which
// it reads once (the wide batched kernel, which reads them once a batch tile,
// loads without it).
constexpr int kRsrcWord3 = 0x00020000;
constexpr int kStreamed = 2;

// Per-(class, gain) entry staged in LDS at byte (class | gain << 9) · 16.
struct LdsEntry {
  uint32_t tlo, thi;    // v_perm table (DevClass::perm; Planes12x: see p12_core;
                        // Golay70: see golay70_core)
  float factor;         // 2^24 · centroid[gain] / (4√m)
  uint32_t aux;         // Slot32: level count; Planes12x, Golay70: f32 added to the
                        // block's sum × factor (0, or an exception's kept contribution)
};
static_assert(sizeof(LdsEntry) * 1024 == kTableBytes, "table entries are 16 bytes");

__device__ __forceinline__ uint32_t align(uint32_t hi, uint32_t lo, uint32_t s) {
  return __builtin_amdgcn_alignbit(hi, lo, s);
}
__device__ __forceinline__ uint32_t perm(uint32_t s0, uint32_t s1, uint32_t sel) {
  return __builtin_amdgcn_perm(s0, s1, sel);
}
// Reinterpret a 32-bit word as two binary16 values.  Takes the word by value:
// applying __builtin_bit_cast directly to an ext_vector element (w.y) reads
// element 0 with this compiler, so vector elements go through this function.
__device__ __forceinline__ half2_t as_h2(uint32_t v) { return __builtin_bit_cast(half2_t, v); }

__device__ __forceinline__ _Float16 as_half(uint32_t h) {
  return __builtin_bit_cast(_Float16, (uint16_t)h);
}

// Coordinates of pair k of h[] (and of the staged x pairs).
__host__ __device__ constexpr void pair_coords(int k, int& c0, int& c1) {
  const int r = k / 3, m = k % 3;
  c0 = m == 0 ? r : (m == 1 ? 4 + r : 8 + r);
  c1 = m == 0 ? 16 + r : (m == 1 ? 20 + r : 12 + r);
}
// The Planes14 record stores its pairs in the host's kPairCoords order, which
// must be this one.
__host__ __device__ constexpr bool pair_order_matches_records() {
  for (int k = 0; k < 12; ++k) {
    int c0 = 0, c1 = 0;
    pair_coords(k, c0, c1);
    if (c0 != kPairCoords[k][0] || c1 != kPairCoords[k][1]) return false;
  }
  return true;
}
static_assert(pair_order_matches_records(), "pair order of the kernels and the records");

// Planes14 record in the four-word window whose record starts at bit sh (0
// or 16): each pair word starts on a 32-bit boundary of the record, so one
// funnel shift each gives it; e16 = (class | gain << 9)·16, the entry's LDS
// byte address.  Pair q = 4w + k of word w is its rotation by 4k masked with
// 0x08070807, which is already the byte-permute selector of the pair's two
// binary16 values (the store order of the record): no transpose, no pair
// gathering.
__device__ __forceinline__ void p14_record(uint32_t w0, uint32_t w1, uint32_t w2, uint32_t w3,
                                           uint32_t sh, uint32_t esh, uint32_t W[3],
                                           uint32_t& e16) {
  W[0] = align(w1, w0, sh);
  W[1] = align(w2, w1, sh);
  W[2] = align(w3, w2, sh);
  e16 = align(w3, w3, esh) & 0x3FF0u;
}
__device__ __forceinline__ void p14_core(const uint32_t W[3], uint32_t tlo, uint32_t thi,
                                         uint32_t h[12]) {
#pragma unroll
  for (int w = 0; w < 3; ++w)
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const uint32_t s = k ? align(W[w], W[w], 4 * k) : W[w];
      h[4 * w + k] = perm(thi, tlo, s & 0x08070807u);
    }
}

__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void* base, uint64_t bytes) {
  const uint32_t n = bytes > 0xFFFFFFFFull ? 0xFFFFFFFFu : (uint32_t)bytes;
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, (int)n, kRsrcWord3);
}

// The LDS entries, built from the device table: one 16-byte load per entry.
__device__ __forceinline__ LdsEntry make_entry(const DevClass* tab, uint32_t e, float cen0,
                                               float cen1) {
  const u32x4a d = *(const u32x4a*)&tab[e & 511u];      // perm[8], inv_norm, info
  LdsEntry t;
  t.tlo = d.x;
  t.thi = d.y;
  t.factor = __builtin_bit_cast(float, (uint32_t)d.z) * kTwo24 * ((e >> 9) ? cen1 : cen0);
  t.aux = d.w & 0xFFu;
  return t;
}

// x of block j in the cores' pair order: three 16-byte loads, then pair k
// (coordinates pair_coords(k)) picked by one v_perm_b32 each.
struct XBlock {
  u32x4a v0, v1, v2;
};
__device__ __forceinline__ XBlock load_x_block(const uint16_t* xj) {
  const u32x4a* src = (const u32x4a*)xj;
  return XBlock{src[0], src[1], src[2]};
}
__device__ __forceinline__ void store_x_block(const XBlock& xb, uint32_t* dst) {
  const uint32_t w[12] = {xb.v0.x, xb.v0.y, xb.v0.z, xb.v0.w, xb.v1.x, xb.v1.y,
                          xb.v1.z, xb.v1.w, xb.v2.x, xb.v2.y, xb.v2.z, xb.v2.w};
  uint32_t o[12];
#pragma unroll
  for (int k = 0; k < 12; ++k) {
    int c0, c1;
    pair_coords(k, c0, c1);
    // low half: half c0 % 2 of word c0 / 2 (selector bytes 0..3 pick S1);
    // high half: half c1 % 2 of word c1 / 2 (bytes 4..7 pick S0)
    const uint32_t sel = (c0 & 1 ? 0x0302u : 0x0100u) | (c1 & 1 ? 0x07060000u : 0x05040000u);
    o[k] = perm(w[c1 >> 1], w[c0 >> 1], sel);
  }
  u32x4a* d = (u32x4a*)dst;
  d[0] = u32x4a{o[0], o[1], o[2], o[3]};
  d[1] = u32x4a{o[4], o[5], o[6], o[7]};
  d[2] = u32x4a{o[8], o[9], o[10], o[11]};
}

}  // namespace leech
