// Device-side helpers shared by the two attention kernels (gfx950).  Not part of the public ABI.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "adsa_internal.h"

namespace adsa {

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// Pointers the kernel reads out of the sequence record are declared as what they are, global memory:
// the accesses then compile to global (not flat) instructions whatever else is done with the value.
#define ADSA_GLOBAL __attribute__((address_space(1)))
typedef ADSA_GLOBAL char gchar;
typedef ADSA_GLOBAL float gfloat;
typedef ADSA_GLOBAL int32_t gint;
typedef ADSA_GLOBAL adsa_seq gseq;

// Addresses have 48 bits: as leading kernel arguments of the attention launches, their low halves and, two to a dword, the rest
constexpr int kLeadBytes = 14 * 4;                 // of the arguments before the block that is not preloaded
__device__ __forceinline__ uint64_t address(uint32_t lo, uint32_t hi) { return ((uint64_t)hi << 32) | lo; }
static inline uint32_t lo32(const void* p) { return (uint32_t)reinterpret_cast<uintptr_t>(p); }
static inline uint32_t hi16s(const void* p, const void* q) {
  return (uint32_t)(reinterpret_cast<uintptr_t>(p) >> 32 & 0xFFFF) | (uint32_t)(reinterpret_cast<uintptr_t>(q) >> 32) << 16;
}

// 16-byte streaming load: K/V rows are read once per step, so keep them out of the caches' way
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ uint4 load_stream16(const gchar* p) {
  const u32x4 v = __builtin_nontemporal_load(reinterpret_cast<const ADSA_GLOBAL u32x4*>(p));
  return make_uint4(v.x, v.y, v.z, v.w);
}
__device__ __forceinline__ uint4 load16(const gchar* p) {
  const u32x4 v = *reinterpret_cast<const ADSA_GLOBAL u32x4*>(p);
  return make_uint4(v.x, v.y, v.z, v.w);
}
__device__ __forceinline__ void store16(gchar* p, const uint4& x) {
  u32x4 v; v.x = x.x; v.y = x.y; v.z = x.z; v.w = x.w;
  *reinterpret_cast<ADSA_GLOBAL u32x4*>(p) = v;
}

__device__ __forceinline__ void store_stream16(gchar* p, const uint4& x) {
  u32x4 v; v.x = x.x; v.y = x.y; v.z = x.z; v.w = x.w;
  __builtin_nontemporal_store(v, reinterpret_cast<ADSA_GLOBAL u32x4*>(p));
}

// One sequence's row of sel_idx.  Entry i of it, or 0 without an access where i >= sel_cap: kernels ask for entries of their first
// round trip before the count has arrived.  The whole index goes into the vector offset (and the instruction's own): those two are
// what a buffer load compares with the descriptor's size, a scalar offset is added behind the check.
struct SlotList {
  __amdgpu_buffer_rsrc_t row;
  __device__ __forceinline__ SlotList(const gint* first, int sel_cap)
      : row(__builtin_amdgcn_make_buffer_rsrc((void*)(const int32_t*)first, 0, sel_cap * 4, 0x00027000)) {}
  __device__ __forceinline__ int operator[](int i) const { return (int)__builtin_amdgcn_raw_buffer_load_b32(row, i * 4, 0, 0); }
};

// Rows of a cache within 32-bit offsets of a uniform address: 16-byte streaming loads that read zeros, without an access, at any
// offset from kRowBufferBytes on.  ~(slot + ADSA_MAX_CAP), as an unsigned number, is such an offset for every slot of a cache, and the
// 16 bytes from there on don't reach the end of the 32 bits.
constexpr uint32_t kRowBufferBytes = 0u - 2 * ADSA_MAX_CAP;
static_assert((ADSA_MAX_CAP & (ADSA_MAX_CAP - 1)) == 0 && ADSA_MAX_CAP >= 16, "slot + ADSA_MAX_CAP is slot ^ ADSA_MAX_CAP");
struct RowBuffer {
  __amdgpu_buffer_rsrc_t rows;
  __device__ __forceinline__ explicit RowBuffer(const gchar* first)
      : rows(__builtin_amdgcn_make_buffer_rsrc((void*)(const char*)first, 0, (int)kRowBufferBytes, 0x00027000)) {}
  __device__ __forceinline__ uint4 operator[](uint32_t offset) const {
    const u32x4 v = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rows, (int)offset, 0, kNonTemporal));
    return make_uint4(v.x, v.y, v.z, v.w);
  }
  static constexpr int kNonTemporal = 2;           // the instruction's cache bits
};

// Round to the nearest bf16, ties to even (v_cvt_pk_bf16_f32; subnormals are kept, a NaN stays one)
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t pack2_bf16(float lo, float hi) {
  const bf16x2 v = {(__bf16)lo, (__bf16)hi};
  return __builtin_bit_cast(uint32_t, v);
}
__device__ __forceinline__ uint32_t f32_to_bf16_rne(float x) { return pack2_bf16(x, 0.0f) & 0xFFFFu; }

// 8 consecutive fp32 values, as two 16-byte vectors -> 8 bf16 in one
__device__ __forceinline__ uint4 pack8_bf16(const uint4& a, const uint4& b) {
  return make_uint4(pack2_bf16(__uint_as_float(a.x), __uint_as_float(a.y)), pack2_bf16(__uint_as_float(a.z), __uint_as_float(a.w)),
                    pack2_bf16(__uint_as_float(b.x), __uint_as_float(b.y)), pack2_bf16(__uint_as_float(b.z), __uint_as_float(b.w)));
}
__device__ __forceinline__ uint4 pack8_bf16(const gchar* f) { return pack8_bf16(load16(f), load16(f + 16)); }

// The record at the end of an attention launch (one thread per sequence); see kAdvance.
__device__ __forceinline__ void advance_step(ADSA_GLOBAL adsa_seq* sq, int mode) {
  if (mode != kAdvanceNone) sq->step = sq->step + 1;
  if (mode == kAdvanceActive) sq->compacted = 0;
}
__device__ __forceinline__ void advance_empty(ADSA_GLOBAL adsa_seq* sq, int mode) {      // a sequence without an attended token
  if (mode == kAdvanceActive && sq->status == 0 && sq->step >= 0) advance_step(sq, mode);
}

// Demands a wave-uniform value that was just loaded in scalar registers AT THIS POINT of the program:
// its load cannot sink below the statement, into a later and then dependent round trip.  (Input only:
// the value itself, and what the compiler knows about where a pointer points, stay as they are.)
template <typename T>
__device__ __forceinline__ void pin_uniform(const T& x) { asm volatile("" : : "s"(x)); }

template <int CTRL>
__device__ __forceinline__ float dpp_f(float x) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xF, 0xF, true));
}

// Value of lane (lane ^ X) for X in {8, 16, 32}: DPP inside a 16-lane row, register-only swaps of
// 16- and 32-lane halves beyond it (both outputs of a swap of x with itself are returned).
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
template <int X>
__device__ __forceinline__ float xor_sum(float x) {
  if constexpr (X == 8) return x + dpp_f<0x128>(x);            // row_ror:8
  else {
    const unsigned u = __float_as_uint(x);
    const u32x2 r = X == 16 ? __builtin_amdgcn_permlane16_swap(u, u, false, false)
                            : __builtin_amdgcn_permlane32_swap(u, u, false, false);
    return __uint_as_float(r.x) + __uint_as_float(r.y);       // one of the two is x itself, the other its partner
  }
}
// (of values of which none is a signalling NaN: fmaxf would first quiet each of them)
__device__ __forceinline__ float max2(float a, float b) {
  float r;
  asm("v_max_f32 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
  return r;
}
template <int X>
__device__ __forceinline__ float xor_max(float x) {
  if constexpr (X == 8) return max2(x, dpp_f<0x128>(x));
  else {
    const unsigned u = __float_as_uint(x);
    const u32x2 r = X == 16 ? __builtin_amdgcn_permlane16_swap(u, u, false, false)
                            : __builtin_amdgcn_permlane32_swap(u, u, false, false);
    return max2(__uint_as_float(r.x), __uint_as_float(r.y));
  }
}

}  // namespace adsa
