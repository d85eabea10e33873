// What the two main attention kernels share: operand types and conversions,
// waits, the kernel arguments and the loads of the plan's records.
#pragma once

#include "attn_device.h"
#include "echo_device.h"
#include "echo_internal.h"

namespace echo {
namespace {

typedef __attribute__((address_space(3))) void lds_void_t;
typedef short shortx4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) shortx4 lds_shortx4_t;

__device__ __forceinline__ bf16x8 as_bf16x8(uint4 v) { return __builtin_bit_cast(bf16x8, v); }

typedef float floatx2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

// Round two floats to bfloat16 (to nearest even) in one v_cvt_pk_bf16_f32.
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(floatx2{lo, hi}, bf16x2));
}

// acc plus the two bfloat16 values packed in w (one v_dot2c_f32_bf16 against
// (1, 1); the products are exact).
__device__ __forceinline__ float add_bf16x2(uint32_t w, float acc) {
  return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, w),
                                         __builtin_bit_cast(bf16x2, 0x3F803F80u), acc, false);
}

__device__ __forceinline__ int swz_pattern(int row) { return ((row & 3) << 2) | ((row >> 2) & 3); }

__device__ __forceinline__ uint64_t uniform64(uint64_t x) {
  const uint32_t lo = __builtin_amdgcn_readfirstlane(uint32_t(x));
  const uint32_t hi = __builtin_amdgcn_readfirstlane(uint32_t(x >> 32));
  return (uint64_t(hi) << 32) | lo;
}

template <int N>
__device__ __forceinline__ void wait_vm() {
  // gfx9 s_waitcnt encoding: vmcnt[3:0] | expcnt[6:4] | lgkmcnt[11:8] | vmcnt_hi[15:14]
  constexpr int imm = (N & 15) | (7 << 4) | (15 << 8) | ((N >> 4) << 14);
  __builtin_amdgcn_s_waitcnt(imm);
}

__device__ __forceinline__ void wait_lds() {
  // lgkmcnt(0); vmcnt and expcnt left at their maxima
  __builtin_amdgcn_s_waitcnt(15 | (7 << 4) | (0 << 8) | (3 << 14));
}

// The wave's index in the workgroup, known to the compiler as wave-uniform (so
// that everything derived from it stays in scalar registers).
__device__ __forceinline__ int wave_id() {
  return __builtin_amdgcn_readfirstlane(int(threadIdx.x) / kWave);
}

struct MainArgs {
  const uint16_t* q;
  const uint16_t* k_new;
  const uint16_t* v_new;
  const uint16_t* k_cache;
  const uint16_t* v_cache;
  const int32_t* block_table;  // paged prefix (else nullptr): see KvSource
  int page_shift;              // log2 of the page size (>= 5: a tile never straddles pages)
  int max_pages;
  const uint32_t* tree_mask;
  int W, hq, hkv, G;
  float scale2;
  float* out;
  float* lse;
};

// Unit descriptors are written by the plan launch and only read here: load
// them through the constant address space (scalar loads when the index is
// wave-uniform).
typedef __attribute__((address_space(4))) const int32_t const_i32_t;
__device__ __forceinline__ Unit load_unit(const Unit* units, int i) {
  static_assert(sizeof(Unit) == 12 * sizeof(int32_t), "unit layout");
  const_i32_t* p = (const_i32_t*)(units + i);
  Unit u;
  u.tile_start = p[0];
  u.tile_end = p[1];
  u.q0 = p[2];
  u.nslots = p[3];
  u.kb = p[4];
  u.P = p[5];
  u.ntail = p[6];
  u.passes = p[7];
  u.rpp = p[8];
  u.group = p[9];
  u.cut = p[10];
  u.wide = p[11];
  return u;
}

// A workgroup's start record, through the constant address space as the units.
__device__ __forceinline__ WgStart load_wg_start(const WgStart* starts, int b) {
  static_assert(sizeof(WgStart) == 16 * sizeof(int32_t), "start record layout");
  const_i32_t* p = (const_i32_t*)(starts + b);
  int32_t w[16];
#pragma unroll
  for (int k = 0; k < 16; ++k) w[k] = p[k];
  return __builtin_bit_cast(WgStart, w);
}

// The tree-mask word of tail tile lt for a row of slot `slot` (0 outside).
__device__ __forceinline__ uint32_t mask_word(const MainArgs& a, const Unit& ud, bool row_ok,
                                              int slot, int lt) {
  return (row_ok && lt >= 0 && lt < ud.ntail && lt < a.W)
             ? a.tree_mask[size_t(slot) * a.W + lt]
             : 0u;
}

}  // namespace
}  // namespace echo
