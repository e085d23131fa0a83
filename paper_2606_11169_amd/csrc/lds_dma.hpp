// Loads from global memory straight into LDS (buffer_load ... lds), used by the GEMM
// and attention kernels.
#pragma once

#include "common.hpp"

namespace lc {
namespace {

typedef __attribute__((ext_vector_type(4))) short s16x4_v;
// LDS addresses stay 32-bit LDS-space pointers throughout (no generic pointers)
typedef __attribute__((address_space(3))) char lds_t;
#define LDS_AS(T, ptr) ((__attribute__((address_space(3))) T *)(ptr))

typedef __attribute__((ext_vector_type(4))) int i32x4_v;

// Raw buffer descriptor (CDNA: dword3 = 0x00020000, stride 0): offsets past
// `bytes` read as zero.
__device__ __forceinline__ i32x4_v make_rsrc(const void *base, uint32_t bytes) {
  const uint64_t a = reinterpret_cast<uint64_t>(base);
  i32x4_v r;
  r[0] = __builtin_amdgcn_readfirstlane((int)(uint32_t)a);
  r[1] = __builtin_amdgcn_readfirstlane((int)((uint32_t)(a >> 32) & 0xFFFFu));
  r[2] = __builtin_amdgcn_readfirstlane((int)bytes);
  r[3] = 0x00020000;
  return r;
}

// 16 bytes per lane from the buffer at byte offset `off` into LDS at
// lds + 16 * lane. Issued as inline assembly: the compiler then does not track
// the load, so it inserts no wait for it before LDS reads of the other stage;
// the step's explicit wait before its barrier is what orders it.
__device__ __forceinline__ void dma16(i32x4_v rs, lds_t *lds, uint32_t off) {
  const uint32_t m0 = __builtin_amdgcn_readfirstlane((uint32_t) reinterpret_cast<uintptr_t>(lds));
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tbuffer_load_dwordx4 %0, %1, 0 offen lds"
               :
               : "v"(off), "s"(rs), "s"(m0)
               : "memory", "m0");
}

// The same with a wave-uniform part of the offset in the instruction's scalar
// offset. The hardware checks only the per-lane offset against the buffer's
// size, so callers use it where every lane's whole offset is inside the
// operand or the lane's own offset is past every size.
__device__ __forceinline__ void dma16s(i32x4_v rs, lds_t *lds, uint32_t voff, uint32_t soff) {
  const uint32_t m0 = __builtin_amdgcn_readfirstlane((uint32_t) reinterpret_cast<uintptr_t>(lds));
  asm volatile("s_mov_b32 m0, %3\n\ts_nop 0\n\tbuffer_load_dwordx4 %0, %1, %2 offen lds"
               :
               : "v"(voff), "s"(rs), "s"(__builtin_amdgcn_readfirstlane(soff)), "s"(m0)
               : "memory", "m0");
}

// 4 bytes per lane into lds + 4 * lane, without and with a scalar part
__device__ __forceinline__ void dma4(i32x4_v rs, lds_t *lds, uint32_t off) {
  const uint32_t m0 = __builtin_amdgcn_readfirstlane((uint32_t) reinterpret_cast<uintptr_t>(lds));
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tbuffer_load_dword %0, %1, 0 offen lds"
               :
               : "v"(off), "s"(rs), "s"(m0)
               : "memory", "m0");
}
__device__ __forceinline__ void dma4s(i32x4_v rs, lds_t *lds, uint32_t voff, uint32_t soff) {
  const uint32_t m0 = __builtin_amdgcn_readfirstlane((uint32_t) reinterpret_cast<uintptr_t>(lds));
  asm volatile("s_mov_b32 m0, %3\n\ts_nop 0\n\tbuffer_load_dword %0, %1, %2 offen lds"
               :
               : "v"(voff), "s"(rs), "s"(__builtin_amdgcn_readfirstlane(soff)), "s"(m0)
               : "memory", "m0");
}

}  // namespace
}  // namespace lc
