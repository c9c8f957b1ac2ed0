// Device-side helpers shared by the single-pass scan kernels: coherent cross-workgroup
// accesses, counted waits, direct HBM -> LDS loads, DPP reductions.
#pragma once

#include "scan_common.h"

namespace skipkv {

typedef __attribute__((__vector_size__(2 * sizeof(__bf16)))) __bf16 bf16x2_t;

// Cross-workgroup communication (the workgroups may sit on different XCDs, whose L2 caches are not
// coherent with each other).  Everything that is communicated - the statistics records of the items, the
// abort word - is accessed ONLY with device-scope relaxed atomics, which are coherent by themselves.
// A record is ONE 8-byte store and carries its own validity (its first word holds a marker until it is
// written), so readers need no ordering between words and writers need no fence or flag.  No device-scope
// fence is used: on this chip such a fence writes back and invalidates a whole L2, which is ruinous when
// thousands of workgroups do it.
__device__ __forceinline__ void coherent_store2(float2 *p, float2 v) {
  unsigned long long u = (unsigned long long)__float_as_uint(v.x) | ((unsigned long long)__float_as_uint(v.y) << 32);
  __hip_atomic_store(reinterpret_cast<unsigned long long *>(p), u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ float2 coherent_load2(const float2 *p) {
  const unsigned long long u =
      __hip_atomic_load(reinterpret_cast<const unsigned long long *>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return make_float2(__uint_as_float((uint32_t)u), __uint_as_float((uint32_t)(u >> 32)));
}

// s_waitcnt immediates (gfx9 encoding: vmcnt[3:0] | expcnt[6:4] | lgkmcnt[11:8] | vmcnt[5:4] << 14)
// A copy of a per-thread value that the compiler cannot trace back to its source: address parts
// derived from it are computed where they are used instead of being kept in registers (or in
// scratch, whose reloads would wait for every key load in flight) across a whole item.
__device__ __forceinline__ int opaque(int x) {
  asm volatile("" : "+v"(x));
  return x;
}

template <int N>
__device__ __forceinline__ void wait_vm() {  // at most N vector-memory operations still outstanding
  __builtin_amdgcn_s_waitcnt((N & 0xF) | (0x7 << 4) | (0xF << 8) | ((N >> 4) << 14));
}
__device__ __forceinline__ void wait_all() { __builtin_amdgcn_s_waitcnt(0); }
// Workgroup barrier for data exchanged through LDS: waits for this wave's LDS operations only, so
// that key loads already in flight for later stages are not drained (a __syncthreads() would).
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
  __builtin_amdgcn_s_barrier();
}

// Direct HBM -> LDS load: every lane fetches 16 bytes from its own global address; the wave's 64
// pieces land at wave_lds_base + lane * 16 (the base travels in M0).  Issued through inline
// assembly on purpose: the compiler orders LDS reads against direct loads it knows about by
// waiting for ALL of them, which would drain the ring of stages on every read; here the stages
// are ordered by hand with wait_vm<>() (loads complete in issue order).  Nothing else in this
// kernel uses M0.
__device__ __forceinline__ void load_to_lds_16(const void *gsrc, void *wave_lds_base) {
  const uint32_t l = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char *)wave_lds_base;
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(l), "v"(gsrc) : "memory");
}

// (lo, hi) fp32 -> packed bf16 pair, round to nearest even (v_cvt_pk_bf16_f32).
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
  bf16x2_t v;
  v[0] = (__bf16)lo;
  v[1] = (__bf16)hi;
  return __builtin_bit_cast(uint32_t, v);
}

__device__ __forceinline__ uint32_t lds_addr(const void *p) {
  return (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) char *)p;
}
__device__ __forceinline__ float lds_read_f32(uint32_t addr) {
  return *(const __attribute__((address_space(3))) float *)(uintptr_t)addr;
}

// Row (16-lane) reductions with the DPP modifier on the arithmetic instruction itself: one instruction per step.  The
// compiler folds the modifier into an addition; around a maximum it would put a second one (for signalling NaNs), so that
// is assembly, whose s_nop covers the two wait states a DPP read needs after a VALU write.  Its result goes where the
// operand is, never into a register of its own: the compiler might choose one that a matrix instruction in flight is
// still going to write (an element of its result that nobody uses), and it keeps the distance that this needs for its own
// instructions only.  The operand has to come from an instruction of the compiler's that is no matrix instruction, for
// the same reason.
#define SKIPKV_DPP_STEP(OP, N) asm volatile("s_nop 1\n\t" OP " %0, %0, %0 row_ror:" #N " row_mask:0xf bank_mask:0xf" : "+v"(v))
__device__ __forceinline__ float row16_max_fast(float v) {
  SKIPKV_DPP_STEP("v_max_f32_dpp", 8);
  SKIPKV_DPP_STEP("v_max_f32_dpp", 4);
  SKIPKV_DPP_STEP("v_max_f32_dpp", 2);
  SKIPKV_DPP_STEP("v_max_f32_dpp", 1);
  return v;
}
__device__ __forceinline__ float row16_sum_fast(float v) {
#define SKIPKV_DPP_ADD(N) v += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x120 + N, 0xf, 0xf, true))
  SKIPKV_DPP_ADD(8);
  SKIPKV_DPP_ADD(4);
  SKIPKV_DPP_ADD(2);
  SKIPKV_DPP_ADD(1);
#undef SKIPKV_DPP_ADD
  return v;
}
#undef SKIPKV_DPP_STEP

typedef __attribute__((__vector_size__(4 * sizeof(short)))) short i16x4;
typedef const __attribute__((address_space(4))) int32_t *ConstIntPtr;  // constant while the kernel runs: scalar loads

// Swizzle of 256-byte rows in LDS: the 16-byte piece p of row r is kept at piece position p ^ swz16(r).  Bits (r0, r1, r2, r3) of the row number go to
// bits (1, 2, 0, 3) of the piece number.  A permutation of bits, hence linear over XOR:
// swz(a ^ b) = swz(a) ^ swz(b).
__host__ __device__ constexpr int swz16(int r) { return ((r & 3) << 1) | ((r >> 2) & 1) | (r & 8); }

// Transposing LDS read: the 16 lanes of a group hand in 16 addresses of 4 consecutive 16-bit
// elements each, read as a 4 x 16 matrix (lanes 4i .. 4i+3 hold row i); lane n gets column n.
__device__ __forceinline__ i16x4 lds_read_tr16(uint32_t addr) {
  return __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) i16x4 *)(uintptr_t)addr);
}

// A uniform 64-bit address as a scalar register pair (the compiler may hold it in vector registers).
__device__ __forceinline__ uint64_t scalar64(const void *p_) {
  const uint64_t p = (uint64_t)(uintptr_t)p_;
  return ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(p >> 32)) << 32) | (uint32_t)__builtin_amdgcn_readfirstlane((int)p);
}
// Direct HBM -> LDS load with a scalar base and a 32-bit offset per lane.  The base may come straight from a
// v_readfirstlane or v_readlane: a vector-memory instruction may read such a register 5 wait states later at
// the earliest, and the compiler, which keeps that distance for its own instructions, does not look into this
// one; hence the s_nop.
__device__ __forceinline__ void load_to_lds_16_sbase(uint64_t sbase, uint32_t voff, void *wave_lds_base) {
  const uint32_t l = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char *)wave_lds_base;
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 4\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(l), "v"(voff), "s"(sbase) : "memory");
}

// The same for one dword per lane: 256 bytes at wave_lds_base + lane * 4.
__device__ __forceinline__ void load_to_lds_4_sbase(uint64_t sbase, uint32_t voff, void *wave_lds_base) {
  const uint32_t l = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char *)wave_lds_base;
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 4\n\tglobal_load_lds_dword %1, %2" ::"s"(l), "v"(voff), "s"(sbase) : "memory");
}

}  // namespace skipkv
