// Loads from memory straight into LDS and transposing reads out of it, for the kernels on the matrix cores.
#pragma once
#include "common.h"

namespace spes {

// raw buffer resource over `bytes` bytes from `base`: loads at byte offsets at or beyond `bytes` deliver zero
typedef __attribute__((ext_vector_type(4))) unsigned int rsrc_t;
__device__ __forceinline__ unsigned uniform(unsigned v) { return (unsigned)__builtin_amdgcn_readfirstlane((int)v); }
__device__ __forceinline__ rsrc_t make_rsrc(unsigned long base, unsigned bytes) {
  return rsrc_t{(unsigned)base, (unsigned)(base >> 32), bytes, 0x00020000u};
}
constexpr unsigned kOutOfRange = 0xfffffff0u;     // at or beyond any resource: operands have less than 2^31 elements of two bytes
// One load per wavefront of 64 x 16 bytes straight into LDS: lane l's bytes, from its own offset into the resource, land at
// the address in M0 + 16 l.  Written as assembly because the compiler makes every LDS read that may follow such a load wait for all of them;
// here the waits stand in the loop.  (The load has no result register, and address and resource are read when it issues.)  M0 is handed from
// the statement that sets it to the load as a value that lives in that register, so the compiler knows of both and keeps its own
// uses of M0 off it.  Between the two there has to be one instruction, and none of the compiler's copies: they stand in one straight run of
// code, and tests/test_lds_loads.py looks at every load that is built.
__device__ __forceinline__ unsigned set_lds_dest(unsigned lds) {
  unsigned m0;
  asm volatile("s_mov_b32 %0, %1" : "={m0}"(m0) : "s"(lds) : "memory");
  return m0;
}
__device__ __forceinline__ void load_to_lds(const rsrc_t& rs, unsigned lane_off, unsigned m0) {
  asm volatile("buffer_load_dwordx4 %0, %1, 0 offen lds" :: "v"(lane_off), "s"(rs), "{m0}"(m0) : "memory");
}
__device__ __forceinline__ void one_instruction() { asm volatile("s_nop 0" ::: "memory"); }
__device__ __forceinline__ void pin(unsigned& v) { asm volatile("" : "+s"(v)); }       // computed here and not elsewhere
// wait until at most N vector-memory operations of this wavefront are outstanding and all of its LDS reads have returned, then
// meet the block's other wavefronts
template <int N>
__device__ __forceinline__ void wait_and_meet() {
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" :: "n"(N) : "memory");
}

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;      // an operand fragment of a 16 x 16 x 32 MFMA
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) short s16x4;
typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
// Transposing LDS read.  Within each group of 16 lanes, lane s supplies the address of four consecutive 16-bit
// elements (think of them as row s of a 16 x 4 matrix); lane i receives column i%4 of rows i/4, i/4+4, i/4+8, i/4+12.
// With lane s pointing at [k0 + s/4][r0 + 4*(s%4)] of a [k][row] tile, lane i gets k0..k0+3 of row r0+i.
__device__ __forceinline__ uint2 lds_read_tr(const bf16_t* p) {
  const s16x4 v = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)p);
  return __builtin_bit_cast(uint2, v);
}
// Between a wavefront's writes to LDS of its own and its reads of what other lanes wrote: the hardware runs them in the order of the program,
// and the compiler, whatever types they have, leaves them in it.  No instruction.
__device__ __forceinline__ void wave_lds_order() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// Loads and stores of a lane's own through a buffer resource: zero, or nothing, at or beyond its end
__device__ __forceinline__ __amdgpu_buffer_rsrc_t tile_rsrc(unsigned long base, unsigned bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<void*>(base), 0, (int)bytes, 0x00020000);
}
__device__ __forceinline__ rsrc_t load16_once(__amdgpu_buffer_rsrc_t rs, unsigned off) {      // (with the non-temporal hint)
  return __builtin_amdgcn_raw_buffer_load_b128(rs, (int)off, 0, 2);
}
__device__ __forceinline__ float load4(__amdgpu_buffer_rsrc_t rs, unsigned off) {
  return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs, (int)off, 0, 0));
}
__device__ __forceinline__ void store16(__amdgpu_buffer_rsrc_t rs, unsigned off, const rsrc_t& v) {
  __builtin_amdgcn_raw_buffer_store_b128(v, rs, (int)off, 0, 0);
}
__device__ __forceinline__ void store4(__amdgpu_buffer_rsrc_t rs, unsigned off, float v) {
  __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v), rs, (int)off, 0, 0);
}

// 16 bytes per lane to base + lane_off with the non-temporal hint, nothing for a lane out of the `bytes` bytes
__device__ __forceinline__ void store_stream16(unsigned long base, unsigned bytes, unsigned lane_off, const uint4& v) {
  const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<void*>(base), 0, (int)bytes, 0x00020000);
  __builtin_amdgcn_raw_buffer_store_b128(rsrc_t{v.x, v.y, v.z, v.w}, rs, (int)lane_off, 0, 2);
}

}  // namespace spes
