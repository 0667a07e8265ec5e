// Shared pieces of the bf16 x bf16 -> fp32 GEMMs on the gfx950 matrix cores (the kernels are in
// gemm_bf16_slab.h and gemm_split3.h): the MFMA operand / accumulator vector types, the fp32 -> bf16
// rounding, and the pointer types and wait of the direct-to-LDS loads.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace asd {

typedef float v16f_b __attribute__((ext_vector_type(16)));   // accumulator of v_mfma_f32_32x32x16_bf16
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));      // its A / B operand: 8 consecutive k of a row
typedef int v16i_b __attribute__((ext_vector_type(16)));      // accumulator of v_mfma_i32_32x32x32_i8
typedef int v4i_b __attribute__((ext_vector_type(4)));        // its A / B operand: 16 consecutive k of a row, one byte each

typedef __attribute__((address_space(3))) void* lds_ptr_t;
typedef const __attribute__((address_space(1))) void* glb_ptr_t;

// 16 bytes a lane from memory into LDS: lane l's from base + off, its own, to dst + 16 l; base and dst are the wavefront's.  As
// a buffer load: a global one counts, for the compiler, as a flat access that may touch LDS, and while one is on its way --
// always, in a pipeline -- it waits for every outstanding LDS read wherever one is needed.  The base takes the whole address (its
// 48 bits, past which there is no memory), so an offset never leaves 32.
__device__ __forceinline__ void load_to_lds(const void* base, uint32_t off, void* dst) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(__builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, -1, 0x00027000),
                                           (lds_ptr_t)dst, 16, (int)off, 0, 0, 0);
}

template <int N>
__device__ __forceinline__ void wait_vmcnt() {
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// Barrier of a workgroup whose LDS stages are refilled by direct loads: this wavefront's reads of LDS are over (its data is
// in registers) before it says so.  (A bare s_barrier doesn't wait for them, and the compiler moves the products that would
// have to behind it; __syncthreads() would also wait for the loads in flight.)
__device__ __forceinline__ void lds_handover() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// Scheduling hints for an MFMA loop.
// `pairs` times {one MFMA, then `per` instructions of class `mask`}
template <int MASK, int PAIRS, int PER>
__device__ __forceinline__ void sched_pairs() {
  if constexpr (PAIRS > 0) {
    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
    __builtin_amdgcn_sched_group_barrier(MASK, PER, 0);
    sched_pairs<MASK, PAIRS - 1, PER>();
  }
}
template <int COUNT>
__device__ __forceinline__ void sched_mfma() {
  if constexpr (COUNT > 0) __builtin_amdgcn_sched_group_barrier(0x008, COUNT, 0);
}

// round to nearest even (finite inputs)
__device__ __forceinline__ uint16_t f32_to_bf16_rne(float f) {
  uint32_t u = __float_as_uint(f);
  u += 0x7fffu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}

__device__ __forceinline__ float bf16_to_f32(uint16_t b) { return __uint_as_float((uint32_t)b << 16); }
// lo term of a two-term activation: bf16(v - float(hi)) (the difference is exact in fp32)
__device__ __forceinline__ uint16_t bf16_lo(float v, uint16_t hi) { return f32_to_bf16_rne(v - bf16_to_f32(hi)); }

// hi and (lo_plane > 0) lo terms of four activations, to p and p + lo_plane
__device__ __forceinline__ void store_act4(uint16_t* p, int64_t lo_plane, float4 v) {
  const uint16_t h0 = f32_to_bf16_rne(v.x), h1 = f32_to_bf16_rne(v.y), h2 = f32_to_bf16_rne(v.z), h3 = f32_to_bf16_rne(v.w);
  *reinterpret_cast<uint2*>(p) = make_uint2((uint32_t)h0 | ((uint32_t)h1 << 16), (uint32_t)h2 | ((uint32_t)h3 << 16));
  if (lo_plane)
    *reinterpret_cast<uint2*>(p + lo_plane) =
        make_uint2((uint32_t)bf16_lo(v.x, h0) | ((uint32_t)bf16_lo(v.y, h1) << 16),
                   (uint32_t)bf16_lo(v.z, h2) | ((uint32_t)bf16_lo(v.w, h3) << 16));
}

}  // namespace asd
