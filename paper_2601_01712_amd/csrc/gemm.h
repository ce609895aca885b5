// What the projection kernels of fp32.h and gemm_bf16.h and the attention kernels share: the two 16-bit
// storage types, the column blocks of a launch and the workgroup order.
#pragma once

#include "common.h"

namespace relaygr {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));
typedef _Float16 f16x8_t __attribute__((ext_vector_type(8)));
typedef _Float16 f16x2_t __attribute__((ext_vector_type(2)));

// The two 16-bit storage types of the MFMA path (bf16: the benchmark's; fp16: the half precision the
// paper mentions as lowering the rank stage, Section 4.2).  Kernels are written against this
// interface: bit patterns in, fp32 out; pack2 rounds to nearest even; mfma is the 32x32x16 product
// of two 8-element fragments (any 16-byte type), mfma16 the 16x16x32 one.
struct Bf16 {
  using elem = __hip_bfloat16;
  static __device__ __forceinline__ float to_f32(uint16_t b) { return __uint_as_float(((uint32_t)b) << 16); }
  static __device__ __forceinline__ float of_word(uint32_t w, int i) { return __uint_as_float((i & 1) ? (w & 0xFFFF0000u) : (w << 16)); }
  static __device__ __forceinline__ uint32_t pack2(float a, float b) {
    f32x2_t v = {a, b};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2_t));     // one v_cvt_pk_bf16_f32
  }
  // c + a.lo * b.lo + a.hi * b.hi on two packed pairs, fp32 accumulate (v_dot2c_f32_bf16)
  static __device__ __forceinline__ float dot2(uint32_t a, uint32_t b, float c) {
    return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, a), __builtin_bit_cast(bf16x2_t, b), c, false);
  }
  template <typename A, typename B>
  static __device__ __forceinline__ f32x16_t mfma(A a, B b, f32x16_t c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, a), __builtin_bit_cast(bf16x8_t, b), c, 0, 0, 0);
  }
  template <typename A, typename B>
  static __device__ __forceinline__ f32x4_t mfma16(A a, B b, f32x4_t c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, a), __builtin_bit_cast(bf16x8_t, b), c, 0, 0, 0);
  }
};
struct F16 {
  using elem = __half;
  static __device__ __forceinline__ float to_f32(uint16_t b) { return (float)__builtin_bit_cast(_Float16, b); }
  static __device__ __forceinline__ float of_word(uint32_t w, int i) { return (float)__builtin_bit_cast(f16x2_t, w)[i & 1]; }
  static __device__ __forceinline__ uint32_t pack2(float a, float b) {
    f32x2_t v = {a, b};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, f16x2_t));      // one v_cvt_pk_f16_f32
  }
  static __device__ __forceinline__ float dot2(uint32_t a, uint32_t b, float c) {
    return __builtin_amdgcn_fdot2(__builtin_bit_cast(f16x2_t, a), __builtin_bit_cast(f16x2_t, b), c, false);
  }
  template <typename A, typename B>
  static __device__ __forceinline__ f32x16_t mfma(A a, B b, f32x16_t c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8_t, a), __builtin_bit_cast(f16x8_t, b), c, 0, 0, 0);
  }
  template <typename A, typename B>
  static __device__ __forceinline__ f32x4_t mfma16(A a, B b, f32x4_t c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8_t, a), __builtin_bit_cast(f16x8_t, b), c, 0, 0, 0);
  }
};
template <typename T> struct HalfOf { using type = Bf16; };
template <> struct HalfOf<__half> { using type = F16; };

// Operands read through a buffer descriptor: the address is a scalar base and offset plus one 32-bit offset per lane, with no 64-bit vector
// arithmetic per load, and what lies beyond `bytes` reads as zero.  load_lds copies 16 bytes per lane straight to LDS (lane l
// to dst + 16 l).  Unlike its global_load_lds form it does not make the compiler wait for ALL outstanding loads at the next
// use of a loaded register: the compiler takes that form for an access to both memories and cannot count past it.
struct BufferView {
  __amdgpu_buffer_rsrc_t rsrc;
  __device__ __forceinline__ BufferView(const void* base, uint32_t bytes)
      : rsrc(__builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, bytes, 0x00020000)) {}
  __device__ __forceinline__ uint4 load(int lane_off, int off) const {
    return __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(rsrc, lane_off, off, 0));
  }
  template <int IMM = 0>       // counts on both sides: dst + IMM takes off + IMM (below 4096)
  __device__ __forceinline__ void load_lds(void* dst, int lane_off, int off) const {
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (__attribute__((address_space(3))) void*)dst, 16, lane_off, off, IMM, 0);
  }
};

// Which output column blocks (of width d) a launch produces: block j of the launch is block
// blk[j] of the weight (f1 on last-layer prefix rows needs only v and k).
struct ColMap {
  int nblk;
  int blk[4];
  int d;   // block width
};

// Workgroups are dispatched round-robin over the 8 XCDs, each with its own L2.  Give each XCD a
// contiguous run of logical tiles (n fastest) so that the N-tiles sharing one A row-panel run on
// the same XCD close together in time.
__device__ __forceinline__ int xcd_remap(int id, int total) {
  int chunk = (total + 7) >> 3;
  return (id & 7) * chunk + (id >> 3);
}

}  // namespace relaygr
