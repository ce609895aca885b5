// Shared device/host declarations of the relay-race kernels (gfx950 only).
//
// Row space of one call.  Every token processed in a call is a "row":
//   [ prefix rows of the users whose prefix is computed in this call, user by user |
//     new rows of every user: that user's suffix tokens, then its candidates ]
// (sequence order of Section 2.3: long-term prefix, short-term / cross tokens, candidates).
// Each row carries its user, its kind, its index inside that segment, the number of keys of
// the user's ordered key sequence [prefix | suffix] it may see (lim), and where its embedding
// comes from.  A candidate additionally sees itself; that term never enters the key sequence.
//
// Cached K/V layout.  Keys are stored in tiles of 64 tokens.  One tile block holds, for every
// layer and head, a K tile (64 tokens x d_head) followed by a V tile (d_head x 64 tokens):
//     base(tile, layer, head) = tile*tile_stride + layer*layer_stride + head*128*dh
//     K element (token r, feature f) at base + KvLayout::k_off(r, f, dh)
//     V element (token r, feature f) at base + KvLayout::v_off(r, f, dh)      (includes the 64*dh K part)
// with tile_stride = n_layers*2*64*d and layer_stride = 2*64*d in the pool, and a single-layer
// form (tile_stride = 2*64*d, layer_stride = 0) in scratch for suffix tokens and for prefixes
// recomputed inside a ranking call.
//   fp32: K row-major [r][f]; V transposed [f][r].
//   bf16: both tiles are stored in the order the 32x32x16 MFMA consumes them, as 1 KiB fragments
//         of 64 lanes x 8 elements, so that a tile in HBM is byte-for-byte the LDS image and every
//         operand fetch is one linear, conflict-free 16-byte read per lane:
//         K fragment (kb, ks): lane (g, l32) holds token kb*32+l32, features ks*16+8g .. +7
//         V fragment (db, kb, m): lane (g, l32) holds feature db*32+l32 and the 8 tokens
//                    kb*32+16m+4g+{0..3}, kb*32+16m+8+4g+{0..3} -- the key order in which the
//                    first product's accumulator hands P to the second product.
#pragma once

#include <hip/hip_runtime.h>
#include <hip/hip_bf16.h>
#include <hip/hip_fp16.h>
#include <stdint.h>

#include "plan.h"

namespace relaygr {

// The descriptors of a batch of few users, small enough to be a kernel argument: the call's first kernel then needs no copy
// to have run before it (see BlobCopy).  The argument is the faster one at every number of users that it could hold (the 4 KiB
// of kernel arguments are full at a little over 40): us a call with it and with the copy command, d = 256, 4 layers, 512 keys and
// 32 candidates a user, 4 users 75 / 80, 16 83 / 86, 24 87 / 91, 40 99 / 103.  So this line is no crossover: it is where the
// argument, which the first launch of every call carries whole, is 1.4 KiB.
constexpr int kInlineUsers = 16;
struct InlineBatch {
  UserDesc users[kInlineUsers];
  int32_t pstart[kInlineUsers + 1], nstart[kInlineUsers + 1];
};

struct RowTables {
  int32_t* user;
  int32_t* kind;
  int32_t* idx;    // index inside the user's segment of that kind
  int32_t* lim;    // keys of [prefix | suffix] visible to this row
  int32_t* src;    // row in the embedding array of its kind
  int32_t* parts;  // attention partial sums of this row: every layer but the last | last layer << 8
};

template <typename T> struct KvLayout;
template <> struct KvLayout<float> {
  static __host__ __device__ __forceinline__ int k_off(int r, int f, int dh) { return r * dh + f; }
  static __host__ __device__ __forceinline__ int v_off(int r, int f, int dh) { return kTile * dh + f * kTile + r; }
};
// both 16-bit storage types: MFMA fragment order
struct KvLayout16 {
  static __host__ __device__ __forceinline__ int k_off(int r, int f, int dh) {
    int kb = r >> 5, l32 = r & 31, ks = f >> 4, g = (f >> 3) & 1, j = f & 7;
    return ((kb * (dh >> 4) + ks) * 64 + g * 32 + l32) * 8 + j;
  }
  static __host__ __device__ __forceinline__ int v_off(int r, int f, int dh) {
    int db = f >> 5, l32 = f & 31, kb = r >> 5, m = (r >> 4) & 1, w = r & 15;
    int g = (w >> 2) & 1, j = ((w >> 3) << 2) | (w & 3);
    return kTile * dh + (((db * 2 + kb) * 2 + m) * 64 + g * 32 + l32) * 8 + j;
  }
};
template <> struct KvLayout<__hip_bfloat16> : KvLayout16 {};
template <> struct KvLayout<__half> : KvLayout16 {};

// ---- element access in the two storage types ------------------------------------------------
template <typename T> struct Elem;
template <> struct Elem<float> {
  static __device__ __forceinline__ float ld(const float* p) { return *p; }
  static __device__ __forceinline__ void st(float* p, float v) { *p = v; }
};
template <> struct Elem<__hip_bfloat16> {
  static __device__ __forceinline__ float ld(const __hip_bfloat16* p) {
    return __uint_as_float(((uint32_t)(*reinterpret_cast<const uint16_t*>(p))) << 16);
  }
  static __device__ __forceinline__ void st(__hip_bfloat16* p, float v) { *p = __float2bfloat16(v); }
};

template <> struct Elem<__half> {
  static __device__ __forceinline__ float ld(const __half* p) { return __half2float(*p); }
  static __device__ __forceinline__ void st(__half* p, float v) { *p = __float2half(v); }
};

__device__ __forceinline__ float bf16_bits_to_float(uint16_t b) { return __uint_as_float(((uint32_t)b) << 16); }
__device__ __forceinline__ uint16_t float_to_bf16_bits(float v) {
  __hip_bfloat16 h = __float2bfloat16(v);
  return *reinterpret_cast<uint16_t*>(&h);
}

// SiLU(t) = t / (1 + exp(-t)), fp32, accurate form (fp32 path and row-wise kernels).
__device__ __forceinline__ float silu_f32(float t) { return t / (1.0f + __expf(-t)); }
// The same through the hardware exp2 and reciprocal approximations (about 1 ulp each): bf16 path.
__device__ __forceinline__ float silu_fast(float t) {
  return t * __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(t * -1.4426950408889634f));
}

// element offset of (row, k) in an array of MFMA-ordered panels of row length K: a panel is 128
// rows, stored as 1 KiB fragments [k/16][(row%128)/32][lane][8], lane = ((k/8)%2)*32 + row%32
__host__ __device__ __forceinline__ size_t panel_off(int row, int k, int K) {
  int panel = row >> 7, rb = (row >> 5) & 3, l32 = row & 31, ks = k >> 4, g = (k >> 3) & 1, j = k & 7;
  return ((size_t)panel * (K >> 4) + ks) * 2048 + (size_t)rb * 512 + (g * 32 + l32) * 8 + j;
}

// Row octets: q, and the new rows' k and v, of the 16-bit SiLU form.  Eight rows at a time, in them the 16-byte chunks of eight features, each of
// the eight rows: [row/8][feature/8][row%8][feature%8].  The last octet of an array holds as many rows as are left, so that the array is as large as
// in row-major order.  `chunk`: feature / 8.  Whoever takes a chunk of 32 consecutive rows (an operand of the attention's product) reads 128 bytes
// in a run, where row-major order gives a memory line for every row.  us a call, d = 512, row-major / octets: one user of 4096 keys and 512 candidates 238 /
// 232, of 800 and 100 183.4 / 177.8; eight of 2048 and 272 new rows at d = 256 126.9 / 122.8.  With at most 32 rows a user one of a workgroup's four
// wavefronts has rows, and there is little to gain: seven of 800 and 32 177.9 / 179.0, 14 of 300 and 32 175.6 / 177.3 (180.7 and 181.3 with the addresses worked
// out in 64 bits for each lane).
__device__ __forceinline__ int octet_step(int row, int n_rows) { return min(8, n_rows - (row & ~7)) * 8; }     // elements between a row's chunks
__device__ __forceinline__ int octet_off(int row, int d) { return (row & ~7) * d + (row & 7) * 8; }  // its chunk 0 (row: in a tile, from an octet's first row on)

// Barrier for data that went through LDS only: unlike __syncthreads() it does not wait for global stores and loads in flight.
__device__ __forceinline__ void lds_barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));
// (the address-space forms are for pointers that were themselves loaded from memory: the compiler cannot tell that those are
// global addresses and would use flat stores, which also hold up the LDS counter)
typedef __attribute__((address_space(1))) u32x4_t gu32x4_t;
__device__ __forceinline__ gu32x4_t* as_global16(uint16_t* p) { return (gu32x4_t*)p; }
// 16 bytes from LDS, as a vector and to be kept one: behind a direct load to LDS the compiler waits for ALL outstanding loads before it
// reads LDS as a struct like uint4 (the reads become those of its members, which it takes for what the load may have written), so that
// a ring of stages in flight is emptied at every step.
__device__ __forceinline__ u32x4_t lds_read16(const uint16_t* p) { return *reinterpret_cast<const u32x4_t*>(p); }

// Sum over the wavefront, in every lane, adding lane i to lane i ^ 32, then ^ 16, ^ 8, ^ 4, ^ 2, ^ 1, on the vector ALU: the
// halves and the 16-lane rows change places (v_permlane32_swap, v_permlane16_swap), and inside a row a rotation by 8 is lane ^ 8, after
// which values repeat every 8 lanes and a rotation by 4 is lane ^ 4, and so on.
template <int CTRL>
// (v + v of the lane the DPP control selects: no LDS crossbar round trip)
__device__ __forceinline__ float dpp_add(float v) {
  return v + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, true));
}
__device__ __forceinline__ float wave_sum(float v) {
  typedef unsigned int u2 __attribute__((ext_vector_type(2)));
  u2 h = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = __uint_as_float(h[0]) + __uint_as_float(h[1]);
  h = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = __uint_as_float(h[0]) + __uint_as_float(h[1]);
  v = dpp_add<0x128>(v);
  v = dpp_add<0x124>(v);
  v = dpp_add<0x122>(v);
  return dpp_add<0x121>(v);
}

// Sum over the four lanes l, l ^ 16, l ^ 32, l ^ 48, in each of them.
__device__ __forceinline__ float rows4_sum(float v) {
  typedef unsigned int u2 __attribute__((ext_vector_type(2)));
  u2 h = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = __uint_as_float(h[0]) + __uint_as_float(h[1]);
  h = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return __uint_as_float(h[0]) + __uint_as_float(h[1]);
}

// Sum over each group of 2, 4, 8, 16 consecutive lanes, left in every lane of the group:
// quad_perm [1,0,3,2], quad_perm [2,3,0,1], row_half_mirror, row_mirror.
__device__ __forceinline__ float lanes2_sum(float v) { return dpp_add<0xB1>(v); }
__device__ __forceinline__ float lanes4_sum(float v) { return dpp_add<0x4E>(lanes2_sum(v)); }
__device__ __forceinline__ float lanes8_sum(float v) { return dpp_add<0x141>(lanes4_sum(v)); }
__device__ __forceinline__ float lanes16_sum(float v) { return dpp_add<0x140>(lanes8_sum(v)); }
// Sum over each half of the wavefront, in every lane of the half.
__device__ __forceinline__ float lanes32_sum(float v) {
  v = lanes16_sum(v);
  const int b = __float_as_int(v);
  const float lo = __int_as_float(__builtin_amdgcn_readlane(b, 0)) + __int_as_float(__builtin_amdgcn_readlane(b, 16));
  const float hi = __int_as_float(__builtin_amdgcn_readlane(b, 32)) + __int_as_float(__builtin_amdgcn_readlane(b, 48));
  return (threadIdx.x & 32) ? hi : lo;
}
// Sum over the wavefront, in every lane: 16-lane sums by DPP, the four of them through scalar registers.
__device__ __forceinline__ float wave_sum_dpp(float v) {
  v = lanes16_sum(v);
  const int b = __float_as_int(v);
  return (__int_as_float(__builtin_amdgcn_readlane(b, 0)) + __int_as_float(__builtin_amdgcn_readlane(b, 16))) +
         (__int_as_float(__builtin_amdgcn_readlane(b, 32)) + __int_as_float(__builtin_amdgcn_readlane(b, 48)));
}

}  // namespace relaygr
