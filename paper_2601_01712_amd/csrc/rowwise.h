// Row-wise work: row-table construction and the call's first LayerNorm.  One 64-lane wavefront owns one
// row of d = 64*E features; lane l holds features [l*E, l*E + E).
#pragma once

#include "common.h"

namespace relaygr {

constexpr int kRowsPerBlock = 4;  // wavefronts (rows) per 256-thread workgroup

// ---- row tables ------------------------------------------------------------------------------
// pstart / nstart: n_users + 1 row boundaries of the prefix rows and of the new rows.  The entry of row r:
// its user, kind, index inside the user's prefix / suffix / candidates, number of keys it sees in the
// [prefix | suffix] sequence, and its row in the caller's embedding array.
struct RowBuild {
  const UserDesc* users;
  const int32_t* pstart;
  const int32_t* nstart;
  int n_users, n_prows;
  int tile_rows, piece_tiles;   // 16-bit attention: rows of a work item, most key tiles of a piece of it (AttnCut::piece_all)
};

// u is the last user with start[u] <= r: the wavefront's lanes compare 64 users' starts at a time, or, for a batch that came as a
// kernel argument, scalar compares do.
template <bool INLINE>
__device__ __forceinline__ RowEntry row_entry(const RowBuild& rb, const InlineBatch& ib, int r, int lane) {
  int lo = -1;
  if constexpr (INLINE) {
    const int32_t* start = (r < rb.n_prows) ? ib.pstart : ib.nstart;
#pragma unroll
    for (int u = 0; u < kInlineUsers; ++u) lo += u < rb.n_users && start[u] <= r ? 1 : 0;
  } else {
    const int32_t* start = (r < rb.n_prows) ? rb.pstart : rb.nstart;
    for (int u0 = 0; u0 < rb.n_users; u0 += 64) {
      const int u = u0 + lane;
      lo += __builtin_popcountll(__builtin_amdgcn_ballot_w64(u < rb.n_users && start[min(u, rb.n_users)] <= r));
    }
  }
  const UserDesc& ud = INLINE ? ib.users[lo] : rb.users[lo];
  const int first = r < rb.n_prows ? (INLINE ? ib.pstart[lo] : rb.pstart[lo]) : (INLINE ? ib.nstart[lo] : rb.nstart[lo]);
  return row_entry_at(ud, lo, r < rb.n_prows, r - first, rb.tile_rows, rb.piece_tiles);
}

// ---- LayerNorm helpers -----------------------------------------------------------------------
template <int E>
__device__ __forceinline__ void ln_stats(const float (&v)[E], int d, float eps, float& mean, float& rstd) {
  float s = 0.f;
#pragma unroll
  for (int e = 0; e < E; ++e) s += v[e];
  mean = wave_sum(s) / (float)d;
  float q = 0.f;
#pragma unroll
  for (int e = 0; e < E; ++e) { float c = v[e] - mean; q += c * c; }
  rstd = rsqrtf(wave_sum(q) / (float)d + eps);
}

// E consecutive values of a row, as fp32, and back (runs of 16 bytes where there are that many).
template <typename T, int N> struct alignas(N * sizeof(T)) Run { T e[N]; };
template <typename T, int E>
__device__ __forceinline__ void ld_row_run(const T* src, float (&v)[E]) {
  constexpr int RUN = E * (int)sizeof(T) >= 16 ? 16 / (int)sizeof(T) : E;
#pragma unroll
  for (int c = 0; c < E; c += RUN) {
    const Run<T, RUN> b = *reinterpret_cast<const Run<T, RUN>*>(src + c);
#pragma unroll
    for (int i = 0; i < RUN; ++i) v[c + i] = Elem<T>::ld(&b.e[i]);
  }
}
template <typename T, int N>
__device__ __forceinline__ void st_run(T* dst, const float* v) {
  Run<T, N> b;
#pragma unroll
  for (int i = 0; i < N; ++i) Elem<T>::st(&b.e[i], v[i]);
  *reinterpret_cast<Run<T, N>*>(dst) = b;
}

// Writes a lane's E consecutive features [lane*E, lane*E+E) of row r, either row-major or into the
// MFMA-ordered panels the bf16 GEMM reads (E and 8 divide one another, so a lane's run never
// straddles a 16-byte fragment chunk unless it is made of whole chunks).
template <typename T, int E, bool PANEL>
__device__ __forceinline__ void store_row_run(T* __restrict__ out, int r, int lane, int d, const float (&v)[E]) {
  constexpr int RUN = E * (int)sizeof(T) >= 16 ? 16 / (int)sizeof(T) : E;
#pragma unroll
  for (int c = 0; c < E; c += RUN) st_run<T, RUN>(out + (PANEL ? panel_off(r, lane * E + c, d) : (size_t)r * d + lane * E + c), v + c);
}

// Unused token slots of a ragged last K/V tile must hold finite values: 0 * NaN would otherwise reach the accumulators
// through the masked-out keys.  The tiles concerned -- the last suffix tile of every user, and in the fp32 path the last
// tile of every computed prefix in every layer (the 16-bit projection writes those zeros itself) -- are cleared
// whole, before the first projection fills in their tokens, by extra workgroups of the call's first kernel: one per user, head
// and (prefix) layer, 16-byte stores.  (As launches of their own, one workgroup per user, they took 13 to 29 us of a call.)
struct TailClear {
  int row_blocks, jobs;      // workgroups that own rows; then `jobs` workgroups that clear
  int n_heads, dh, kv_layers;   // kv_layers: prefix layers to clear (0: none), then one more "layer" for the suffix
  void* sfx;                 // suffix K/V space; null: no suffix in this call
};
template <typename T>
__device__ __forceinline__ void clear_tail_tile(const TailClear& tc, const UserDesc& ud, int job) {
  const int head = job % tc.n_heads, layer = job / tc.n_heads % (tc.kv_layers + 1);
  T* tile;
  if (layer < tc.kv_layers) {
    if (ud.prow0 < 0 || ud.L % kTile == 0 || (layer > 0 && ud.kv_layer_stride == 0)) return;
    tile = const_cast<T*>(reinterpret_cast<const T*>(ud.kv)) + ud.kv_tile0 + (int64_t)(ud.L / kTile) * ud.kv_tile_stride + (int64_t)layer * ud.kv_layer_stride;
  } else {
    if (tc.sfx == nullptr || ud.nrow0 < 0 || ud.S % kTile == 0) return;
    tile = reinterpret_cast<T*>(tc.sfx) + ud.sfx_tile0 + (int64_t)(ud.S / kTile) * (2 * kTile * tc.dh * tc.n_heads);
  }
  uint4* dst = reinterpret_cast<uint4*>(tile + (int64_t)head * 2 * kTile * tc.dh);
  const int n16 = 2 * kTile * tc.dh * (int)sizeof(T) / 16;
  for (int i = threadIdx.x; i < n16; i += blockDim.x) dst[i] = make_uint4(0, 0, 0, 0);
}

// The rest of a small batch's descriptors -- what the later kernels read -- is fetched from the call's pinned staging slot
// by the last workgroups of the first kernel, kBlobChunk bytes each, beside the rows' work; each then tells the host in `flags`
// (pinned too) that its part of the slot has been read.  A copy command and the event behind it took 6 to 19 us of a call.
constexpr int kBlobChunk = 4096;
struct BlobCopy {
  const uint4* src;          // pinned host memory; null: a copy command has brought the descriptors
  uint4* dst;
  uint32_t* flags;
  uint32_t seq;
  int n16;                   // 16-byte pieces
};

// First kernel of a call.  A wavefront works out its row's table entry and writes it for the kernels that follow (the
// call's row tables are built here, not by a launch of their own), fetches the row from its embedding array, writes it to
// the fp32 residual stream x and its input LayerNorm (step 1 of the first layer) xh = LN(x; g, b) in the storage type; later
// layers get theirs from the layer tail.
template <typename T, int E, bool PANEL, bool INLINE>
__global__ __launch_bounds__(256) void ln_in_kernel(float* __restrict__ x, T* __restrict__ xh,
                                                    const T* __restrict__ gain, const T* __restrict__ offs,
                                                    const T* __restrict__ emb_prefix, const T* __restrict__ emb_suffix,
                                                    const T* __restrict__ emb_cand, RowTables rt, RowBuild rb, TailClear tc, BlobCopy bc,
                                                    InlineBatch ib, int n_rows, float eps) {
  const int d = 64 * E;
  if ((int)blockIdx.x >= tc.row_blocks) {
    const int job = (int)blockIdx.x - tc.row_blocks, chunk = job - tc.jobs;
    if (chunk < 0) {
      const int u = job / (tc.n_heads * (tc.kv_layers + 1));
      if constexpr (INLINE) clear_tail_tile<T>(tc, ib.users[u], job);
      else clear_tail_tile<T>(tc, rb.users[u], job);
    } else {
      const int i = chunk * (kBlobChunk / 16) + (int)threadIdx.x;
      if (i < bc.n16) bc.dst[i] = bc.src[i];
      __syncthreads();       // every thread has its piece: the slot is free
      if (threadIdx.x == 0) __hip_atomic_store(bc.flags + chunk, bc.seq, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    }
    return;
  }
  const int r = blockIdx.x * kRowsPerBlock + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (r >= n_rows) return;
  const int lane = threadIdx.x & 63;
  float v[E], gv[E], bv[E];
  ld_row_run<T, E>(gain + lane * E, gv);
  ld_row_run<T, E>(offs + lane * E, bv);
  const RowEntry e = row_entry<INLINE>(rb, ib, r, lane);
  if (lane == 0) { rt.user[r] = e.user; rt.kind[r] = e.kind; rt.idx[r] = e.idx; rt.lim[r] = e.lim; rt.src[r] = e.src; rt.parts[r] = e.parts; }
  if (e.kind == kRowPad) {   // keep filler rows finite
#pragma unroll
    for (int i = 0; i < E; ++i) v[i] = 0.f;
    store_row_run<T, E, PANEL>(xh, r, lane, d, v);
    return;
  }
  ld_row_run<T, E>((e.kind == kRowPrefix ? emb_prefix : e.kind == kRowSuffix ? emb_suffix : emb_cand) + (size_t)e.src * d + lane * E, v);
  store_row_run<float, E, false>(x, r, lane, d, v);
  float mean, rstd;
  ln_stats<E>(v, d, eps, mean, rstd);
#pragma unroll
  for (int i = 0; i < E; ++i) v[i] = (v[i] - mean) * rstd * gv[i] + bv[i];
  store_row_run<T, E, PANEL>(xh, r, lane, d, v);
}

}  // namespace relaygr
