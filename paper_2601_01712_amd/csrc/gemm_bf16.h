// bf16 projection GEMMs on the 32x32x16 MFMA: C[tokens, features] = A[tokens, K] * W[features, K]^T
// with the layer's pointwise work fused in (steps 2 and 4 of a layer):
//   f1: SiLU(xh W1^T + b1) split into u | v | q | k and written where the next kernel wants it:
//       u, q (and k, v of candidate rows) row-major; k, v of prefix / suffix rows straight into the
//       K/V tile layout of the pool or of scratch;
//   f2: x <- x + y W2^T + b2 on the fp32 residual stream.
//
// Operand layout.  Both operands live in global memory already in MFMA fragment order ("panels"):
// a panel is 128 rows x K, stored as 1 KiB fragments [k-step ks = k/16][row block rb = (row%128)/32]
// [lane][8], lane (g, l32) holding row rb*32 + l32, k = ks*16 + 8g .. +7.  The LayerNorm kernels
// write activations that way and the weights are re-packed once per context.  A k-tile of a panel
// is therefore one contiguous run of bytes that is copied HBM -> LDS with direct 16-byte-per-lane
// loads (fully coalesced, no registers), lands as the exact LDS image the MFMA reads, and every
// operand fetch is one linear ds_read_b128 with no bank conflicts.  Because token and feature
// fragments have the same shape, either can be the MFMA's row operand: "feature-major" products
// leave each lane with 4 consecutive features of one token (what row-major outputs and K tiles
// want), "token-major" products leave 4 consecutive tokens of one feature (exactly a V-tile
// fragment, and what the fp32 residual update wants).
#pragma once

#include <type_traits>

#include "common.h"
#include "gemm.h"
#include "launch_rules.h"

namespace relaygr {

constexpr int kPanelRows = 128;
constexpr int kGemmKTile = 32;          // k per main-loop step (2 MFMA k-steps)
constexpr int kPrefixRowAlign = 256;    // prefix rows of a user start at a multiple of this in the row space

// Re-packs a row-major [N, K] weight into panels.
__global__ void pack_weight_kernel(const uint16_t* __restrict__ w, uint16_t* __restrict__ packed, int N, int K) {
  int idx = blockIdx.x * blockDim.x + threadIdx.x;   // one 8-element chunk per thread
  int chunks_per_row = K >> 3;
  if (idx >= N * chunks_per_row) return;
  int n = idx / chunks_per_row, kc = idx - n * chunks_per_row;
  uint4 v = *reinterpret_cast<const uint4*>(w + (size_t)n * K + kc * 8);
  *reinterpret_cast<uint4*>(packed + panel_off(n, kc * 8, K)) = v;
}

// Wavefronts of a layer-tail workgroup, and the 16-feature blocks of W2 that each of them multiplies by.
constexpr int tail_waves(int d) { return d <= 128 ? 4 : 8; }
constexpr int tail_blocks(int d) { return d / 16 / tail_waves(d); }

// Re-packs a row-major [d, d] weight for the layer tail: 1 KiB fragments of 16 rows x 32 k in the 16x16x32 MFMA's operand order
// (lane = ((k/8)%4)*16 + n%16), in the order in which a wavefront reads its tail_blocks(d) blocks: [wavefront][k/32][block][lane][8].
// (With [block][k/32] the wavefronts of a workgroup were at the same few of an L2's channels at any time, at d = 512 every 16 KiB.)
__global__ void pack_weight16_kernel(const uint16_t* __restrict__ w, uint16_t* __restrict__ packed, int d) {
  int idx = blockIdx.x * blockDim.x + threadIdx.x;   // one 8-element chunk per thread
  int chunks_per_row = d >> 3;
  if (idx >= d * chunks_per_row) return;
  int n = idx / chunks_per_row, kc = idx - n * chunks_per_row;
  uint4 v = *reinterpret_cast<const uint4*>(w + (size_t)n * d + kc * 8);
  const int fb = tail_blocks(d), blk = n >> 4;
  *reinterpret_cast<uint4*>(packed + (((size_t)(blk / fb * (d >> 5) + (kc >> 2)) * fb + blk % fb) * 64 + (kc & 3) * 16 + (n & 15)) * 8) = v;
}

// ---- main loop ----------------------------------------------------------------------------------
// Workgroup tile: 64*TM tokens x 64*TN features, 4 wavefronts as 2 x 2, each owning TM x TN blocks of
// 32 x 32.  LDS holds a ring of NSTAGE stages of [token pieces | feature pieces], a piece being one
// 1 KiB fragment; NSTAGE-1 stages are in flight while one is consumed, because with K of a few
// hundred a tile is short and the ramp of its operand stream would otherwise dominate it.
template <int TM, int TN, int NSTAGE>
struct GemmTile {
  static constexpr int BMt = 64 * TM, BNf = 64 * TN;
  static constexpr int TOK_PIECES = (BMt / 32) * 2, FEAT_PIECES = (BNf / 32) * 2;   // per stage (2 k-steps)
  static constexpr int PIECES = TOK_PIECES + FEAT_PIECES;
  static constexpr int STAGE = PIECES * 512;   // elements
  static constexpr int LDS_ELEMS = NSTAGE * STAGE;
  static constexpr int LOADS_PER_WAVE = PIECES / 4;
  static_assert(PIECES % 4 == 0, "pieces are dealt evenly to the 4 wavefronts");
  static_assert(TOK_PIECES % 4 == 0, "and a wavefront's n-th piece is the same operand's in all of them");
  static_assert((TM == 1 || TM % 2 == 0) && (TN == 1 || TN % 2 == 0), "a tile is half a 128-row panel or whole panels");
  // piece q of an operand of `blocks` 64-row blocks whose tile starts at row r0: byte offset from its first panel (K rows of 4 KiB per 16 k)
  static __device__ __forceinline__ int piece_off(int blocks, int q, int r0, int KS) {
    const int panel = blocks >= 2 ? q >> 3 : 0, ksl = blocks >= 2 ? (q >> 2) & 1 : q >> 1, rb = blocks >= 2 ? q & 3 : ((r0 >> 5) & 3) + (q & 1);
    return (panel * KS + ksl) * 4096 + rb * 1024;
  }
  static __device__ __forceinline__ int frag(int blocks, int rb, int ksl) { return (blocks >= 2 ? ((rb >> 2) * 2 + ksl) * 4 + (rb & 3) : ksl * 2 + rb) * 512; }
};

// start() asks for the first stages; run() waits for them one by one.  What a kernel needs besides the operands it loads between
// the two or before.  KT > 0: K is 32 * KT and the steps are unrolled, with the exact number of younger stages in each wait; KT <= NSTAGE:
// the operands are asked for whole.  KT = 0: K is known at run time.
// FEATURE_MAJOR: features are the MFMA row operand (lane = token column, 4-feature runs per lane).
template <typename H, int TM, int TN, int NSTAGE, int KT>
struct GemmLoop {
  using G = GemmTile<TM, TN, NSTAGE>;
  static constexpr bool WHOLE = KT > 0 && KT <= NSTAGE;
  static constexpr int AHEAD = WHOLE ? KT : NSTAGE - 1;     // stages asked for before the first step
  const char *a, *w;          // first panel of the tile's rows of each operand
  uint16_t* lds;
  int K, lane, wave, src[G::LOADS_PER_WAVE];

  __device__ __forceinline__ GemmLoop(const uint16_t* A, const uint16_t* W, int K_, int m0, int n0, uint16_t* lds_)
      : a(reinterpret_cast<const char*>(A + (size_t)(m0 >> 7) * (K_ >> 4) * 2048)),
        w(reinterpret_cast<const char*>(W + (size_t)(n0 >> 7) * (K_ >> 4) * 2048)),
        lds(lds_), K(K_), lane(threadIdx.x & 63), wave(__builtin_amdgcn_readfirstlane(threadIdx.x >> 6)) {
#pragma unroll
    for (int i = 0; i < G::LOADS_PER_WAVE; ++i) {
      const int p = wave + 4 * i;
      src[i] = 4 * i < G::TOK_PIECES ? G::piece_off(TM, p, m0, K >> 4) : G::piece_off(TN, p - G::TOK_PIECES, n0, K >> 4);
    }
  }
  __device__ __forceinline__ void issue(int kt, int slot) {
#pragma unroll
    for (int i = 0; i < G::LOADS_PER_WAVE; ++i) {
      // (scalar base and offset, one 32-bit offset per lane; not the buffer form, behind which the compiler waits for all stages
      // wherever LDS is read)
      const char* s = (4 * i < G::TOK_PIECES ? a : w) + (src[i] + kt * 8192);
      __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(s + (uint32_t)(lane * 16)),
                                       (__attribute__((address_space(3))) void*)(lds + slot * G::STAGE + (wave + 4 * i) * 512), 16, 0, 0);
    }
  }
  __device__ __forceinline__ void start() {
#pragma unroll
    for (int s = 0; s < AHEAD; ++s)
      if (KT > 0 ? s < KT : s < K / kGemmKTile) issue(s, s);
  }
  template <bool FEATURE_MAJOR>
  __device__ __forceinline__ void step(int slot, f32x16_t (&acc)[TM][TN]) {
    const int wm = wave >> 1, wn = wave & 1;
    const uint16_t* tokp = lds + slot * G::STAGE + lane * 8;
    const uint16_t* featp = tokp + G::TOK_PIECES * 512;
    // fetch the fragments of both k-steps first, so that the second set's LDS latency hides under
    // the first set's MFMAs
    u32x4_t tf[2][TM], ff[2][TN];
#pragma unroll
    for (int ksl = 0; ksl < 2; ++ksl) {
#pragma unroll
      for (int i = 0; i < TM; ++i) tf[ksl][i] = lds_read16(tokp + G::frag(TM, wm * TM + i, ksl));
#pragma unroll
      for (int j = 0; j < TN; ++j) ff[ksl][j] = lds_read16(featp + G::frag(TN, wn * TN + j, ksl));
    }
    __builtin_amdgcn_sched_barrier(0);   // keep all the reads ahead of the MFMAs
#pragma unroll
    for (int ksl = 0; ksl < 2; ++ksl)
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
          acc[i][j] = FEATURE_MAJOR ? H::mfma(ff[ksl][j], tf[ksl][i], acc[i][j]) : H::mfma(tf[ksl][i], ff[ksl][j], acc[i][j]);
  }
  template <int YOUNGER>      // this stage must have landed, YOUNGER ones may stay in flight
  __device__ __forceinline__ void wait() {
    // (a bare s_barrier: __syncthreads() would also make the compiler wait for every outstanding load,
    // i.e. for the stages that are meant to stay in flight)
    // (and this wavefront's reads of the stage before are done: its slot is refilled next)
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(YOUNGER * G::LOADS_PER_WAVE) : "memory");
    __builtin_amdgcn_s_barrier();   // so are every wavefront's
    asm volatile("" ::: "memory");
  }
  template <bool FEATURE_MAJOR, int T>
  __device__ __forceinline__ void steps(f32x16_t (&acc)[TM][TN]) {
    if constexpr (T < KT) {
      wait<(WHOLE || KT - 1 - T < NSTAGE - 2 ? KT - 1 - T : NSTAGE - 2)>();
      if constexpr (!WHOLE && T + NSTAGE - 1 < KT) issue(T + NSTAGE - 1, (T + NSTAGE - 1) % NSTAGE);
      step<FEATURE_MAJOR>(T % NSTAGE, acc);
      steps<FEATURE_MAJOR, T + 1>(acc);
    }
  }
  template <bool FEATURE_MAJOR>
  __device__ __forceinline__ void run(f32x16_t (&acc)[TM][TN]) {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;
    if constexpr (KT > 0) {
      steps<FEATURE_MAJOR, 0>(acc);
    } else {
      const int n_kt = K / kGemmKTile;
      int slot = 0;
      for (int kt = 0; kt < n_kt; ++kt) {
        if (kt + NSTAGE - 2 < n_kt) wait<NSTAGE - 2>();
        else wait<0>();                 // near the end fewer are outstanding: wait for all of them
        if (kt + NSTAGE - 1 < n_kt) issue(kt + NSTAGE - 1, slot == 0 ? NSTAGE - 1 : slot - 1);
        step<FEATURE_MAJOR>(slot, acc);
        slot = (slot == NSTAGE - 1) ? 0 : slot + 1;
      }
    }
    lds_barrier();   // every wavefront is done reading LDS: the epilogue may reuse it
  }
};

// ---- f1 -------------------------------------------------------------------------------------------
struct F1Params {
  const uint16_t* A;        // xh panels
  const uint16_t* W;        // packed W1 [4d, d]
  const uint16_t* bias;     // [4d]
  uint16_t* u; uint16_t* q; uint16_t* knew; uint16_t* vnew; uint16_t* sfx;
  const UserDesc* users;
  RowTables rt;
  int d, dh, n_prows, layer, row_begin, row_end, n_mtiles;
  ColMap cm;
  float q_mul;
  int octets;               // q, and k and v of new rows, leave in row octets (octet_off) and not row-major
  int stream_out;           // weight-stationary kernel: outputs leave with streaming stores (launches that write far more than L2 holds)
};

// Streaming stores (the `nt` hint): for kernel outputs that nothing in the same launch reads back.  A plain store
// allocates its line in the XCD's L2, and a launch that writes tens of megabytes pushes out the operand lines the
// workgroups of that XCD share (token panels, weight slices, K/V tiles), which are then fetched again and again
// from the memory side; marked non-temporal, the output lines leave L2 first.  Measured on the projection GEMM
// at 65 536 rows: 225 us with plain stores, 152 us with these (150 us with no stores at all).  Not a general win:
// a workgroup ends only when its stores are acknowledged, which a streaming store is later than a cached one --
// the attention kernel's partial sums and the layer tail's outputs, written once at the end of short-lived
// workgroups, got 13 % and 5-17 % slower with it and keep plain stores.
__device__ __forceinline__ void st_out(uint16_t* dst, uint4 v, int stream) {
  gu32x4_t* g = as_global16(dst);
  if (stream) __builtin_nontemporal_store(u32x4_t{v.x, v.y, v.z, v.w}, g);
  else *g = u32x4_t{v.x, v.y, v.z, v.w};
}

constexpr int kF1TM = 4, kF1TN = 2, kF1Stages = 3;   // 256 tokens x 128 features per workgroup
// KT: 32-wide steps of K, 0: known at run time (the big tile).
template <typename H, int TM, int TN, int NSTAGE, int KT>
__global__ __launch_bounds__(256, TM == 4 ? 2 : NSTAGE == 3 ? 3 : 1) void f1_gemm_bf16_kernel(F1Params p) {
  constexpr int ROWS = 64 * TM;                  // tokens per workgroup tile
  constexpr int kStageLd = 64 * TN + 8;          // epilogue staging row stride (elements)
  using G = GemmTile<TM, TN, NSTAGE>;
  constexpr int LDS_ELEMS = (G::LDS_ELEMS > ROWS * kStageLd) ? G::LDS_ELEMS : ROWS * kStageLd;
  __shared__ __attribute__((aligned(16))) uint16_t lds[LDS_ELEMS];

  const int d = KT > 0 ? KT * kGemmKTile : p.d;
  const int ntiles_per_blk = d / G::BNf;
  const int n_ntiles = p.cm.nblk * ntiles_per_blk;
  const int total = p.n_mtiles * n_ntiles;
  const int logical = xcd_remap(blockIdx.x, total);
  if (logical >= total) return;
  // an XCD's workgroups take neighbouring tiles: of one row tile, or, in launches of few rows, of one column tile, so that
  // each XCD fetches its part of W1 and not all of it
  constexpr bool by_cols = TM < 4;
  const int mt = by_cols ? logical % p.n_mtiles : logical / n_ntiles, nt = by_cols ? logical / p.n_mtiles : logical - mt * n_ntiles;
  const int m0 = p.row_begin + mt * G::BMt;
  const int blk = p.cm.blk[nt / ntiles_per_blk];           // 0 u, 1 v, 2 q, 3 k
  const int c0 = (nt % ntiles_per_blk) * G::BNf;            // first feature inside the block
  const int n0 = blk * d + c0;

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1, l32 = lane & 31, g = lane >> 5;
  const int dh = p.dh, dh_sh = 31 - __builtin_clz(dh);   // d_head is a power of two
  // A tile of prefix rows is one user's consecutive prefix positions starting at a multiple of 256
  // (row-space alignment), possibly followed by padding rows.
  const bool prefix_tile = m0 < p.n_prows;
  const int pos0 = prefix_tile ? p.rt.idx[m0] : 0;         // a multiple of 64
  const int tile_user = prefix_tile ? p.rt.user[m0] : 0;
  if (prefix_tile && p.rt.kind[m0] == kRowPad) return;     // filler behind the user's last K/V tile

  // In the store phase a thread owns 16-byte chunk fc of rows t0 + RPP*it of the tile.  Neighbouring threads take neighbouring chunks of a row where
  // rows are stored whole, and one chunk of the eight rows of an octet where these lie side by side (row octets, K tiles).  The kinds of new rows (candidate or suffix) and the biases are asked for first, so that run()'s waits, which count younger loads, need not count them.
  constexpr int CH = 8 * TN, RPP = 256 / CH, ITS = ROWS / RPP;   // chunks of a row, rows per pass of the store phase, passes
  const bool by_kind = (blk == 1 || blk == 3) && !prefix_tile;
  const bool octets = p.octets && (blk == 2 || by_kind), rows_first = octets || (blk == 3 && prefix_tile);
  const int rsh = rows_first ? 3 : 0;                        // (a scalar: selected by lane, it would be two branches ahead of the first loads)
  const int t0 = (tid >> rsh) / CH << rsh | (tid & ((1 << rsh) - 1)), fc = (tid >> rsh) % CH;
  int kinds[ITS];
#pragma unroll
  for (int it = 0; it < ITS; ++it) kinds[it] = kRowCand;
  if (by_kind) {
#pragma unroll
    for (int it = 0; it < ITS; ++it) kinds[it] = p.rt.kind[min(m0 + t0 + RPP * it, p.row_end - 1)];
  }
  uint2 bias[TN][4];
#pragma unroll
  for (int j = 0; j < TN; ++j)
#pragma unroll
    for (int e4 = 0; e4 < 4; ++e4) bias[j][e4] = *reinterpret_cast<const uint2*>(p.bias + n0 + wn * (32 * TN) + j * 32 + 8 * e4 + 4 * g);
  asm volatile("" ::: "memory");
  GemmLoop<H, TM, TN, NSTAGE, KT> loop(p.A, p.W, d, m0, n0, lds);
  loop.start();                                             // before everything else that the tile needs
  // Where this thread's chunks go, worked out while the tiles are on their way (the compiler would load the pointers behind the product, a round trip
  // before the first store: 608 workgroups of 64 x 128 tiles 14.35 / 14.19 us).  Row-major: octets of one row.  A pass is whole octets, so that a
  // thread's places are one row stride apart.
  // (u and q of filler rows are written too: nothing reads them, and a filler row's inputs are zeros)
  const int in_octet = octets ? 7 : 0;
  uint32_t at0 = (t0 & ~in_octet) * d * 2 + (t0 & in_octet) * 16 + (c0 / 8 + fc) * (in_octet + 1) * 16;
  int n_rows = p.row_end - m0;
  uint16_t* rows_out = blk == 0 ? p.u + (size_t)m0 * d : blk == 2 ? p.q + (size_t)m0 * d : (blk == 3 ? p.knew : p.vnew) + ((int64_t)m0 - p.n_prows) * d;
  asm volatile("" : "+v"(at0), "+s"(n_rows), "+s"(rows_out));

  f32x16_t acc[TM][TN];

  if (blk == 1 && prefix_tile) {
    // ---- V of prefix rows: token-major product; the accumulator of a 32-token x 32-feature block
    // is, lane for lane, two V-tile fragments (m = 0, 1), stored as 1 KiB contiguous runs.
    loop.template run<false>(acc);
    const UserDesc& tud = p.users[tile_user];               // (read here, not before the product: it is two more round trips)
    const int L = tud.L, Lceil = (L + kTile - 1) / kTile * kTile;
    const int64_t kv_stride = tud.kv_tile_stride;
    uint16_t* kvb = reinterpret_cast<uint16_t*>(const_cast<void*>(tud.kv)) + tud.kv_tile0 + (int64_t)(pos0 >> 6) * kv_stride +
                    (int64_t)p.layer * tud.kv_layer_stride;  // the K/V tile of the first 64 rows
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const int c = c0 + wn * (32 * TN) + j * 32;                  // first feature of this 32-feature block
      const int head = c >> dh_sh, db = (c - (head << dh_sh)) >> 5;
      const float bias = H::to_f32(p.bias[n0 + wn * (32 * TN) + j * 32 + l32]);
#pragma unroll
      for (int i = 0; i < TM; ++i) {
        const int tok0 = pos0 + wm * (32 * TM) + i * 32;    // first token of this 32-token block
        if (tok0 >= Lceil) continue;
        const int kb = (tok0 >> 5) & 1;
        uint16_t* frag = kvb + (int64_t)((tok0 - pos0) >> 6) * kv_stride + head * 2 * kTile * dh + kTile * dh;
#pragma unroll
        for (int m = 0; m < 2; ++m) {
          uint32_t w[4];
#pragma unroll
          for (int h = 0; h < 2; ++h) {
            const int e4 = 2 * m + h;
            float v[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              const int tok = tok0 + 8 * e4 + 4 * g + r;
              float val = silu_fast(acc[i][j][4 * e4 + r] + bias);
              v[r] = tok < L ? val : 0.f;                    // the ragged tail of the last tile holds zeros
            }
            w[2 * h] = H::pack2(v[0], v[1]);
            w[2 * h + 1] = H::pack2(v[2], v[3]);
          }
          st_out(frag + (((db * 2 + kb) * 2 + m) * 64 + lane) * 8, make_uint4(w[0], w[1], w[2], w[3]), 0);
        }
      }
    }
    return;
  }

  // ---- everything else: feature-major product, staged through LDS as [token][feature] so that
  // every global store is a 16-byte chunk of 8 consecutive features of one token.
  loop.template run<true>(acc);
  const float mul = (blk == 2) ? p.q_mul : 1.0f;
#pragma unroll
  for (int j = 0; j < TN; ++j)
#pragma unroll
    for (int e4 = 0; e4 < 4; ++e4) {
      const int f = wn * (32 * TN) + j * 32 + 8 * e4 + 4 * g;  // 4 consecutive features held by this lane
      const uint2 bb = bias[j][e4];
      const float b0 = H::to_f32(bb.x & 0xFFFF), b1 = H::to_f32(bb.x >> 16);
      const float b2 = H::to_f32(bb.y & 0xFFFF), b3 = H::to_f32(bb.y >> 16);
#pragma unroll
      for (int i = 0; i < TM; ++i) {
        const int t = wm * (32 * TM) + i * 32 + l32;
        uint2 w;
        w.x = H::pack2(silu_fast(acc[i][j][4 * e4] + b0) * mul, silu_fast(acc[i][j][4 * e4 + 1] + b1) * mul);
        w.y = H::pack2(silu_fast(acc[i][j][4 * e4 + 2] + b2) * mul, silu_fast(acc[i][j][4 * e4 + 3] + b3) * mul);
        *reinterpret_cast<uint2*>(&lds[t * kStageLd + f]) = w;
      }
    }
  lds_barrier();
  // ROWS tokens x CH chunks of 8 features
  const int c = c0 + fc * 8;                                 // feature inside the block
  const int head = c >> dh_sh, f = c - (head << dh_sh);
  if (blk == 3 && prefix_tile) {                             // K of prefix rows (V took the other path)
    const UserDesc& tud = p.users[tile_user];               // (as above)
    const int L = tud.L, Lceil = (L + kTile - 1) / kTile * kTile;
    const int64_t kv_stride = tud.kv_tile_stride;
    uint16_t* kvb = reinterpret_cast<uint16_t*>(const_cast<void*>(tud.kv)) + tud.kv_tile0 + (int64_t)(pos0 >> 6) * kv_stride +
                    (int64_t)p.layer * tud.kv_layer_stride;  // the K/V tile of the first 64 rows
#pragma unroll
    for (int it = 0; it < ITS; ++it) {
      const int t = t0 + RPP * it, pos = pos0 + t;
      if (t >= n_rows || pos >= Lceil) continue;             // filler beyond the user's last tile
      uint4 val = *reinterpret_cast<const uint4*>(&lds[t * kStageLd + fc * 8]);
      if (pos >= L) val = make_uint4(0, 0, 0, 0);            // ragged tail of the last tile: zeros
      st_out(kvb + (int64_t)(t >> 6) * kv_stride + head * 2 * kTile * dh + KvLayout16::k_off(t & 63, f, dh), val, 0);
    }
    return;
  }
  const bool ragged = octets && n_rows < ROWS && (n_rows & 7);
#pragma unroll
  for (int it = 0; it < ITS; ++it) {
    const int t = t0 + RPP * it;
    if (t >= n_rows) continue;
    const uint4 val = *reinterpret_cast<const uint4*>(&lds[t * kStageLd + fc * 8]);
    if (kinds[it] == kRowCand) {
      uint32_t at = at0 + RPP * it * d * 2;
      if (ragged && t >= (n_rows & ~7)) at -= (c >> 3) * (8 - (n_rows & 7)) * 16;      // the last octet, of the rows that are left
      st_out(reinterpret_cast<uint16_t*>(reinterpret_cast<char*>(rows_out) + at), val, 0);
    } else {                                                 // k or v of a suffix row
      const int row = m0 + t, idx = p.rt.idx[row], rr = idx & 63;
      uint16_t* base = p.sfx + p.users[p.rt.user[row]].sfx_tile0 + (int64_t)(idx >> 6) * (2 * kTile * d) + head * 2 * kTile * dh;
      if (blk == 3) {
        st_out(base + KvLayout16::k_off(rr, f, dh), val, 0);
      } else {   // V: its 8 features go to 8 different fragments
        const uint32_t w[4] = {val.x, val.y, val.z, val.w};
#pragma unroll
        for (int x = 0; x < 8; ++x) base[KvLayout16::v_off(rr, f + x, dh)] = (uint16_t)(w[x >> 1] >> (16 * (x & 1)));
      }
    }
  }
}

// ---- f1, weight-stationary form ----------------------------------------------------------------
// For launches beyond the tiles above (f1_tile).  One persistent workgroup of 8 wavefronts per compute unit
// keeps a 128-feature slice of W1 (128 x D, up to 128 KiB) in LDS for its whole life and walks 64-row units
// of its share of the rows; the workgroups of one XCD take the same row groups, so that a token panel comes
// from memory once per XCD.  Each wavefront owns whole units (64 rows x 128 features, 2 x 4 MFMA blocks):
// its token fragments go from global memory straight into registers, PF k-steps ahead (a token fragment is
// 1 KiB of contiguous panel bytes, one 16-byte load per lane), the weight fragments are linear LDS reads one
// k-step ahead, and nothing in the main loop waits for another wavefront: no barrier after the slice has
// landed, so the two wavefronts of a SIMD drift apart and one's epilogue (vector ALU, stores) runs beside
// the other's main loop (matrix cores).  The accumulators start from the bias.  Results are staged through
// 4 KiB of wavefront-private LDS (32 tokens x 64 features, 16-byte chunks swizzled by token so that neither
// the 8-byte writes nor the 16-byte reads pile up on a bank) and leave as 128-byte row segments; V of prefix
// rows takes the token-major product, whose accumulators are V-tile fragments as they stand.  Launches that
// write far more than the L2s hold use streaming stores (see st_out): with plain stores the output lines
// evict the token panels the workgroups of an XCD share and the kernel runs at the speed of the re-fetches
// (65 536 x 2048 x 512 stand-alone: 225 us plain, 152 us streaming, 205 us for the tiled kernel above); small
// launches keep plain stores, because what they write fits the L2s and the attention and layer-tail kernels
// read it straight back (8192 rows: the layer tail is 2 us slower behind streaming stores).
constexpr int kF1WsPF = 4;          // k-steps of token fragments in flight per wavefront
constexpr int kF1StreamMinRows = 16384;   // from here on a launch writes 64 MiB and more (at d = 512): streaming stores

template <typename H, int D, bool FEATURE_MAJOR>
__device__ __forceinline__ void f1_ws_mainloop(const uint16_t* __restrict__ tp0, const uint16_t* __restrict__ tp1,
                                               const uint16_t* wlane, f32x16_t (&acc)[2][4]) {
  constexpr int KS = D / 16, PF = kF1WsPF;
  uint4 t[PF][2], ff[2][4];
#pragma unroll
  for (int pf = 0; pf < PF; ++pf) {
    t[pf][0] = *reinterpret_cast<const uint4*>(tp0 + (size_t)pf * 2048);
    t[pf][1] = *reinterpret_cast<const uint4*>(tp1 + (size_t)pf * 2048);
  }
#pragma unroll
  for (int j = 0; j < 4; ++j) ff[0][j] = *reinterpret_cast<const uint4*>(wlane + j * 512);
  // The last PF k-steps are a copy of the loop's body without loads: were the loads inside the loop conditional, the
  // compiler could not count them and would wait for ALL outstanding ones wherever it needs the oldest.
  auto k_steps = [&](auto more_tag, int ks0) {
    constexpr bool MORE = decltype(more_tag)::value;
#pragma unroll
    for (int pf = 0; pf < PF; ++pf) {
      const int ks = ks0 + pf, cur = pf & 1, nxt = cur ^ 1;
      if (MORE || pf + 1 < PF) {
#pragma unroll
        for (int j = 0; j < 4; ++j) ff[nxt][j] = *reinterpret_cast<const uint4*>(wlane + ((ks + 1) * 4 + j) * 512);
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j)
          acc[i][j] = FEATURE_MAJOR ? H::mfma(ff[cur][j], t[pf][i], acc[i][j]) : H::mfma(t[pf][i], ff[cur][j], acc[i][j]);
      if constexpr (MORE) {
        t[pf][0] = *reinterpret_cast<const uint4*>(tp0 + (size_t)(ks + PF) * 2048);
        t[pf][1] = *reinterpret_cast<const uint4*>(tp1 + (size_t)(ks + PF) * 2048);
      }
    }
  };
#pragma unroll 1
  for (int ks0 = 0; ks0 < KS - PF; ks0 += PF) k_steps(std::true_type(), ks0);
  k_steps(std::false_type(), KS - PF);
}

template <typename H, int D>
__global__ __launch_bounds__(512, 1) void f1_ws_bf16_kernel(F1Params p) {
  constexpr int KS = D / 16;
  static_assert(KS % kF1WsPF == 0 && (KS * 4) % 8 == 0, "shape");
  __shared__ __attribute__((aligned(16))) uint16_t wl[KS * 2048];       // 128 features x D, fragment order
  __shared__ __attribute__((aligned(16))) uint16_t stage[8 * 32 * 64];   // per wavefront: 32 tokens x 64 features
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), l32 = lane & 31, g = lane >> 5;
  constexpr int d = D;
  const int dh = p.dh, dh_sh = 31 - __builtin_clz(dh);       // d_head is a power of two
  const int slices_per_blk = d >> 7;
  const int n_slices = p.cm.nblk * slices_per_blk;
  const int n_rg = (int)gridDim.x / n_slices;                 // row groups: a multiple of 8 (host)
  const int xcd = blockIdx.x & 7, idx = blockIdx.x >> 3;
  const int slice = idx % n_slices;
  const int rg = xcd * (n_rg >> 3) + idx / n_slices;
  const int blk = p.cm.blk[slice / slices_per_blk];            // 0 u, 1 v, 2 q, 3 k
  const int c0 = (slice % slices_per_blk) * 128;               // first feature inside the block
  const int n0 = blk * d + c0;
  {
    const uint16_t* src = p.W + (size_t)(n0 >> 7) * KS * 2048;
#pragma unroll
    for (int it = 0; it < KS * 4 / 8; ++it) {
      const int piece = it * 8 + wave;
      __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(src + piece * 512 + lane * 8),
                                       (__attribute__((address_space(3))) void*)(wl + piece * 512), 16, 0, 0);
    }
  }
  const int n_units = (p.row_end - p.row_begin + 63) >> 6;
  const int upr = (n_units + n_rg - 1) / n_rg;
  const int u_begin = rg * upr, u_end = min(n_units, u_begin + upr);
  // (the first unit's row kinds and the biases are touched while the slice is on its way, so that the unit's start finds them in the cache)
  const int first_row = p.row_begin + (u_begin + wave) * 64 + lane;
  int touched = 0;
  if (first_row < p.row_end) touched = p.rt.kind[first_row];
  touched ^= *reinterpret_cast<const int*>(p.bias + n0 + lane * 2);
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  const uint16_t* wlane = wl + lane * 8;
  uint16_t* st = stage + wave * (32 * 64);
  const float mul = (blk == 2) ? p.q_mul : 1.0f;
  if (touched == 0x5a17c0de && p.q_mul < 0.f) st[0] = 0;       // never taken: keeps the loads

  for (int unit = u_begin + wave; unit < u_end; unit += 8) {
    const int m0 = p.row_begin + unit * 64;                    // row_begin is a multiple of 64 (host)
    const int B = m0 >> 5;
    const uint16_t* tp0 = p.A + ((size_t)(B >> 2) * KS) * 2048 + (B & 3) * 512 + lane * 8;
    const uint16_t* tp1 = p.A + ((size_t)((B + 1) >> 2) * KS) * 2048 + ((B + 1) & 3) * 512 + lane * 8;
    // a unit of prefix rows lies inside one user's (256-aligned) prefix region: consecutive positions from pos0
    const bool prefix_unit = m0 < p.n_prows;
    int pos0 = 0, L = 0;
    uint16_t* tile = nullptr;                                  // the unit's K/V tile (all heads)
    if (prefix_unit) {
      pos0 = p.rt.idx[m0];                                     // a multiple of 64: the unit is one K/V tile
      const UserDesc& tud = p.users[p.rt.user[m0]];
      L = tud.L;
      if (pos0 >= (L + kTile - 1) / kTile * kTile) continue;   // filler behind the user's last tile
      tile = reinterpret_cast<uint16_t*>(const_cast<void*>(tud.kv)) + tud.kv_tile0 + (int64_t)(pos0 >> 6) * tud.kv_tile_stride +
             (int64_t)p.layer * tud.kv_layer_stride;
    }
    // new rows: candidates throughout (their k and v go row-major, as u and q do), or suffix rows among them
    const int kind_row = m0 + lane < p.row_end ? p.rt.kind[m0 + lane] : kRowCand;
    f32x16_t acc[2][4];

    if (blk == 1 && prefix_unit) {
      // ---- V of prefix rows: token-major product, accumulators are V-tile fragments
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const float b = H::to_f32(p.bias[n0 + j * 32 + l32]);
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int e = 0; e < 16; ++e) acc[i][j][e] = b;
      }
      f1_ws_mainloop<H, D, false>(tp0, tp1, wlane, acc);
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int c = c0 + j * 32;
        const int head = c >> dh_sh, db = (c - (head << dh_sh)) >> 5;
        uint16_t* frag = tile + head * 2 * kTile * dh + kTile * dh;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          const int tok0 = pos0 + i * 32, kb = i;
#pragma unroll
          for (int m = 0; m < 2; ++m) {
            uint32_t w[4];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
              const int e4 = 2 * m + h;
              float v[4];
#pragma unroll
              for (int r = 0; r < 4; ++r) {
                const int tok = tok0 + 8 * e4 + 4 * g + r;
                const float val = silu_fast(acc[i][j][4 * e4 + r]);
                v[r] = tok < L ? val : 0.f;                  // the ragged tail of the last tile holds zeros
              }
              w[2 * h] = H::pack2(v[0], v[1]);
              w[2 * h + 1] = H::pack2(v[2], v[3]);
            }
            st_out(frag + (((db * 2 + kb) * 2 + m) * 64 + lane) * 8, make_uint4(w[0], w[1], w[2], w[3]), p.stream_out);
          }
        }
      }
      continue;
    }

    // ---- everything else: feature-major product (a lane ends up with 4-feature runs of one token)
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int e4 = 0; e4 < 4; ++e4) {
        const uint2 bb = *reinterpret_cast<const uint2*>(p.bias + n0 + j * 32 + 8 * e4 + 4 * g);
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          acc[i][j][4 * e4] = H::to_f32(bb.x & 0xFFFF);
          acc[i][j][4 * e4 + 1] = H::to_f32(bb.x >> 16);
          acc[i][j][4 * e4 + 2] = H::to_f32(bb.y & 0xFFFF);
          acc[i][j][4 * e4 + 3] = H::to_f32(bb.y >> 16);
        }
      }
    f1_ws_mainloop<H, D, true>(tp0, tp1, wlane, acc);
    const bool any_suffix = !prefix_unit && __builtin_amdgcn_ballot_w64(kind_row != kRowCand) != 0;
    // where 16-byte chunk (row tk of block i, features c0 + jh*64 + fc*8 ..) goes: row-major, or the K tile of a prefix unit
    const bool row_major = blk == 0 || blk == 2 || !prefix_unit;
    // this lane stores chunk fc of rows tk0 + 8 n of a 32-row block (neighbouring lanes: see the tiled kernel)
    const bool octets = p.octets && row_major && blk != 0, rows_first = octets || !row_major;
    const int tk0 = rows_first ? lane & 7 : lane >> 3;
    uint16_t* rows_out = blk == 0 ? p.u + (size_t)m0 * d : blk == 2 ? p.q + (size_t)m0 * d : (blk == 3 ? p.knew : p.vnew) + ((int64_t)m0 - p.n_prows) * d;
    const int n_rows = p.row_end - m0;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
#pragma unroll
      for (int jh = 0; jh < 2; ++jh) {
#pragma unroll
        for (int jj = 0; jj < 2; ++jj) {
          const int j = jh * 2 + jj;
#pragma unroll
          for (int e4 = 0; e4 < 4; ++e4) {
            const int fl = jj * 32 + 8 * e4 + 4 * g;
            uint2 w;
            w.x = H::pack2(silu_fast(acc[i][j][4 * e4]) * mul, silu_fast(acc[i][j][4 * e4 + 1]) * mul);
            w.y = H::pack2(silu_fast(acc[i][j][4 * e4 + 2]) * mul, silu_fast(acc[i][j][4 * e4 + 3]) * mul);
            *reinterpret_cast<uint2*>(st + l32 * 64 + (((fl >> 3) ^ (l32 & 7)) << 3) + (fl & 7)) = w;
          }
        }
        __builtin_amdgcn_wave_barrier();   // LDS serves a wavefront's accesses in order: the reads below see the writes above
        int fc = rows_first ? lane >> 3 : lane & 7;
        // (opaque to the compiler: otherwise it hoists the index arithmetic of the rare suffix-V scatter below out of
        // the unit loop, 32 values per lane that it then has to spill -- 16 MiB of scratch writes per launch)
        asm volatile("" : "+v"(fc));
        const int c = c0 + jh * 64 + fc * 8;                     // feature inside the block
        const int head = c >> dh_sh, f = c - (head << dh_sh);
        auto staged = [&](int n) {                               // chunk fc of row tk0 + 8 n (tk & 7 == tk0 & 7)
          return *reinterpret_cast<const uint4*>(st + (tk0 + 8 * n) * 64 + ((fc ^ (tk0 & 7)) << 3));
        };
        if (row_major && !(any_suffix && (blk == 1 || blk == 3))) {
          // (u and q of filler rows are written too: nothing reads them, and a filler row's inputs are zeros)
          uint16_t* dst = rows_out + (octets ? i * 32 * d + tk0 * 8 : (i * 32 + tk0) * d + c);
#pragma unroll
          for (int n = 0; n < 4; ++n) {
            const int rl = i * 32 + tk0 + 8 * n;
            if (rl < n_rows) st_out(dst + n * 8 * d + (octets ? (c >> 3) * octet_step(rl, n_rows) : 0), staged(n), p.stream_out);
          }
        } else if (prefix_unit) {                                // K of prefix rows (V took the other path)
          uint16_t* kt = tile + head * 2 * kTile * dh;
#pragma unroll
          for (int n = 0; n < 4; ++n) {
            const int rr = i * 32 + tk0 + 8 * n;
            uint4 v = staged(n);
            if (pos0 + rr >= L) v = make_uint4(0, 0, 0, 0);       // ragged tail of the last tile: zeros
            st_out(kt + KvLayout16::k_off(rr, f, dh), v, p.stream_out);
          }
        } else {                                                 // k or v of new rows with suffix rows among them
#pragma unroll 1
          for (int n = 0; n < 4; ++n) {
            const int rl = i * 32 + tk0 + 8 * n, row = m0 + rl;
            if (rl >= n_rows) break;
            const uint4 v = staged(n);
            if (p.rt.kind[row] == kRowCand) {
              st_out(rows_out + (octets ? octet_off(rl, d) + (c >> 3) * octet_step(rl, n_rows) : rl * d + c), v, p.stream_out);
              continue;
            }
            const int pos = p.rt.idx[row], rr = pos & 63;
            uint16_t* base = p.sfx + p.users[p.rt.user[row]].sfx_tile0 + (int64_t)(pos >> 6) * (2 * kTile * d) + head * 2 * kTile * dh;
            if (blk == 3) {
              st_out(base + KvLayout16::k_off(rr, f, dh), v, p.stream_out);
            } else {   // V: its 8 features go to 8 different fragments
              const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
              for (int x = 0; x < 8; ++x) base[KvLayout16::v_off(rr, f + x, dh)] = (uint16_t)(w[x >> 1] >> (16 * (x & 1)));
            }
          }
        }
        __builtin_amdgcn_wave_barrier();   // the next pass overwrites the staging area
      }
    }
  }
}

// ---- gate + f2 + next layer's input LayerNorm in one kernel ------------------------------------
// Everything between the attention of one layer and the projections of the next is local to a row:
//   y  = LN((sum of key-split partial sums + a candidate's self term) / n; g_at, b_at) * u
//   x <- x + y W2^T + b2
//   xh = LN(x; next layer's g_in, b_in)
// so one workgroup takes up to 16*TB rows over the full width D and does all three: y never goes to HBM,
// the residual row is read and written once, and two row-wise passes disappear.  Each wavefront
// gates VROWS/NW rows (lane = D/64 consecutive features, DPP reductions) and writes them into LDS as
// MFMA token fragments shared by all wavefronts; it owns FB = D/16/NW feature blocks of the product and
// streams its own slice of the packed W2 (no wavefront shares weights with another) from L2 straight into registers, PF k-steps
// ahead, and in small launches the first WL k-steps into LDS beside them.  The 16x16x32 product: a block of 16 rows is the smallest,
// and launches of a few hundred rows take 8 or 16 rows per workgroup (the 32x32x16 one multiplied 24 empty rows beside 8).
// Feature-major: a lane ends up with one token and runs of 4 features, so the row statistics of the second LayerNorm are
// a lane-local sum, two lane exchanges and one exchange between wavefronts through LDS.
// What bounds it: a chain of memory round trips.  A compute unit takes about 64 bytes a clock, and W2 is 512 KB of that for every
// workgroup (d = 512), so global loads that depend on no result go out as early as the registers allow: the rows' split sums, W2's first
// k-steps and the residual rows before the first wait; and the gate waits for its own loads only, which takes loads the compiler can
// count (none behind a branch, none in the global_load_lds form: see BufferView) and barriers that wait for LDS alone.  Not so: the launches with
// weights in LDS wait once, between gate and product, for all that has been asked for; and where EARLY_LN is false (64-row workgroups at
// d = 512) gain and offset are loaded in the output pass, one round trip for each feature block behind the stores of the one before.
// Of the launch's time from its first workgroup's start to its last one's end, at 512 rows of 8 pieces, d = 512: split sums summed after
// 2.2 us, tokens written 2.7, first weights there 4.6, product 6.5, statistics 7.6, end 9.4; before (32x32x16, weights requested
// behind the sums, two-pass statistics behind barriers that waited for the residual stores) 2.3, 3.2, 4.6, 7.4, 9.1, 10.5.
struct F2LnParams {
  // gate inputs
  const float* part;        // [pieces][rows][D] unnormalised attention sums; rt.parts says how many a row has
  int parts_shift;          // 0, or 8 for the last layer
  int parts_all;            // the same number for every row of the launch, known without the table (0: look it up)
  size_t split_stride;
  const uint16_t* u;        // [rows, D]
  const uint16_t* q;        // [rows, D] (pre-scaled); null: the attention kernel has added the candidates' own keys already
  const uint16_t* knew;     // [new rows, D] row-major k and v of suffix and candidate rows
  const uint16_t* vnew;
  const uint16_t* gate_gain;
  const uint16_t* gate_offs;
  int n_prows, dh;
  // softmax form (kernels instantiated with SM): part holds sums of exp2(t - m) v, ml the (m, l) of every row, head and
  // split as [split][row][head][2]; the splits and the candidate's own key are merged here
  const float* ml;
  size_t ml_stride;
  int n_heads;
  const uint16_t* W;        // packed W2 [D, D]
  const uint16_t* bias;     // b2 [D]
  float* x;                 // residual stream [rows, D], updated in place
  uint16_t* xh;             // LN(x) panels for the next layer; nullptr: none wanted (last layer)
  const uint16_t* gain;     // next layer's input LayerNorm
  const uint16_t* offs;
  RowTables rt;
  int row_begin, row_end;   // row_begin is a multiple of 32
  float eps;
  // last layer of a ranking call: instead of xh, score_c = <w_score, LN(x; gain, offs)> + b_score for
  // candidate rows, written at the candidate's position in the caller's order (scores != nullptr)
  const uint16_t* w_score;
  float b_score;
  float* scores;
};


// E consecutive bf16 values (E = 2, 4, 8 or 16; address aligned to 2*E bytes, at most 16) as packed words.
template <int E>
__device__ __forceinline__ void ld_bf16_run(const uint16_t* src, uint32_t (&w)[E / 2]) {
  if constexpr (E == 2) {
    w[0] = *reinterpret_cast<const uint32_t*>(src);
  } else if constexpr (E == 4) {
    const uint2 v = *reinterpret_cast<const uint2*>(src);
    w[0] = v.x; w[1] = v.y;
  } else {
#pragma unroll
    for (int c = 0; c < E / 8; ++c) {
      const uint4 v = *reinterpret_cast<const uint4*>(src + 8 * c);
      w[4 * c] = v.x; w[4 * c + 1] = v.y; w[4 * c + 2] = v.z; w[4 * c + 3] = v.w;
    }
  }
}

// One row of the attention combine + gate, by one wavefront, lane owning features [lane*E, lane*E+E).
// SELF: the row's own q, k, v are wanted (softmax form: the candidate's own key is merged here; in the
// SiLU form the attention kernel has it in its sums already).
template <int E, bool SELF>
struct GateRow {
  float o[E];
  uint32_t ub[E / 2], qb[SELF ? E / 2 : 1], kb[SELF ? E / 2 : 1], vb[SELF ? E / 2 : 1];
  int n, kind;
  float mpart, lpart;   // softmax form: reference score of o and the matching sum of weights
};

template <int E>
__device__ __forceinline__ void ld_f32_run(const float* src, float (&v)[E]) {
  if constexpr (E == 2) {
    const float2 t = *reinterpret_cast<const float2*>(src);
    v[0] = t.x; v[1] = t.y;
  } else {
#pragma unroll
    for (int c = 0; c < E / 4; ++c) {
      const float4 t = *reinterpret_cast<const float4*>(src + 4 * c);
      v[4 * c] = t.x; v[4 * c + 1] = t.y; v[4 * c + 2] = t.z; v[4 * c + 3] = t.w;
    }
  }
}

// The partial sums of G rows, summed in the order of their pieces, NB pieces (all G rows each) in flight at a
// time: a row of 8 pieces waits for 8 / NB round trips to memory per group of rows, not for one per
// row and piece.  begin() issues the rows' other inputs and the first NB pieces; the caller may issue further
// loads before finish() adds them up and walks the remaining ones.
// Rows beyond the launch read the workgroup's first row instead and are marked as filler.
template <int D, bool SM, int G, int NB>
struct GateLoad {
  static constexpr int E = D / 64;
  size_t base[G];
  const float* mlr[G];
  float M[G];
  int cnt[G], cmax;           // pieces of each row (uniform over the wavefront), the most of the group
  float buf[NB][G][E];
  float2 mlb[NB][G];

  // (NB pieces of every row without a condition, so that the compiler can count the loads and wait for these alone: a row with
  // fewer pieces repeats its last one, which add() leaves out.  That is a load and NB - 1 times the registers for nothing where no row
  // has that many, so that the launch picks NB: see sums_at_once)
  __device__ __forceinline__ void issue(const F2LnParams& p, int sp0) {
#pragma unroll
    for (int k = 0; k < NB; ++k)
#pragma unroll
      for (int r = 0; r < G; ++r) {
        const int sp = min(sp0 + k, cnt[r] - 1);
        ld_f32_run<E>(p.part + sp * p.split_stride + base[r], buf[k][r]);
        if constexpr (SM) mlb[k][r] = *reinterpret_cast<const float2*>(mlr[r] + sp * p.ml_stride);
      }
  }
  __device__ __forceinline__ void add(const F2LnParams& p, int sp0, GateRow<E, SM> (&gr)[G]) {
#pragma unroll
    for (int k = 0; k < NB; ++k)
#pragma unroll
      for (int r = 0; r < G; ++r) {
        float w = sp0 + k < cnt[r] ? 1.0f : 0.0f;      // (a branch here, and the compiler would move the loads behind it)
        if constexpr (SM) {
          w = (mlb[k][r].x == -INFINITY) ? 0.f : w * __builtin_amdgcn_exp2f(mlb[k][r].x - M[r]);
          gr[r].lpart += w * mlb[k][r].y;
        }
#pragma unroll
        for (int i = 0; i < E; ++i) gr[r].o[i] = fmaf(w, buf[k][r][i], gr[r].o[i]);
      }
  }
  __device__ __forceinline__ void begin(const F2LnParams& p, int row_first, int row_safe, int lane, GateRow<E, SM> (&gr)[G]) {
#pragma unroll
    for (int r = 0; r < G; ++r) {
      const bool ok = row_first + r < p.row_end;
      const int row = ok ? row_first + r : row_safe;
      const int kind = p.rt.kind[row];
      gr[r].kind = ok ? kind : kRowPad;
      gr[r].n = p.rt.lim[row];
      cnt[r] = p.parts_all ? p.parts_all : __builtin_amdgcn_readfirstlane((p.rt.parts[row] >> p.parts_shift) & 255);
      cmax = r == 0 ? cnt[r] : max(cmax, cnt[r]);
      base[r] = (size_t)row * D + lane * E;
      ld_bf16_run<E>(p.u + base[r], gr[r].ub);
      mlr[r] = nullptr;
      M[r] = 0.f;
      if constexpr (SM) {
#pragma unroll
        for (int i = 0; i < E / 2; ++i) gr[r].qb[i] = gr[r].kb[i] = gr[r].vb[i] = 0u;
        if (row >= p.n_prows) {   // suffix and candidate rows have row-major q, k, v (only candidates use them)
          const size_t nb = (size_t)(row - p.n_prows) * D + lane * E;
          ld_bf16_run<E>(p.q + base[r], gr[r].qb);
          ld_bf16_run<E>(p.knew + nb, gr[r].kb);
          ld_bf16_run<E>(p.vnew + nb, gr[r].vb);
        }
        // split s counts with weight 2^(m_s - M), M the largest m_s of this lane's head
        mlr[r] = p.ml + ((size_t)row * p.n_heads + lane * E / p.dh) * 2;
        float m = -INFINITY;
#pragma unroll
        for (int sp = 0; sp < 8; ++sp) m = fmaxf(m, mlr[r][(size_t)min(sp, cnt[r] - 1) * p.ml_stride]);   // at most 8 pieces
        M[r] = m;
      }
      gr[r].mpart = M[r];
      gr[r].lpart = SM ? 0.f : 1.f;
#pragma unroll
      for (int i = 0; i < E; ++i) gr[r].o[i] = 0.f;
    }
    issue(p, 0);
  }
  __device__ __forceinline__ void finish(const F2LnParams& p, GateRow<E, SM> (&gr)[G]) {
    add(p, 0, gr);
    if constexpr (NB < kMaxPieces) {
      for (int sp0 = NB; sp0 < cmax; sp0 += NB) {
        issue(p, sp0);
        add(p, sp0, gr);
      }
    }
  }
};

// Token fragments of the layer tail in LDS: blocks of 16 rows, in each the 16-byte chunk of row r and features 8c .. 8c+7 at
// chunk c * 16 + (r ^ c) % 16.  The product's operand (lane: row lane % 16, chunk 4 k-step + lane / 16) is then four whole runs of
// 256 bytes, and a row's chunks, which the gate's lanes write together, lie on different banks.
template <int D>
__device__ __forceinline__ int tok_off(int row, int c) { return ((row >> 4) * (D * 2) + c * 16 + ((row ^ c) & 15)) * 8; }

// Finishes G rows at once (their reductions interleave) and writes y (16 bits) into the token fragments: rows lr0 .. lr0 + G - 1
// of the workgroup.
template <typename H, int D, int G, bool SM>
__device__ __forceinline__ void finish_gate_rows(const F2LnParams& p, GateRow<D / 64, SM> (&gr)[G], int lane, uint16_t* tok, int lr0,
                                                 const uint32_t (&gw)[D / 128], const uint32_t (&ow)[D / 128]) {
  constexpr int E = D / 64;
  float s[G], inv_n[G];
#pragma unroll
  for (int r = 0; r < G; ++r) {
    int n = gr[r].n;
    float lsum = gr[r].lpart;
    if constexpr (!SM) {
      if (gr[r].kind == kRowCand) n += 1;   // the own key is in the attention kernel's sums already; it counts as a visible key
    } else if (gr[r].kind == kRowCand) {      // the candidate's own key, per head
      float dot = 0.f;
#pragma unroll
      for (int i = 0; i < E; ++i) dot += H::of_word(gr[r].qb[i >> 1], i) * H::of_word(gr[r].kb[i >> 1], i);
      // the lanes of one head are dh/E consecutive lanes
      const int hl = p.dh / E;
      if (hl == 2) dot = lanes2_sum(dot);
      else if (hl == 4) dot = lanes4_sum(dot);
      else if (hl == 8) dot = lanes8_sum(dot);
      else if (hl == 16) dot = lanes16_sum(dot);
      else if (hl == 32) dot = lanes32_sum(dot);
      else if (hl == 64) dot = wave_sum_dpp(dot);
      // the stored q carries alpha * log2(e), so dot is the own key's score in the units of m; bring the
      // merged splits and the own key to their common maximum
      const float Mn = fmaxf(gr[r].mpart, dot);
      const float c = (gr[r].mpart == -INFINITY) ? 0.f : __builtin_amdgcn_exp2f(gr[r].mpart - Mn);
      const float ws = __builtin_amdgcn_exp2f(dot - Mn);
#pragma unroll
      for (int i = 0; i < E; ++i) gr[r].o[i] = gr[r].o[i] * c + ws * H::of_word(gr[r].vb[i >> 1], i);
      lsum = lsum * c + ws;
    }
    inv_n[r] = SM ? 1.0f / (lsum > 0.f ? lsum : 1.0f) : 1.0f / (float)(n > 0 ? n : 1);
    s[r] = 0.f;
#pragma unroll
    for (int i = 0; i < E; ++i) { gr[r].o[i] *= inv_n[r]; s[r] += gr[r].o[i]; }
  }
  float mean[G], qv[G];
#pragma unroll
  for (int r = 0; r < G; ++r) mean[r] = wave_sum_dpp(s[r]) * (1.0f / (float)D);
#pragma unroll
  for (int r = 0; r < G; ++r) {
    qv[r] = 0.f;
#pragma unroll
    for (int i = 0; i < E; ++i) { const float c = gr[r].o[i] - mean[r]; qv[r] += c * c; }
  }
#pragma unroll
  for (int r = 0; r < G; ++r) {
    const float rstd = rsqrtf(wave_sum_dpp(qv[r]) * (1.0f / (float)D) + p.eps);
    uint32_t yw[E / 2];
#pragma unroll
    for (int i = 0; i < E / 2; ++i) {
      float z0 = (gr[r].o[2 * i] - mean[r]) * rstd * H::of_word(gw[i], 0) + H::of_word(ow[i], 0);
      float z1 = (gr[r].o[2 * i + 1] - mean[r]) * rstd * H::of_word(gw[i], 1) + H::of_word(ow[i], 1);
      f32x2_t two = {z0 * H::of_word(gr[r].ub[i], 0), z1 * H::of_word(gr[r].ub[i], 1)};
      if (gr[r].kind == kRowPad) { two[0] = 0.f; two[1] = 0.f; }
      yw[i] = H::pack2(two[0], two[1]);
    }
    constexpr int RUN = E < 8 ? E : 8;
#pragma unroll
    for (int c = 0; c < E; c += RUN) {
      const int f = lane * E + c;
      uint16_t* dst = tok + tok_off<D>(lr0 + r, f >> 3) + (f & 7);
      if constexpr (RUN == 2) *reinterpret_cast<uint32_t*>(dst) = yw[c / 2];
      else if constexpr (RUN == 4) *reinterpret_cast<uint2*>(dst) = make_uint2(yw[c / 2], yw[c / 2 + 1]);
      else *reinterpret_cast<uint4*>(dst) = make_uint4(yw[c / 2], yw[c / 2 + 1], yw[c / 2 + 2], yw[c / 2 + 3]);
    }
  }
}

// ---- L2 warm-up -----------------------------------------------------------------------------------
// Workgroups that stream the same operand run in step, so without help every slice of it is a first
// touch for the whole XCD and costs a full trip to HBM or the memory-side cache, with only the few
// k-steps in flight to cover it.  Instead, each workgroup asks for one 4-byte word of every 128-byte
// line of ITS share of the operand when it starts: together the sharers pull the whole operand into
// their XCD's L2 in one round trip, and the later loads hit L2.  (Measured: 9 % off the layer-tail
// kernel, whose W2 stream waits on latency; the same warm-up made the f1 GEMM 9 % slower -- its
// operand stream is bound by L2 -> LDS bandwidth, not latency -- and is not used there.)
// Touches lines [share * per, share * per + per) of `lines` lines, per = lines / n_shares, at most
// MAXLD loads per thread, all issued at once (a thread with fewer lines to touch repeats its last one);
// v receives the words (to be consumed by a never-taken branch once the loads are known to have landed).
template <int MAXLD>
__device__ __forceinline__ void l2_touch(const void* base, int lines, int share, int n_shares, int tid, int n_threads, int (&v)[MAXLD]) {
  const int per = lines / n_shares;
  const char* b = reinterpret_cast<const char*>(base) + (size_t)share * per * 128;
#pragma unroll
  for (int u = 0; u < MAXLD; ++u) {
    const int i = min(tid + u * n_threads, per - 1);
    v[u] = (u == 0 || (u * n_threads < per)) ? *reinterpret_cast<const int*>(b + (size_t)i * 128) : 0;
  }
}

// OCC = 2: built to fit two workgroups on a compute unit (128 registers per lane), so that one's gate
// phase (memory) overlaps the other's product phase (L2 and matrix cores) when a launch has several
// workgroups per unit: fewer k-steps and gate rows in flight, and the weight fragments and the
// residual rows are requested after the gate instead of before it.
// VR < 16 * TB: a workgroup takes only VR rows (a partly filled row block).  For launches of a few hundred to a
// few thousand rows (one user per call): with 32 rows each they would occupy a few dozen compute units, each
// pulling 16 KiB of split partial sums per row through its own memory path; with VR = 8 or 16 four times or
// twice as many units share that.
// NB: pieces of each row's sums in flight (sums_at_once), with rows enough for every wavefront no more than two, at d = 1024 with more than 8 rows one.
// d = 1024, 32 rows a workgroup: one k-step of weights in flight; two rows' sums, and gain and offset of the output pass behind the gate (us a call with one
// row's and in the output pass / so: 16 users of 4096 keys 2146 / 2132, 40 of 1000 3527 / 3510, 12 of 2000 1419 / 1412; with four k-steps as well 2130,
// 3512, 1415, the same within what the runs differ by, 2 to 8).  8 and 16 rows: four k-steps (softmax form, with q, k and v of the rows: two), which
// 16 rows gain from (one of each / so: five users of 500 keys and 800 candidates 816 / 804, pre-inference of 3500 keys 838 / 827, full recompute of
// 2000 752 / 742; 8 rows, one user of 4096 keys and 512 candidates 428 / 430).
// WL > 0: launches of at most one workgroup per compute unit.  The first WL k-steps of each wavefront's weights go straight to
// LDS and the next PF into registers, all requested before the gate, which waits for other memory; the product then finds them there.
template <typename H, int D, int NW, int TB, bool SM, int OCC, int VR, int WL, int NB>
__global__ __launch_bounds__(NW * 64, OCC == 2 ? 4 : 1) void f2_ln_bf16_kernel(F2LnParams p) {
  constexpr int KS = D / 32;            // k-steps
  constexpr int FB = D / 16 / NW;       // 16-feature blocks per wavefront
  constexpr int PF = FB >= 8 ? (TB > 1 ? 1 : SM ? 2 : 4) : (OCC == 2 ? 2 : 4);   // k-steps of weight fragments in flight per wavefront
  constexpr int ROWS = 16 * TB;         // rows of the product: TB blocks of 16 share one pass over W2
  static_assert(NW == tail_waves(D) && FB == tail_blocks(D) && FB * NW * 16 == D && (KS - WL) % PF == 0 && KS - WL >= PF, "shape");
  __shared__ __attribute__((aligned(16))) uint16_t tok[ROWS * D];         // tok_off
  __shared__ __attribute__((aligned(16))) uint16_t wlds[WL > 0 ? NW * WL * FB * 512 : 8];
  // per wavefront: sums, squares and score parts of ROWS rows (where the weights fill the LDS, in the wavefront's own part of them)
  constexpr int RED = WL > 0 ? WL * FB * 256 : 3 * ROWS;
  static_assert(RED >= 3 * ROWS, "room for the rows' sums");
  __shared__ float red_own[WL > 0 ? 1 : NW * RED];
  float* red = WL > 0 ? reinterpret_cast<float*>(wlds) : red_own;
  constexpr int VROWS = VR;             // rows this workgroup really has
  static_assert(VROWS <= ROWS && VROWS % NW == 0, "whole rows per wavefront");
  const int row0 = p.row_begin + blockIdx.x * VROWS;
  if (row0 >= p.row_end) return;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), l16 = lane & 15, q = lane >> 4;

  // The gate makes the tokens: each wavefront takes VROWS/NW rows, a few at a time
  // so that their loads are in flight together.  The first group's loads go out before anything
  // else, since they are what the workgroup needs first.
  constexpr int RPW = VROWS / NW, GMAX = OCC == 2 ? 2 : (D >= 1024 ? (SM ? 1 : 2) : TB * FB >= 16 ? 2 : (SM ? 2 : 4)), GROUP = RPW < GMAX ? RPW : GMAX;
  static_assert(RPW >= 1 && RPW % GROUP == 0, "rows per wavefront");
  GateRow<D / 64, SM> gr[GROUP];
  uint32_t gw[D / 128], ow[D / 128];
  GateLoad<D, SM, GROUP, NB> gl;
  gl.begin(p, row0 + wave * RPW, row0, lane, gr);
  ld_bf16_run<D / 64>(p.gate_gain + lane * (D / 64), gw);
  ld_bf16_run<D / 64>(p.gate_offs + lane * (D / 64), ow);

  // this wavefront's weight fragments: feature blocks wave*FB .. +FB-1, each KS fragments of 1 KiB
  const BufferView w2(p.W, D * D * 2);
  auto w_off = [&](int j, int ks) { return ((wave * KS + (ks & (KS - 1))) * FB + j) * 1024; };
  static_assert((KS & (KS - 1)) == 0, "k-steps: a power of two");
  // the workgroups of an XCD walk the k-steps from different starting points, so that at any moment
  // they ask the XCD's L2 for different slices of W2 instead of all for the same one
  // (the sum over k then runs in a different order per block; for prefix rows the starting point is
  // taken from the block's position inside its user's prefix, not from the block index, so that a user's
  // place in the batch does not enter the K/V that a pre-inference leaves in the pool)
  const int blk_id = row0 >= p.n_prows ? (int)blockIdx.x : WL > 0 ? (row0 & (kPrefixRowAlign - 1)) / VROWS : p.rt.idx[row0] / VROWS;
  const int rot = ((blk_id >> 3) * PF) & (KS - 1);
  if constexpr (WL > 0) {
#pragma unroll
    for (int i = 0; i < WL; ++i)
#pragma unroll
      for (int j = 0; j < FB; ++j)
        w2.load_lds(wlds + ((wave * WL + i) * FB + j) * 512, lane * 16, w_off(j, PF + i + rot));
  }

  // L2 warm-up of W2 (every workgroup streams all of it, in step): the workgroups of an XCD (every
  // eighth one) each ask for a slice now, so that the product phase below finds W2 in L2
  int touched[4] = {0, 0, 0, 0};
  if constexpr (WL == 0) {
    const int wgs_per_xcd = (int)gridDim.x >> 3;
    const int n_slices = wgs_per_xcd < 1 ? 1 : (wgs_per_xcd < 16 ? wgs_per_xcd : 16);
    l2_touch<4>(p.W, D * D / 64, ((int)blockIdx.x >> 3) % n_slices, n_slices, (int)threadIdx.x, NW * 64, touched);
  }

  uint4 wf[PF][FB];
  auto prefetch_w = [&]() {
#pragma unroll
    for (int i = 0; i < PF; ++i)
#pragma unroll
      for (int j = 0; j < FB; ++j) wf[i][j] = w2.load(lane * 16, w_off(j, i + rot));
  };
  // The accumulators start from the residual row plus the bias, fetched now so that the gate and
  // the product hide the latency (the row's kind is only needed when results are stored): element
  // r of acc[b][j] is feature (wave*FB + j)*16 + 4*q + r of token row0 + 16*b + l16.
  bool in_range[TB], live[TB];
  float* const x0 = p.x + (size_t)row0 * D;
  auto x_off = [&](int b) { return in_range[b] ? (16 * b + l16) * D : 0; };
  int kind_ep[TB];
  f32x4_t acc[TB][FB];
  uint2 b2[FB];
  auto load_residual = [&]() {
#pragma unroll
    for (int b = 0; b < TB; ++b) {
      const int row = row0 + 16 * b + l16;
      in_range[b] = row < p.row_end && 16 * b + l16 < VROWS;
      kind_ep[b] = p.rt.kind[in_range[b] ? row : row0];
#pragma unroll
      for (int j = 0; j < FB; ++j) acc[b][j] = *reinterpret_cast<const f32x4_t*>(x0 + x_off(b) + (wave * FB + j) * 16 + 4 * q);
    }
#pragma unroll
    for (int j = 0; j < FB; ++j) b2[j] = *reinterpret_cast<const uint2*>(p.bias + (wave * FB + j) * 16 + 4 * q);
  };
  auto add_bias = [&]() {
#pragma unroll
    for (int j = 0; j < FB; ++j) {
      const f32x4_t bv = {H::to_f32(b2[j].x & 0xFFFF), H::to_f32(b2[j].x >> 16), H::to_f32(b2[j].y & 0xFFFF), H::to_f32(b2[j].y >> 16)};
#pragma unroll
      for (int b = 0; b < TB; ++b) acc[b][j] += bv;
    }
  };
  // gain and offset of the LayerNorm that follows the product: requested early where the registers allow it,
  // so that the output pass does not wait for them
  constexpr bool EARLY_LN = OCC == 1;
  uint2 lng[FB], lno[FB];
  auto load_ln = [&]() {
#pragma unroll
    for (int j = 0; j < FB; ++j) {
      const int c = (wave * FB + j) * 16 + 4 * q;
      lng[j] = *reinterpret_cast<const uint2*>(p.gain + c);
      lno[j] = *reinterpret_cast<const uint2*>(p.offs + c);
    }
  };

  // The residual rows are requested now, behind the rows' first loads; the weight fragments once the
  // split buffers are free; then the first rows are reduced and written as token fragments, and
  // further groups of rows follow.
  constexpr bool EARLY_W = OCC == 1 && !SM && D < 1024;      // elsewhere the registers do not allow it
  constexpr bool W_FIRST = EARLY_W && WL > 0 && GROUP == 1;  // (with a single row's sums in flight there is room for the weights too)
  constexpr bool LN_FIRST = EARLY_LN && WL > 0 && KS == PF + WL;
  if constexpr (W_FIRST) prefetch_w();
  if constexpr (EARLY_W) load_residual();
  if constexpr (LN_FIRST) load_ln();
  gl.finish(p, gr);
  if constexpr (EARLY_W && !W_FIRST) prefetch_w();           // in flight while the rows are normalised and written to LDS
  finish_gate_rows<H, D, GROUP, SM>(p, gr, lane, tok, wave * RPW, gw, ow);
#pragma unroll
  for (int r0 = GROUP; r0 < RPW; r0 += GROUP) {
    gl.begin(p, row0 + wave * RPW + r0, row0, lane, gr);
    gl.finish(p, gr);
    finish_gate_rows<H, D, GROUP, SM>(p, gr, lane, tok, wave * RPW + r0, gw, ow);
  }
  if constexpr (WL > 0) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");     // this wavefront's weights are in LDS
  lds_barrier();
  if ((touched[0] ^ touched[1] ^ touched[2] ^ touched[3]) == 0x5a17c0de && p.eps < 0.f) red[0] = 0.f;   // never taken: keeps the warm-up loads
  if constexpr (!EARLY_W) { prefetch_w(); load_residual(); }
  __builtin_amdgcn_sched_barrier(0);                         // (where no weights are in LDS, the residual rows are not waited for before this)
  add_bias();
  if constexpr (EARLY_LN && WL == 0) load_ln();
  auto multiply = [&](int ks, const auto& w) {
    const uint16_t* tk = &tok[tok_off<D>(l16, 4 * ks + q)];      // (the same chunk of every block of 16 rows)
#pragma unroll
    for (int b = 0; b < TB; ++b) {
      const u32x4_t tf = lds_read16(tk + b * (16 * D));
#pragma unroll
      for (int j = 0; j < FB; ++j) acc[b][j] = H::mfma16(w[j], tf, acc[b][j]);
    }
  };
  // (the last PF k-steps apart from the loop, so that the loads in it are unconditional: see f1_ws_mainloop)
  auto k_steps = [&](auto more_tag, int ks0, int next) {
    constexpr bool MORE = decltype(more_tag)::value;
#pragma unroll
    for (int i = 0; i < PF; ++i) {
      const int ks = (ks0 + i + rot) & (KS - 1);
      multiply(ks, wf[i]);
      if constexpr (MORE) {
#pragma unroll
        for (int j = 0; j < FB; ++j) wf[i][j] = w2.load(lane * 16, w_off(j, ks + next));
      }
    }
  };
  int ks0 = 0;
  if constexpr (WL > 0) {      // the k-steps in registers, which then take the first ones behind those in LDS, and while these come, the ones in LDS
    k_steps(std::integral_constant<bool, (KS > PF + WL)>(), 0, PF + WL);
#pragma unroll
    for (int i = 0; i < WL; ++i) {
      u32x4_t wv[FB];
#pragma unroll
      for (int j = 0; j < FB; ++j) wv[j] = lds_read16(wlds + ((wave * WL + i) * FB + j) * 512 + lane * 8);
      multiply((PF + i + rot) & (KS - 1), wv);
    }
    ks0 = PF + WL;
    if constexpr (EARLY_LN && !LN_FIRST) load_ln();
  }
  if constexpr (KS > (WL > 0 ? PF + WL : 0)) {
#pragma unroll 1
    for (; ks0 < KS - PF; ks0 += PF) k_steps(std::true_type(), ks0, PF);
    k_steps(std::false_type(), KS - PF, PF);
  }

  // the new residual rows go back; their sums start the LayerNorm statistics
  const bool want_score = p.scores != nullptr;
  float s1[TB];
#pragma unroll
  for (int b = 0; b < TB; ++b) {
    live[b] = in_range[b] && kind_ep[b] != kRowPad;
    s1[b] = 0.f;
#pragma unroll
    for (int j = 0; j < FB; ++j) {
      const f32x4_t v = acc[b][j];
      if (live[b] && !want_score) *reinterpret_cast<f32x4_t*>(x0 + x_off(b) + (wave * FB + j) * 16 + 4 * q) = v;   // nothing reads x after the score head
      s1[b] += (v[0] + v[1]) + (v[2] + v[3]);
    }
  }
  if (p.xh == nullptr && !want_score) return;          // uniform over the grid

  // LayerNorm of the new residual rows.  Every wavefront has the sum and the squares around its own mean of its FB * 16 features; one
  // exchange through LDS makes them the row's: squares around the row's mean are those around the parts' means plus the parts'
  // distances.  (Barriers that leave the residual rows' stores in flight: __syncthreads() would wait for them.)
  constexpr float kOwn = FB * 16;
  float* mine = red + wave * RED;
#pragma unroll
  for (int b = 0; b < TB; ++b) {
    s1[b] = rows4_sum(s1[b]);
    const float m = s1[b] * (1.0f / kOwn);
    float s2 = 0.f;
#pragma unroll
    for (int j = 0; j < FB; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) { const float c = acc[b][j][e] - m; s2 += c * c; }
    s2 = rows4_sum(s2);
    if (q == 0) { mine[16 * b + l16] = s1[b]; mine[ROWS + 16 * b + l16] = s2; }
  }
  lds_barrier();
  const uint16_t* gain = p.gain + wave * FB * 16 + 4 * q;
  const uint16_t* offs = p.offs + wave * FB * 16 + 4 * q;
#pragma unroll
  for (int b = 0; b < TB; ++b) {
    float ps[NW], mean = 0.f, var = 0.f;
#pragma unroll
    for (int w = 0; w < NW; ++w) { ps[w] = red[w * RED + 16 * b + l16]; mean += ps[w]; }
    mean *= 1.0f / (float)D;
#pragma unroll
    for (int w = 0; w < NW; ++w) { const float c = ps[w] * (1.0f / kOwn) - mean; var += red[w * RED + ROWS + 16 * b + l16] + kOwn * c * c; }
    const float rstd = rsqrtf(var * (1.0f / (float)D) + p.eps);
    float sc = 0.f;
    // the row's place in the panels: its 16-byte chunk of features 16 j + 8 (q / 2), 4 features each for two lanes
    uint16_t* out = p.xh + (in_range[b] ? panel_off(row0 + 16 * b + l16, wave * FB * 16 + 4 * q, D) : 0);
#pragma unroll
    for (int j = 0; j < FB; ++j) {
      const uint2 gg = EARLY_LN ? lng[j] : *reinterpret_cast<const uint2*>(gain + j * 16);
      const uint2 oo = EARLY_LN ? lno[j] : *reinterpret_cast<const uint2*>(offs + j * 16);
      float z0 = (acc[b][j][0] - mean) * rstd * H::to_f32(gg.x & 0xFFFF) + H::to_f32(oo.x & 0xFFFF);
      float z1 = (acc[b][j][1] - mean) * rstd * H::to_f32(gg.x >> 16) + H::to_f32(oo.x >> 16);
      float z2 = (acc[b][j][2] - mean) * rstd * H::to_f32(gg.y & 0xFFFF) + H::to_f32(oo.y & 0xFFFF);
      float z3 = (acc[b][j][3] - mean) * rstd * H::to_f32(gg.y >> 16) + H::to_f32(oo.y >> 16);
      if (want_score) {       // uniform over the grid: the score head's dot product, reduced like the statistics above
        const uint2 ww = *reinterpret_cast<const uint2*>(p.w_score + (wave * FB + j) * 16 + 4 * q);
        sc += z0 * H::to_f32(ww.x & 0xFFFF);
        sc += z1 * H::to_f32(ww.x >> 16);
        sc += z2 * H::to_f32(ww.y & 0xFFFF);
        sc += z3 * H::to_f32(ww.y >> 16);
      } else if (in_range[b]) {
        if (!live[b]) z0 = z1 = z2 = z3 = 0.f;     // filler rows stay finite
        *reinterpret_cast<uint2*>(out + j * 2048) = make_uint2(H::pack2(z0, z1), H::pack2(z2, z3));
      }
    }
    if (want_score) {
      sc = rows4_sum(sc);
      if (q == 0) mine[2 * ROWS + 16 * b + l16] = sc;
    }
  }
  if (want_score) {
    lds_barrier();
    if (wave == 0 && q == 0) {
#pragma unroll
      for (int b = 0; b < TB; ++b) {
        float total = p.b_score;
#pragma unroll
        for (int w = 0; w < NW; ++w) total += red[w * RED + 2 * ROWS + 16 * b + l16];
        const int row = row0 + 16 * b + l16;
        if (in_range[b] && kind_ep[b] == kRowCand) p.scores[p.rt.src[row]] = total;
      }
    }
  }
}

}  // namespace relaygr
