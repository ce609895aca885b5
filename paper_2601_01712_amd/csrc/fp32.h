// The fp32 path's kernels on the fp32 matrix instructions (v_mfma_f32_32x32x2_f32 / 16x16x4_f32: full fp32 products and
// sums): attention, the u|v|q|k projection, and the layer tail.  One idea is common to all three.  An fp32 fragment is
// one float per lane and k-step, so a lane would have to load single floats; but the order in which a contraction walks
// k is free as long as both operands agree, and with MFMA t of a group of four taking k = 8m + 4g + t (32-row form; g the
// lane's half) a lane's operands for four MFMAs are four consecutive floats of one row: one 16-byte load straight from
// row-major memory, no staging, no barrier.  The rows a wavefront reads come back through L1 over the next loads (a row's
// 128-byte line feeds four of them), and at 64 cycles per MFMA a wavefront asks for at most 2 KiB per 256 cycles.
#pragma once

#include "attention.h"
#include "common.h"
#include "gemm.h"
#include "rowwise.h"

namespace relaygr {

typedef float f32x4v_t __attribute__((ext_vector_type(4)));

__device__ __forceinline__ f32x16_t mfma32_f32(float a, float b, f32x16_t c) { return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0); }
__device__ __forceinline__ f32x4v_t mfma16_f32(float a, float b, f32x4v_t c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }
__device__ __forceinline__ float f4_at(const float4& v, int i) { return i == 0 ? v.x : i == 1 ? v.y : i == 2 ? v.z : v.w; }

// ---- attention ------------------------------------------------------------------------------------
// A wavefront owns 32 rows of one user and head and a range of 32-key half tiles:
//   S^T[32 keys][32 rows] = K (rows of the MFMA) x Q^T, P = SiLU(S) on the vector ALU, O^T += V^T x P^T,
// where the accumulator of S^T (lane = row, keys 8*(e/4) + 4g + e%4) is element by element the operand of the second
// product, and V is stored transposed, so that its operand is again 16 consecutive bytes.  Every operand is loaded
// straight from the K/V tile; the loads of a half tile's V and of the next one's K are issued a product (2048 cycles at
// d_head 64) before they are needed.  Nothing is shared, so nothing waits: two wavefronts a SIMD, one's SiLU beside the
// other's products.  The products take 4 cycles of a SIMD's matrix pipe per score element at d_head 64, 7 of the 19 us below; the
// rest is SiLU on the vector ALU and what two wavefronts do not hide of each other's waits.
// gs = 8: the eight wavefronts of a workgroup take the same rows and consecutive parts of the keys and add their sums
// in LDS (in a fixed order): calls of few rows fill the chip without writing a partial sum for every part.
// 512 rows x 2048 keys x 4 heads of 64: 19 us a launch (57 TFLOP/s); one thread per row over LDS-broadcast keys took 277.
constexpr int kF32Team = 8;
template <int DH, bool SOFTMAX>
__global__ __launch_bounds__(kF32Team * 64, 2) void attn_f32_kernel(AttnParams p) {
  constexpr int KM = DH / 8, DB = DH / 32;
  constexpr int NT = kF32Team;
  __shared__ float4 xch[NT][DB * 4][64];             // the team's sums, 4 elements a slot
  __shared__ float2 xml[SOFTMAX ? NT : 1][SOFTMAX ? 64 : 1];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), l32 = lane & 31, g = lane >> 5;
  const bool team = p.gs > 1;
  const int total = p.n_tiles * p.n_heads * p.nsplit;
  const int n_wg = team ? total : (total + NT - 1) / NT;
  const int wg = xcd_remap(blockIdx.x, n_wg);
  if (wg >= n_wg) return;
  const int item = team ? wg : wg * NT + wave;
  if (item >= total) return;                         // (only without a team, where no wavefront meets a barrier)
  const int tile_i = item % p.n_tiles, hs = item / p.n_tiles;
  const int head = hs % p.n_heads, split_ext = hs / p.n_heads;
  const AttnTile at = p.tiles[tile_i];
  // half tiles this item sees: [prefix | suffix], and this wavefront's part of them
  const int n_hp = ((at.kind == 0 ? at.pos0 + at.nrows : at.L) + 31) >> 5;
  const int n_h = n_hp + (at.kind == 0 ? 0 : (at.S + 31) >> 5);
  const int parts = team ? p.nsplit * NT : p.nsplit, part_i = team ? split_ext * NT + wave : split_ext;
  const int per = (n_h + parts - 1) / parts;
  const int h0 = min(part_i * per, n_h), h1 = min(h0 + per, n_h);

  const bool ok = l32 < at.nrows;
  const int row = at.row0 + (ok ? l32 : 0);
  const int lim = at.lim(l32);
  const float* kv = reinterpret_cast<const float*>(at.kv) + (int64_t)p.layer * at.layer_stride(p.d) + (int64_t)head * 2 * kTile * DH;
  const float* sf = reinterpret_cast<const float*>(p.sfx) + at.sfx_tile0 + (int64_t)head * 2 * kTile * DH;
  auto tile_of = [&](int h) -> const float* {        // start of the tile half h lies in
    return h < n_hp ? kv + (int64_t)(h >> 1) * at.kv_tile_stride : sf + (int64_t)((h - n_hp) >> 1) * (2 * kTile * p.d);
  };
  auto half_of = [&](int h) { return (h < n_hp ? h : h - n_hp) & 1; };
  float4 kf[KM], vf[DB][4], qf[KM];
  auto load_k = [&](int h) {
    const float* src = tile_of(h) + (half_of(h) * 32 + l32) * DH + 4 * g;
#pragma unroll
    for (int m = 0; m < KM; ++m) kf[m] = *reinterpret_cast<const float4*>(src + 8 * m);
  };
  auto load_v = [&](int h) {
    const float* src = tile_of(h) + kTile * DH + l32 * kTile + half_of(h) * 32 + 4 * g;
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
      for (int e4 = 0; e4 < 4; ++e4) vf[db][e4] = *reinterpret_cast<const float4*>(src + db * 32 * kTile + 8 * e4);
  };
  f32x16_t o[DB];
#pragma unroll
  for (int db = 0; db < DB; ++db)
#pragma unroll
    for (int e = 0; e < 16; ++e) o[db][e] = 0.f;
  float mref = -INFINITY, lsum = 0.f;                // softmax form: running maximum, this lane's sum of exp(s - m)

  constexpr bool AHEAD = DH < 128;                   // d_head 128: K and V fragments take turns in the registers
  if (h0 < h1) {
    if constexpr (AHEAD) load_k(h0);
    const float* qrow = reinterpret_cast<const float*>(p.q) + (size_t)row * p.d + head * DH + 4 * g;
#pragma unroll
    for (int m = 0; m < KM; ++m) {
      const float4 q = *reinterpret_cast<const float4*>(qrow + 8 * m);
      qf[m] = make_float4(q.x * p.score_mul, q.y * p.score_mul, q.z * p.score_mul, q.w * p.score_mul);
    }
    for (int h = h0; h < h1; ++h) {
      if constexpr (AHEAD) load_v(h);
      else load_k(h);
      f32x16_t s;
#pragma unroll
      for (int e = 0; e < 16; ++e) s[e] = 0.f;
#pragma unroll
      for (int m = 0; m < KM; ++m)
#pragma unroll
        for (int t = 0; t < 4; ++t) s = mfma32_f32(f4_at(kf[m], t), f4_at(qf[m], t), s);
      if constexpr (!AHEAD) load_v(h);
      else if (h + 1 < h1) load_k(h + 1);
      const bool is_sfx = h >= n_hp;
      const int key0 = is_sfx ? at.L + (h - n_hp) * 32 : h * 32;
      const int vis = min(lim, is_sfx ? at.L + at.S : at.L) - key0 - 4 * g;   // element e is visible iff 8*(e/4) + e%4 < vis
      if constexpr (SOFTMAX) {
        float mx = -INFINITY;
#pragma unroll
        for (int e = 0; e < 16; ++e) mx = fmaxf(mx, (8 * (e >> 2) + (e & 3) < vis) ? s[e] : -INFINITY);
        mx = fmaxf(mx, __shfl_xor(mx, 32, 64));      // the two lanes of a row share one reference
        const float mn = fmaxf(mref, mx);
        if (__builtin_amdgcn_ballot_w64(mn > mref)) {
          const float c = mn == mref ? 1.0f : __expf(mref - mn);
          lsum *= c;
#pragma unroll
          for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int e = 0; e < 16; ++e) o[db][e] *= c;
          mref = mn;
        }
      }
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const bool see = 8 * (e >> 2) + (e & 3) < vis;
        float pe = SOFTMAX ? __expf(s[e] - mref) : silu_f32(s[e]);
        pe = see ? pe : 0.f;
        if constexpr (SOFTMAX) lsum += pe;
        s[e] = pe;
      }
#pragma unroll
      for (int e = 0; e < 16; ++e)
#pragma unroll
        for (int db = 0; db < DB; ++db) o[db] = mfma32_f32(f4_at(vf[db][e >> 2], e & 3), s[e], o[db]);
    }
  }
  if constexpr (SOFTMAX) lsum += __shfl_xor(lsum, 32, 64);
  float* dst = p.part + split_ext * p.split_stride + (size_t)row * p.d + head * DH + 4 * g;
  float* mlp = p.ml + split_ext * p.ml_stride + ((size_t)row * p.n_heads + head) * 2;
  if (!team) {
    if (!ok) return;
    if constexpr (SOFTMAX) {
      if (g == 0) *reinterpret_cast<float2*>(mlp) = make_float2(mref, lsum);
    }
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
      for (int e4 = 0; e4 < 4; ++e4)
        *reinterpret_cast<float4*>(dst + db * 32 + 8 * e4) = make_float4(o[db][4 * e4], o[db][4 * e4 + 1], o[db][4 * e4 + 2], o[db][4 * e4 + 3]);
    return;
  }
#pragma unroll
  for (int db = 0; db < DB; ++db)
#pragma unroll
    for (int e4 = 0; e4 < 4; ++e4) xch[wave][db * 4 + e4][lane] = make_float4(o[db][4 * e4], o[db][4 * e4 + 1], o[db][4 * e4 + 2], o[db][4 * e4 + 3]);
  if constexpr (SOFTMAX) xml[wave][lane] = make_float2(mref, lsum);
  __syncthreads();
  if (!ok) return;
  float w[NT];                                       // softmax form: what brings the sums to their common maximum
  if constexpr (SOFTMAX) {
    float M = -INFINITY, l = 0.f;
#pragma unroll
    for (int k = 0; k < NT; ++k) M = fmaxf(M, xml[k][lane].x);
#pragma unroll
    for (int k = 0; k < NT; ++k) {
      const float2 t = xml[k][lane];
      w[k] = t.x == -INFINITY ? 0.f : __expf(t.x - M);
      l += w[k] * t.y;
    }
    if (wave == 0 && g == 0) *reinterpret_cast<float2*>(mlp) = make_float2(M, l);
  }
  for (int c = wave; c < DB * 4; c += NT) {          // each wavefront adds up its share of the features
    float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
    for (int k = 0; k < NT; ++k) {
      const float4 t = xch[k][c][lane];
      const float wk = SOFTMAX ? w[k] : 1.0f;
      v.x += wk * t.x; v.y += wk * t.y; v.z += wk * t.z; v.w += wk * t.w;
    }
    *reinterpret_cast<float4*>(dst + (c >> 2) * 32 + 8 * (c & 3)) = v;
  }
}

// ---- u | v | q | k projection: SiLU(xh W1^T + b1) and where it goes ---------------------------------
struct F1F32Params {
  const float* A;            // xh [rows, d]
  const float* W;            // W1 [4d, d]
  const float* bias;
  float* u; float* q; float* knew; float* vnew; float* sfx;
  const UserDesc* users;
  RowTables rt;
  int d, dh, n_prows, layer, row_begin, row_end, n_mtiles;
  ColMap cm;
};

// Stores the four values of rows r0 .. r0+3 (of these kinds, read for v and k only) in feature c of block blk (0 u, 1 v, 2 q, 3 k).
__device__ __forceinline__ void f1_f32_store(const F1F32Params& p, int blk, int c, int r0, const float (&v)[4], const int (&kinds)[4]) {
  const int head = c / p.dh, f = c - head * p.dh;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int r = r0 + i;
    if (r >= p.row_end) return;
    if (blk == 0 || blk == 2) { (blk == 0 ? p.u : p.q)[(size_t)r * p.d + c] = v[i]; continue; }
    const int kind = kinds[i];
    if (kind == kRowCand) { (blk == 3 ? p.knew : p.vnew)[(size_t)(r - p.n_prows) * p.d + c] = v[i]; continue; }
    const UserDesc& ud = p.users[p.rt.user[r]];
    const int idx = p.rt.idx[r], rr = idx % kTile;
    float* base = kind == kRowPrefix ? const_cast<float*>(reinterpret_cast<const float*>(ud.kv)) + ud.kv_tile0 + (int64_t)(idx / kTile) * ud.kv_tile_stride +
                                           (int64_t)p.layer * ud.kv_layer_stride
                                     : p.sfx + ud.sfx_tile0 + (int64_t)(idx / kTile) * (2 * kTile * p.d);
    base += (int64_t)head * 2 * kTile * p.dh;
    base[blk == 3 ? KvLayout<float>::k_off(rr, f, p.dh) : KvLayout<float>::v_off(rr, f, p.dh)] = v[i];
  }
}

// A wavefront multiplies 32*TB tokens by 32*TB features over k, operands straight from row-major memory, PF groups of 8 k
// in flight.  KSLICE = 0: four wavefronts as 2 x 2 such blocks, each over the whole of k.  KSLICE = d/4 (TB = 1): the four
// take a quarter of k each of ONE 32 x 32 block and add in LDS -- for launches of a few hundred rows, where it is the
// length of the k loop that counts (64 cycles an MFMA, k/2 of them: 3.4 us at d = 256) and not the traffic.  At its 64 (or
// fewer) k a wavefront asks for both operands whole, and for the bias and row kinds its end needs, before its first product:
// 512 rows at d = 256 11.2 -> 8.5 us, the d = 64 request's 16 rows 5.2 -> 4.0 us a launch.
template <int TB, int KSLICE>
__global__ __launch_bounds__(256, TB == 1 ? 4 : 2) void f1_f32_kernel(F1F32Params p) {
  constexpr bool KSPLIT = KSLICE > 0;
  constexpr int PF = KSPLIT ? (KSLICE >= 64 ? 8 : KSLICE / 8) : 2, WG = KSPLIT ? 32 : 64 * TB;  // tokens (and features) of a workgroup
  __shared__ float red[KSPLIT ? 4 : 1][KSPLIT ? 16 : 1][64];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), l32 = lane & 31, g = lane >> 5;
  const int nt_blk = p.cm.d / WG, n_nt = p.cm.nblk * nt_blk, total = p.n_mtiles * n_nt;
  const int logical = xcd_remap(blockIdx.x, total);
  if (logical >= total) return;
  const int mt = logical / n_nt, nt = logical - mt * n_nt;
  const int blk = p.cm.blk[nt / nt_blk];
  const int m0 = p.row_begin + mt * WG + (KSPLIT ? 0 : (wave >> 1) * 32 * TB);
  const int c0 = (nt % nt_blk) * WG + (KSPLIT ? 0 : (wave & 1) * 32 * TB);   // first feature inside the block
  const int k_len = KSPLIT ? KSLICE : p.d, k0 = KSPLIT ? wave * k_len : 0;
  const float *a[TB], *w[TB];
#pragma unroll
  for (int i = 0; i < TB; ++i) {
    a[i] = p.A + (size_t)min(m0 + 32 * i + l32, p.row_end - 1) * p.d + k0 + 4 * g;
    w[i] = p.W + (size_t)(blk * p.d + c0 + 32 * i + l32) * p.d + k0 + 4 * g;
  }
  f32x16_t acc[TB][TB];                              // tokens x features: lane = feature, tokens 8*(e/4) + 4g + e%4
#pragma unroll
  for (int i = 0; i < TB; ++i)
#pragma unroll
    for (int j = 0; j < TB; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;
  // what the end of the cut form waits for, asked for now: its bias and the kinds of the four rows this wavefront finishes
  float b_early = 0.f;
  int kinds[4] = {};
  if constexpr (KSPLIT) {
    b_early = p.bias[blk * p.d + c0 + l32];
    if (blk == 1 || blk == 3)
#pragma unroll
      for (int i = 0; i < 4; ++i) kinds[i] = p.rt.kind[min(m0 + 8 * wave + 4 * g + i, p.row_end - 1)];
  }
  float4 af[PF][TB], wf[PF][TB];
  auto load = [&](int s, int k) {
#pragma unroll
    for (int i = 0; i < TB; ++i) { af[s][i] = *reinterpret_cast<const float4*>(a[i] + k); wf[s][i] = *reinterpret_cast<const float4*>(w[i] + k); }
  };
#pragma unroll
  for (int s = 0; s < PF; ++s)
    load(s, min(8 * s, k_len - 8));
  if constexpr (KSPLIT) __builtin_amdgcn_sched_barrier(0);   // all of them before the first product: the compiler would spread them to save registers
  for (int k = 0; k < k_len; k += 8 * PF) {
#pragma unroll
    for (int s = 0; s < PF; ++s) {
      if (k + 8 * s >= k_len) break;                 // (k_len is a multiple of 16)
      float4 ca[TB], cw[TB];
#pragma unroll
      for (int i = 0; i < TB; ++i) { ca[i] = af[s][i]; cw[i] = wf[s][i]; }
      if (8 * PF != KSLICE) load(s, min(k + 8 * (s + PF), k_len - 8));       // unconditional, so that the compiler can count what is outstanding
#pragma unroll
      for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int i = 0; i < TB; ++i)
#pragma unroll
          for (int j = 0; j < TB; ++j) acc[i][j] = mfma32_f32(f4_at(ca[i], t), f4_at(cw[j], t), acc[i][j]);
    }
  }
  if constexpr (KSPLIT) {
#pragma unroll
    for (int e = 0; e < 16; ++e) red[wave][e][lane] = acc[0][0][e];
    __syncthreads();
    float v[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int e = 4 * wave + i;                    // this wavefront finishes tokens 8*wave + 4g + i
      v[i] = silu_f32(((red[0][e][lane] + red[1][e][lane]) + (red[2][e][lane] + red[3][e][lane])) + b_early);
    }
    f1_f32_store(p, blk, c0 + l32, m0 + 8 * wave + 4 * g, v, kinds);
  } else {
#pragma unroll
    for (int j = 0; j < TB; ++j) {
      const int c = c0 + 32 * j + l32;
      const float b = p.bias[blk * p.d + c];
#pragma unroll
      for (int i = 0; i < TB; ++i)
#pragma unroll
        for (int e4 = 0; e4 < 4; ++e4) {
          float v[4];
#pragma unroll
          for (int x = 0; x < 4; ++x) v[x] = silu_f32(acc[i][j][4 * e4 + x] + b);
          int kinds[4] = {};
          if (blk == 1 || blk == 3)
#pragma unroll
            for (int x = 0; x < 4; ++x) kinds[x] = p.rt.kind[min(m0 + 32 * i + 8 * e4 + 4 * g + x, p.row_end - 1)];
          f1_f32_store(p, blk, c, m0 + 32 * i + 8 * e4 + 4 * g, v, kinds);
        }
    }
  }
}

// ---- layer tail: combine, gate, output projection, residual, next LayerNorm or score head ------------
// As in the 16-bit path everything between the attention and the next projections is local to a row: a workgroup takes 16
// rows over the full width.  Each of its 16 wavefronts gates a row (lane = d/64 features) into LDS; the product is feature-major
// (16x16x4: a lane ends up with 4 consecutive features of one token), W2 streamed from L2 straight into registers, PF
// groups of 16 k ahead, the two that share the rows' lines together; LayerNorm statistics by two lane exchanges and one exchange between
// wavefronts.  512 rows at d = 256: 12.2 us (13.4 with the groups apart), bound by the chain of trips to memory and by W2 (256 KiB) through one
// compute unit's path.  With the groups apart, more of W2 in flight, up to a wavefront's whole share of it in registers with the residual row, made
// it 15.4 us.
struct TailF32Params {
  const float* part; int nsplit; size_t split_stride;
  const float* ml; size_t ml_stride; int n_heads;   // softmax form
  const float* u; const float* q; const float* knew; const float* vnew;
  const float *gate_gain, *gate_offs;
  const float *W, *bias;     // W2 [d, d], b2
  float* x;                  // residual stream, updated in place
  float* xh;                 // LN(x) for the next layer; nullptr: none wanted
  const float *gain, *offs;  // next layer's input LayerNorm, or the score head's
  RowTables rt;
  int n_prows, dh, row_begin, row_end;
  float alpha, eps;
  const float* w_score; float b_score; float* scores;   // last layer of a ranking call
};

template <int D, bool SM>
__global__ __launch_bounds__(1024) void tail_f32_kernel(TailF32Params p) {
  constexpr int E = D / 64, NW = D >= 256 ? 16 : D / 16;   // wavefronts that take part in the product (all 16 gate a row each)
  constexpr int FB = D / 16 / NW, MS = D / 16, PF = FB >= 4 ? 2 : FB == 2 ? 4 : MS >= 8 ? 8 : 4, YS = D + 4;
  constexpr int NB = E >= 16 ? 1 : E >= 8 ? (SM ? 2 : 4) : 8;   // partial sums of the row in flight
  __shared__ float ys[16][YS];                       // rows 16 bytes apart in banks: 16 lanes' 16-byte reads take 64 banks
  __shared__ float red[3][NW][16];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int row0 = p.row_begin + blockIdx.x * 16;
  const int tk = lane & 15, g4 = lane >> 4;
  const bool product = wave < NW;

  // this wavefront's row: everything that depends on no other load first
  const int r = min(row0 + wave, p.row_end - 1);
  const bool real = row0 + wave < p.row_end;
  const size_t base = (size_t)r * D + lane * E;
  float pb[NB][E];
  auto load_parts = [&](int s0) {
#pragma unroll
    for (int k = 0; k < NB; ++k)
      if (s0 + k < p.nsplit) ld_row_run<float, E>(p.part + (s0 + k) * p.split_stride + base, pb[k]);
  };
  load_parts(0);
  float ug[E], qs[E], ks[E], vs[E], gg[E], go[E];
  ld_row_run<float, E>(p.u + base, ug);
  const bool new_row = r >= p.n_prows;               // only a new row can be a candidate, which has q, k and v rows
#pragma unroll
  for (int i = 0; i < E; ++i) qs[i] = ks[i] = vs[i] = 0.f;
  if (new_row) {
    const size_t nb = (size_t)(r - p.n_prows) * D + lane * E;
    ld_row_run<float, E>(p.q + base, qs);
    ld_row_run<float, E>(p.knew + nb, ks);
    ld_row_run<float, E>(p.vnew + nb, vs);
  }
  const int kind = p.rt.kind[r], seen = p.rt.lim[r];
  float ms[8], ls[8];
  if constexpr (SM) {
    const float* mlr = p.ml + ((size_t)r * p.n_heads + lane * E / p.dh) * 2;
#pragma unroll
    for (int s = 0; s < 8; ++s) {
      const float2 t = *reinterpret_cast<const float2*>(mlr + min(s, p.nsplit - 1) * p.ml_stride);
      ms[s] = s < p.nsplit ? t.x : -INFINITY;
      ls[s] = t.y;
    }
  }
  constexpr bool EARLY = E < 16;                     // d = 1024: the registers do not allow it
  if constexpr (EARLY) {
    ld_row_run<float, E>(p.gate_gain + lane * E, gg);
    ld_row_run<float, E>(p.gate_offs + lane * E, go);
  }
  // first weight fragments
  const float* w[FB];
  float4 wf[PF][FB];
#pragma unroll
  for (int j = 0; j < FB; ++j) w[j] = p.W + (size_t)(((product ? wave : 0) * FB + j) * 16 + tk) * D + 4 * g4;
  auto first_w = [&]() {
#pragma unroll
    for (int s = 0; s < PF; ++s)
#pragma unroll
      for (int j = 0; j < FB; ++j) wf[s][j] = *reinterpret_cast<const float4*>(w[j] + 16 * s);
  };
  if constexpr (EARLY) first_w();

  const bool cand = kind == kRowCand;
  float o[E], n = (float)seen, dot = 0.f, M = -INFINITY, l = 0.f;
#pragma unroll
  for (int i = 0; i < E; ++i) { o[i] = 0.f; dot += qs[i] * ks[i]; }
  for (int m = (p.dh / E) >> 1; m > 0; m >>= 1) dot += __shfl_xor(dot, m, 64);   // lanes of one head are consecutive
  const float tself = dot * p.alpha;
  if constexpr (SM) {                                // pieces and the own key by weights exp(m_s - M)
    M = cand ? tself : -INFINITY;
#pragma unroll
    for (int s = 0; s < 8; ++s) M = fmaxf(M, ms[s]);
  }
#pragma unroll
  for (int s0 = 0; s0 < 8; s0 += NB) {
    if (s0 >= p.nsplit) break;
    if (s0 > 0) load_parts(s0);
#pragma unroll
    for (int k = 0; k < NB; ++k) {
      if (s0 + k >= p.nsplit) break;
      float wt = 1.0f;
      if constexpr (SM) {
        wt = ms[s0 + k] == -INFINITY ? 0.f : __expf(ms[s0 + k] - M);
        l += wt * ls[s0 + k];
      }
#pragma unroll
      for (int i = 0; i < E; ++i) o[i] += wt * pb[k][i];
    }
  }
  if (cand) {
    const float pe = SM ? __expf(tself - M) : silu_f32(tself);
#pragma unroll
    for (int i = 0; i < E; ++i) o[i] += pe * vs[i];
    l += pe;
    n += 1.0f;
  }
  const float inv_n = 1.0f / (SM ? l : n);
#pragma unroll
  for (int i = 0; i < E; ++i) o[i] *= inv_n;
  {
    float mean, rstd, y[E];
    ln_stats<E>(o, D, p.eps, mean, rstd);
    if constexpr (!EARLY) {
      ld_row_run<float, E>(p.gate_gain + lane * E, gg);
      ld_row_run<float, E>(p.gate_offs + lane * E, go);
    }
#pragma unroll
    for (int i = 0; i < E; ++i) y[i] = real ? ((o[i] - mean) * rstd * gg[i] + go[i]) * ug[i] : 0.f;
    store_row_run<float, E, false>(&ys[0][0], wave, lane, YS, y);
  }
  if constexpr (!EARLY) first_w();
  // element e of acc[j] is feature (wave*FB + j)*16 + 4*g4 + e.  The product is summed by itself and added to the residual row
  // once, at the end: sums that start from the residual value, which is much larger, round to its last place in every step
  // (scores of the two-layer d = 64 model 4.9e-7 from the same model in float64, against 1.2e-7)
  const int row = row0 + tk;
  const bool live = row < p.row_end;
  float* xrow = p.x + (size_t)(live ? row : row0) * D;
  f32x4v_t acc[FB];
  float4 xv[FB], bv[FB];
#pragma unroll
  for (int j = 0; j < FB; ++j) {
    const int c = ((product ? wave : 0) * FB + j) * 16 + 4 * g4;
    xv[j] = *reinterpret_cast<const float4*>(xrow + c);
    bv[j] = *reinterpret_cast<const float4*>(p.bias + c);
    acc[j] = f32x4v_t{0.f, 0.f, 0.f, 0.f};
  }
  __syncthreads();
  const float* yl = &ys[tk][4 * g4];
  if (product) for (int m0 = 0; m0 < MS; m0 += PF) {
#pragma unroll
    for (int s = 0; s < PF; ++s) {
      const float4 y = *reinterpret_cast<const float4*>(yl + 16 * (m0 + s));
#pragma unroll
      for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int j = 0; j < FB; ++j) acc[j] = mfma16_f32(f4_at(wf[s][j], t), f4_at(y, t), acc[j]);
      // (the next fragments by twos: two groups of 16 k are one 128-byte line of each row, and sixteen wavefronts ask for more between one
      // group and the next than the L1 holds, so that it fetched every line twice.  By fours, fewer are in flight: d = 512 344 -> 349 us a call.
      // Unconditional, so that the compiler can count what is outstanding.)
      if (s & 1) {
#pragma unroll
        for (int j = 0; j < FB; ++j)
#pragma unroll
          for (int h = 1; h >= 0; --h) wf[s - h][j] = *reinterpret_cast<const float4*>(w[j] + 16 * min(m0 + s - h + PF, MS - 1 - h));
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  }
  const bool want_score = p.scores != nullptr;
  float s1 = 0.f;
#pragma unroll
  for (int j = 0; j < FB; ++j) {
    const int c = (wave * FB + j) * 16 + 4 * g4;
    acc[j][0] = xv[j].x + (acc[j][0] + bv[j].x); acc[j][1] = xv[j].y + (acc[j][1] + bv[j].y);
    acc[j][2] = xv[j].z + (acc[j][2] + bv[j].z); acc[j][3] = xv[j].w + (acc[j][3] + bv[j].w);
    if (product && live && !want_score) *reinterpret_cast<float4*>(xrow + c) = make_float4(acc[j][0], acc[j][1], acc[j][2], acc[j][3]);
    s1 += (acc[j][0] + acc[j][1]) + (acc[j][2] + acc[j][3]);
  }
  if (p.xh == nullptr && !want_score) return;        // uniform over the grid
  // sum over the row: this lane's features, the four lanes of the token, the wavefronts
  auto row_sum = [&](float v, int k) {
    v += __shfl_xor(v, 16, 64);
    v += __shfl_xor(v, 32, 64);
    if (product && g4 == 0) red[k][wave][tk] = v;
    __syncthreads();
    float t = 0.f;
#pragma unroll
    for (int wv = 0; wv < NW; ++wv) t += red[k][wv][tk];
    return t;
  };
  const float mean = row_sum(s1, 0) * (1.0f / (float)D);
  float s2 = 0.f;
#pragma unroll
  for (int j = 0; j < FB; ++j)
#pragma unroll
    for (int e = 0; e < 4; ++e) { const float c = acc[j][e] - mean; s2 += c * c; }
  const float rstd = rsqrtf(row_sum(s2, 1) * (1.0f / (float)D) + p.eps);
  float sc = 0.f;
#pragma unroll
  for (int j = 0; j < FB; ++j) {
    if (!product) break;
    const int c = (wave * FB + j) * 16 + 4 * g4;
    const float4 gg = *reinterpret_cast<const float4*>(p.gain + c), oo = *reinterpret_cast<const float4*>(p.offs + c);
    float4 z;
    z.x = (acc[j][0] - mean) * rstd * gg.x + oo.x;
    z.y = (acc[j][1] - mean) * rstd * gg.y + oo.y;
    z.z = (acc[j][2] - mean) * rstd * gg.z + oo.z;
    z.w = (acc[j][3] - mean) * rstd * gg.w + oo.w;
    if (want_score) {
      const float4 ww = *reinterpret_cast<const float4*>(p.w_score + c);
      sc += (z.x * ww.x + z.y * ww.y) + (z.z * ww.z + z.w * ww.w);
    } else if (live) {
      *reinterpret_cast<float4*>(p.xh + (size_t)row * D + c) = z;
    }
  }
  if (want_score) {
    const float total = row_sum(sc, 2);
    if (wave == 0 && g4 == 0 && live && p.rt.kind[row] == kRowCand) p.scores[p.rt.src[row]] = total + p.b_score;
  }
}

}  // namespace relaygr
