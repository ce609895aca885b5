// The plan of a call's attention work: its row tiles, how a launch's row tiles are cut along the keys, and how many partial
// sums every row of the row space then has.  The list of work items is made on the host and the rows' entries on the GPU,
// and the layer tail reads as many partial sums as a row's entry says, so both are worked out by the functions here.
// No HIP in this file: the tests compile it with the host compiler.
#pragma once

#include <stdint.h>

#include <algorithm>
#include <vector>

#ifdef __HIP__
#define RELAYGR_HD __host__ __device__ __forceinline__
#else
#define RELAYGR_HD inline
#endif

namespace relaygr {

constexpr int kTile = 64;   // tokens per K/V tile

// kRowPad: filler between users in the prefix region of the row space (prefix rows of a user start
// at an aligned row so that GEMM tiles never straddle users); it carries the user and a position >= L.
enum RowKind : int32_t { kRowPrefix = 0, kRowSuffix = 1, kRowCand = 2, kRowPad = 3 };

struct UserDesc {
  const void* kv;          // space holding this user's prefix K/V (pool slab or scratch)
  int64_t kv_tile0;        // element offset of the user's tile 0, layer 0, head 0
  int64_t kv_tile_stride;  // elements between consecutive tiles
  int64_t kv_layer_stride; // elements between layers (0 in single-layer scratch)
  int64_t sfx_tile0;       // element offset of the user's suffix tile 0 in the suffix scratch space
  int32_t L, S, M;
  int32_t prow0;           // first prefix row of this user in the call's row space, -1 if not computed
  int32_t nrow0;           // first new row (suffix rows, then candidates), -1 if the call has none
  int32_t prefix_src0, suffix_src0, cand_src0;  // first row in each embedding array
  int32_t parts, parts_last;   // 16-bit path: partial sums of a new row of this user, in every layer but the last / in the last
};
static_assert(sizeof(UserDesc) == 80, "UserDesc layout");

// One attention work item: nrows (<= rows per workgroup) consecutive rows of one user, with everything about the user that
// the attention kernels need (a workgroup's start is a chain of dependent loads: this is one of them instead of three).
struct AttnTile {
  int32_t user;
  int32_t row0;     // first row in the call's row space
  int32_t nrows;
  int32_t kind;     // 0: prefix rows (causal over the prefix); 1: new rows
  int32_t pos0;     // prefix rows: position of row0 in the prefix; new rows: index among new rows
  // 16-bit kernel: an item is one of `parts` pieces of its rows' key sequence, key tiles [t0, t1) of the concatenated list
  // [prefix tiles | suffix tiles], and writes partial sum number `part`
  int32_t t0, t1;
  int32_t part : 16, parts : 16;   // (one word, which a kernel reads with the scalars around it; a 16-bit field takes a vector load)
  const void* kv;          // the user's prefix tile 0, layer 0, head 0 (pool slab or scratch)
  int64_t kv_tile_stride;  // elements between its tiles
  int64_t sfx_tile0;       // UserDesc::sfx_tile0
  int32_t L, S;
  // elements between the layers of a tile: 0 in single-layer scratch (a pool of one layer has the same tile stride, and layer 0)
  RELAYGR_HD int64_t layer_stride(int d) const { return kv_tile_stride == (int64_t)2 * kTile * d ? 0 : (int64_t)2 * kTile * d; }
  // keys of [prefix | suffix] that local row lr sees; 0 beyond the item's rows
  RELAYGR_HD int lim(int lr) const {
    const int t = pos0 + lr;
    return lr >= nrows ? 0 : kind == 0 || t < S ? (kind == 0 ? t + 1 : L + t + 1) : L + S;
  }
};
static_assert(sizeof(AttnTile) == 64, "AttnTile layout");

// A row's entry in the row tables: its user, kind, index inside that user's prefix / suffix / candidates, number of keys of
// [prefix | suffix] it sees, row in the embedding array of its kind, and attention partial sums (RowTables::parts).
struct RowEntry { int user, kind, idx, lim, src, parts; };

// Pieces of the key sequence of the causal work item that starts at position pos0 (a function of the position alone, so
// that the layer tail and the host agree without a table).
RELAYGR_HD int causal_parts(int pos0, int tile_rows, int piece_tiles) {
  return ((pos0 + tile_rows) / kTile + piece_tiles - 1) / piece_tiles;
}

// Entry of row t of a user's prefix rows (filler rows behind the prefix included), or of its new rows (suffix, then candidates).
RELAYGR_HD RowEntry row_entry_at(const UserDesc& ud, int user, bool prefix_region, int t, int tile_rows, int piece_tiles) {
  RowEntry e;
  e.user = user;
  if (prefix_region) {
    e.idx = t;
    if (t < ud.L) { e.kind = kRowPrefix; e.lim = t + 1; e.src = ud.prefix_src0 + t; }
    else          { e.kind = kRowPad; e.lim = 0; e.src = 0; }
    // (a filler row's sums are read and dropped; behind the user's last row tile its position could ask for more than any real row has)
    e.parts = t < ud.L ? causal_parts(t / tile_rows * tile_rows, tile_rows, piece_tiles) : 1;
  } else {
    e.parts = ud.parts | ud.parts_last << 8;
    if (t < ud.S) { e.kind = kRowSuffix; e.idx = t; e.lim = ud.L + t + 1; e.src = ud.suffix_src0 + t; }
    else          { e.kind = kRowCand; e.idx = t - ud.S; e.lim = ud.L + ud.S; e.src = ud.cand_src0 + e.idx; }
  }
  return e;
}

// Key tiles in a row tile's list [prefix | suffix].
inline int key_tiles(const AttnTile& a) {
  return a.kind == 0 ? (a.pos0 + a.nrows + kTile - 1) / kTile : (a.L + kTile - 1) / kTile + (a.S + kTile - 1) / kTile;
}

// 128-row blocks of a work item of the 16-bit kernel: two 32-row blocks for each of four wavefronts (d_head 128: one for each of eight).  It reads half as
// much L2 (d_head 64: and LDS) per score element with 256-row items; they are used when that still yields at least one workgroup per compute unit.
inline int attn_row_blocks(const std::vector<UserDesc>& users, int heads, int dh) {
  if (dh != 64 && dh != 128) return 1;
  int64_t items256 = 0;
  for (const UserDesc& ud : users) {
    if (ud.nrow0 >= 0) items256 += (ud.S + ud.M + 255) / 256;
    if (ud.prow0 >= 0) items256 += (ud.L + 255) / 256;
  }
  return items256 * heads >= 256 ? 2 : 1;
}

// The call's row tiles of at most tile_rows rows: new rows, and the prefix rows that are computed in this call.
inline void attn_row_tiles(const std::vector<UserDesc>& users, int tile_rows, std::vector<AttnTile>& rows_new, std::vector<AttnTile>& rows_prefix) {
  for (int u = 0; u < (int)users.size(); ++u) {
    const UserDesc& ud = users[u];
    const int Tn = ud.S + ud.M;
    if (ud.nrow0 >= 0)
      for (int t0 = 0; t0 < Tn; t0 += tile_rows) rows_new.push_back({u, ud.nrow0 + t0, std::min(tile_rows, Tn - t0), 1, t0, 0, 0, 0, 1, nullptr, ud.kv_tile_stride, ud.sfx_tile0, ud.L, ud.S});
    if (ud.prow0 >= 0)
      for (int i0 = 0; i0 < ud.L; i0 += tile_rows) rows_prefix.push_back({u, ud.prow0 + i0, std::min(tile_rows, ud.L - i0), 0, i0, 0, 0, 0, 1, nullptr, ud.kv_tile_stride, ud.sfx_tile0, ud.L, ud.S});
  }
}

// 16-bit attention: how a launch's row tiles (each with its list of 64-key tiles) are cut into pieces along the keys.
// The chip takes `slots` workgroups at a time and deals the list out longest first.  Unequal items: a launch is done soon after
// total / slots key tiles a slot unless single items are longer than that (one user's causal prefill has one item of all key
// tiles and one of two, a jagged batch one user of 16 384 keys among short ones), so pieces are cut to at most that share.  Items
// of about the same length: into as many pieces each as fit the chip at once, for one more would put a third workgroup on some
// compute units, or a second on some of those that a pair of pieces fills, and the launch would wait for it (12 users of 4096 keys
// and 300 candidates at d = 256: 4 pieces 255 us a call, 3 pieces 200; 40 of 1024 keys and 128 candidates at d = 512: 2 pieces
// 690, uncut 636).  Only launches of less than kPieceRounds rounds are cut, as there is too little behind their long items to hide
// them: each further piece of a row is an fp32 partial sum more for the layer tail to read, and so a piece has kMinPieceTiles key
// tiles (a workgroup's own start and end cost about as much as six).  Equal items of at most 32 rows are one wavefront's work each,
// and three of a workgroup's four only help to move tiles: their chain is what the launch takes, and where two pieces each fit the
// chip they are cut in two from kMinPieceTiles / 2 on (512 keys, us a call uncut and in two pieces of 4 tiles: 40 users of 32
// candidates at d = 256 103 / 99.5, 30 at d = 512 and d_head 128 147 / 137; with 100 candidates, 20 users at d = 512 153 / 159).
// Launches that leave more than half of the slots free are another matter: their pieces run by themselves, and the shorter
// chain is worth more than the sums.  Where a call computes no prefix, its rows are cut into as many pieces as keep half of the
// slots free, of no less than kFinePieceTiles.  (d = 512, one user, us a call in pieces of 8 / 4 / 2 / 1 tiles: 512 keys and 64
// candidates 257 / 238 / 231 / 231, 1024 and 512 263 / 250 / 254; 2048 and 64 in pieces of 8 / 4 263 / 247.  More than half full:
// 8 users at d = 128 with 2048 keys and 272 new rows, 240 pieces of 7 tiles 115, 336 of 5 126; d = 1024, 2048 keys and 512
// candidates, 128 pieces of 8 on 256 slots 611, 256 of 4 646.)  It is a number of pieces and no length, so that where it is
// kMaxPieces, up to slots / (2 kMaxPieces) (row tile, head) pairs, a row's sums do not depend on how long the histories of the call's other
// users are.
// Lists with prefix rows are of unequal items that thin out towards their end, and small ones are launches of a few dozen workgroups: their least
// piece is kMinCausalPieceTiles.  How far that pays is a matter of the slots that the list fills uncut: three eighths of them without new rows, and
// three sixteenths with new rows, whose sums the last layer reads as well (us a call with at least 8 / 4 tiles, d = 256 and 512 of 4 and 8 layers.
// Pre-inference of 600 keys 66.2 / 60.1 and 189 / 178, four users of 600 85.6 / 81.2 and 273 / 267, of 1000 92.1 / 90.4 and, at half of the slots,
// 313 / 322; 16 users of 1000 194.8 / 204.7.  Full recompute of 600 keys and 64 candidates 82.5 / 77.1 and 216 / 208, of 1000 and 64 255 / 248; beyond
// the line four users of 1000 and 256, one of them uncached, 278 / 286, 32 users of 1000 and 64, nine uncached, 213 / 239.)
constexpr int kMinPieceTiles = 8, kMinCausalPieceTiles = 4, kFinePieceTiles = 2, kMaxPieces = 8, kPieceRounds = 4, kMaxSlots = 512;
inline int least_piece(size_t rows_new, size_t rows_prefix, int heads, int slots) {      // (row tiles)
  const bool few = 16 * (rows_new + rows_prefix) * heads <= (size_t)(rows_new ? 3 : 6) * slots;
  return rows_prefix && few ? kMinCausalPieceTiles : kMinPieceTiles;
}
// Pieces a cut list has at most: the launch has under kPieceRounds * kMaxSlots (row tile, head) pairs, each cut in at most kMaxPieces.
inline int max_cut_items(int n_heads) { return kMaxPieces * kPieceRounds * kMaxSlots / n_heads; }
inline int piece_tiles(int64_t items, int64_t total_key_tiles, int least_key_tiles, int most_key_tiles, int most_rows, int slots, int min_piece) {
  if (items >= (int64_t)kPieceRounds * slots || items == 0) return std::max(1, most_key_tiles);
  auto into = [&](int64_t pieces) { pieces = std::max<int64_t>(1, std::min<int64_t>(pieces, kMaxPieces)); return (most_key_tiles + pieces - 1) / pieces; };
  const bool equal = 4 * (int64_t)least_key_tiles >= 3 * (int64_t)most_key_tiles;
  int64_t c = equal ? into(slots / items) : (total_key_tiles + slots - 1) / slots;
  c = std::max<int64_t>({c, min_piece, into(kMaxPieces)});
  if (equal && most_rows <= 32 && slots / items >= 2) c = std::min(c, std::max<int64_t>(kMinPieceTiles / 2, into(2)));
  return (int)std::max<int64_t>(1, std::min<int64_t>(c, most_key_tiles));
}

inline int fine_pieces(int64_t items, int slots) { return items == 0 ? 1 : (int)std::max<int64_t>(1, std::min<int64_t>(slots / 2 / items, kMaxPieces)); }

// Pieces of a row tile of new rows with nk key tiles.
inline int new_row_parts(int nk, int piece, int fine) {
  if (nk == 0) return 1;
  const int parts = std::max((nk + piece - 1) / piece, std::min(fine, (nk + kFinePieceTiles - 1) / kFinePieceTiles));
  const int per = (nk + parts - 1) / parts;
  return (nk + per - 1) / per;                       // (none of them empty)
}

// The launch lists of a call's attention and what the layer tail has to know of them.
struct AttnCut {
  std::vector<AttnTile> all, last;                   // every layer but the last; the last layer (no prefix rows)
  int piece_all = 1 << 20, piece_last = 1 << 20;     // most key tiles of a piece
  int fine = 1;                                      // pieces a row tile of new rows has even if they are shorter (fine_pieces)
  int parts_all = 1, parts_last = 1;                 // partial sums of every row (0: rows differ)
  int nsplit = 1;                                    // partial sums a row can have (fp32: has)
  int gs = 1;                                        // key splits added inside an attention workgroup (AttnParams::gs)
};

// Fills `out` with the pieces of at most `piece` key tiles (new rows: new_row_parts of them), longest first; returns the most pieces of a row tile.
inline int cut_pieces(const std::vector<AttnTile>& rows_new, const std::vector<AttnTile>* rows_prefix, int tile_rows, int piece, int fine, std::vector<AttnTile>& out, int* uniform) {
  out.clear();
  int lo = kMaxPieces + 1, hi = 0;
  auto add = [&](AttnTile a, int parts) {
    const int nk = key_tiles(a), per = (nk + parts - 1) / parts;
    lo = std::min(lo, parts); hi = std::max(hi, parts);
    a.parts = (int16_t)parts;
    for (int k = 0; k < parts; ++k) { a.part = (int16_t)k; a.t0 = std::min(k * per, nk); a.t1 = std::min(a.t0 + per, nk); out.push_back(a); }
  };
  for (const AttnTile& a : rows_new) add(a, new_row_parts(key_tiles(a), piece, fine));
  if (rows_prefix) for (const AttnTile& a : *rows_prefix) add(a, causal_parts(a.pos0, tile_rows, piece));
  std::stable_sort(out.begin(), out.end(), [](const AttnTile& a, const AttnTile& b) { return a.t1 - a.t0 > b.t1 - b.t0; });
  *uniform = hi == 0 ? 1 : lo == hi ? lo : 0;
  return hi;
}

// The 16-bit path's lists.  fits(cut): whether a call cut like that fits its scratch; asked until it does or nothing is cut.
template <class Fits>
inline void cut_attention(const std::vector<AttnTile>& rows_new, const std::vector<AttnTile>& rows_prefix, int heads, int dh, int tile_rows, int n_cus, AttnCut& c, Fits fits) {
  int64_t kt_new = 0, kt_prefix = 0;
  int least_new = 1 << 30, most_new = 0, least_prefix = 1 << 30, most_prefix = 0, most_rows = 0;
  for (const AttnTile& a : rows_new) { const int k = key_tiles(a); kt_new += k; least_new = std::min(least_new, k); most_new = std::max(most_new, k); most_rows = std::max(most_rows, a.nrows); }
  for (const AttnTile& a : rows_prefix) { const int k = key_tiles(a); kt_prefix += k; least_prefix = std::min(least_prefix, k); most_prefix = std::max(most_prefix, k); }
  const int slots = std::min(kMaxSlots, dh == 128 ? n_cus : 2 * n_cus);   // workgroups the chip takes at a time
  c.piece_all = piece_tiles((int64_t)(rows_new.size() + rows_prefix.size()) * heads, (kt_new + kt_prefix) * heads, std::min(least_new, least_prefix),
                            std::max(most_new, most_prefix ? most_prefix + tile_rows / kTile : 0), most_prefix ? tile_rows : most_rows, slots,
                            least_piece(rows_new.size(), rows_prefix.size(), heads, slots));
  c.piece_last = piece_tiles((int64_t)rows_new.size() * heads, kt_new * heads, least_new, most_new, most_rows, slots, kMinPieceTiles);
  const bool one_list = rows_prefix.empty();       // the last layer's list is then the same: not sent twice
  if (one_list) c.fine = fine_pieces((int64_t)rows_new.size() * heads, slots);
  auto cut = [&]() {
    const int h1 = cut_pieces(rows_new, &rows_prefix, tile_rows, c.piece_all, c.fine, c.all, &c.parts_all);
    const int h2 = cut_pieces(rows_new, nullptr, tile_rows, c.piece_last, c.fine, c.last, &c.parts_last);
    c.nsplit = std::max({1, h1, h2});
  };
  for (;;) {
    cut();
    const bool uncut = c.all.size() == rows_new.size() + rows_prefix.size() && c.last.size() == rows_new.size();
    if (uncut || (fits(c) && c.nsplit <= kMaxPieces)) break;
    c.piece_all *= 2; c.piece_last *= 2; c.fine = std::max(1, c.fine / 2);
  }
  // d_head 64: two pieces of a row go to the two wavefront groups of one workgroup, which add their
  // sums in LDS -- half the partial sums for the layer tail to read -- where every row has the same even number of them and
  // half the workgroups still give every compute unit one (with fewer, e.g. one user with 512 candidates, the attention
  // launch itself gets 25 % slower)
  if (dh == 64 && one_list && c.parts_all > 0 && c.parts_all % 2 == 0 && (int64_t)rows_new.size() * heads * (c.parts_all / 2) >= n_cus) {
    c.gs = 2;
    c.fine = 1;
    c.piece_all = c.piece_last = (most_new + c.parts_all / 2 - 1) / (c.parts_all / 2);
    cut();
  }
  if (one_list) c.last.clear();
}

// Partial sums of the users' new rows.
inline void set_user_parts(std::vector<UserDesc>& users, const AttnCut& c) {
  for (UserDesc& ud : users) {
    const int nk = (ud.L + kTile - 1) / kTile + (ud.S + kTile - 1) / kTile;
    ud.parts = new_row_parts(nk, c.piece_all, c.fine);
    ud.parts_last = new_row_parts(nk, c.piece_last, c.fine);
  }
}

}  // namespace relaygr
