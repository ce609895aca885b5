// Host build of the attention plan (csrc/plan.h) and of the launch rules (csrc/launch_rules.h) for tests/plan_util.py: plans one call and
// checks the plan row by row, and says which kernels the call's launches take.
#include <cstdio>
#include <cstring>
#include <vector>

#include "../paper_2601_01712_amd/csrc/launch_rules.h"

using namespace relaygr;

static constexpr int kRowAlign = 256;   // prefix rows of a user start at a multiple of this (16-bit path)

static int complain(char* msg, const char* what, int user, int row, int got, int want) {
  snprintf(msg, 256, "%s: user %d, row or item %d: %d against %d", what, user, row, got, want);
  return 1;
}

// computed[u]: the call computes user u's prefix rows; new_rows: it has suffix and candidate rows (no pre-inference call).
// most_sums: partial sums a row may have for the call to fit its scratch.  info: row blocks, nsplit, gs, items, rows' filler max,
// sums of a row in flight in the layer tail of the last layer and of the others, key tiles from which on two wavefront groups share a piece
// in the SiLU and in the softmax form, key tiles of the longest piece.
extern "C" int plan_check(int n, const int32_t* L, const int32_t* S, const int32_t* M, const uint8_t* computed, int new_rows,
                          int heads, int dh, int n_cus, int most_sums, int32_t* info, char* msg) {
  std::vector<UserDesc> users(n);
  int prow = 0, nrow = 0;
  for (int u = 0; u < n; ++u) {
    UserDesc& ud = users[u];
    memset(&ud, 0, sizeof(ud));
    ud.L = L[u]; ud.S = new_rows ? S[u] : 0; ud.M = new_rows ? M[u] : 0;
    ud.prow0 = computed[u] ? prow : -1;
    if (computed[u]) prow += (ud.L + kRowAlign - 1) / kRowAlign * kRowAlign;
    ud.nrow0 = new_rows ? nrow : -1;
    nrow += ud.S + ud.M;
  }
  for (UserDesc& ud : users) if (ud.nrow0 >= 0) ud.nrow0 += prow;
  const int nq = attn_row_blocks(users, heads, dh), rpt = 128 * nq;
  std::vector<AttnTile> rows_new, rows_prefix;
  attn_row_tiles(users, rpt, rows_new, rows_prefix);
  AttnCut cut;
  cut_attention(rows_new, rows_prefix, heads, dh, rpt, n_cus, cut, [&](const AttnCut& k) { return k.nsplit <= most_sums; });
  set_user_parts(users, cut);
  info[0] = nq; info[1] = cut.nsplit; info[2] = cut.gs; info[3] = (int)cut.all.size(); info[4] = 0;
  info[5] = sums_at_once(cut.parts_last, cut.nsplit); info[6] = sums_at_once(cut.parts_all, cut.nsplit);
  for (int sm = 0; sm < 2; ++sm) info[7 + sm] = attn_shared_tiles(sm, heads, dh, !rows_prefix.empty(), cut, n_cus);
  info[9] = cut.all.empty() ? 0 : cut.all[0].t1 - cut.all[0].t0;

  // every list holds each row tile's pieces once: numbered 0 .. parts - 1, the key tiles in order and without a gap
  const int n_rows = prow + nrow;
  std::vector<int> have_all(n_rows, 0), have_last(n_rows, 0);
  const bool own_last = !rows_prefix.empty();
  for (int which = 0; which < 2; ++which) {
    const std::vector<AttnTile>& list = which && own_last ? cut.last : cut.all;
    std::vector<int>& have = which ? have_last : have_all;
    std::vector<std::vector<const AttnTile*>> at(n_rows);
    for (const AttnTile& a : list) {
      if (a.part < 0 || a.part >= a.parts || a.parts > cut.nsplit) return complain(msg, "piece number", a.user, a.row0, a.part, a.parts);
      if (at[a.row0].empty()) at[a.row0].resize(a.parts, nullptr);
      if ((int)at[a.row0].size() != a.parts || at[a.row0][a.part]) return complain(msg, "piece twice", a.user, a.row0, a.part, a.parts);
      at[a.row0][a.part] = &a;
    }
    for (int r = 0; r < n_rows; ++r) {
      if (at[r].empty()) continue;
      int t = 0;
      for (const AttnTile* a : at[r]) {
        if (!a) return complain(msg, "piece missing", -1, r, 0, (int)at[r].size());
        if (a->t0 != t || a->t1 < a->t0) return complain(msg, "piece start", a->user, r, a->t0, t);
        t = a->t1;
      }
      if (t != key_tiles(*at[r][0])) return complain(msg, "key tiles covered", at[r][0]->user, r, t, key_tiles(*at[r][0]));
      for (int i = 0; i < at[r][0]->nrows; ++i) have[r + i] = (int)at[r].size();
    }
  }

  // and every row's entry says as many sums as its row tile has pieces, filler rows no more than the buffers hold
  for (int u = 0; u < n; ++u) {
    const UserDesc& ud = users[u];
    if (ud.prow0 >= 0)
      for (int t = 0; t < (ud.L + kRowAlign - 1) / kRowAlign * kRowAlign; ++t) {
        const RowEntry e = row_entry_at(ud, u, true, t, rpt, cut.piece_all);
        if (e.kind != (t < ud.L ? kRowPrefix : kRowPad)) return complain(msg, "kind", u, t, e.kind, -1);
        if (e.kind == kRowPad && e.parts > info[4]) info[4] = e.parts;
        if (e.parts < 1 || e.parts > cut.nsplit) return complain(msg, "sums of a prefix-region row", u, t, e.parts, cut.nsplit);
        if (t < ud.L && e.parts != have_all[ud.prow0 + t]) return complain(msg, "sums of a prefix row", u, t, e.parts, have_all[ud.prow0 + t]);
        if (t < ud.L && cut.parts_all && e.parts != cut.parts_all) return complain(msg, "sums of every row", u, t, e.parts, cut.parts_all);
      }
    for (int t = 0; ud.nrow0 >= 0 && t < ud.S + ud.M; ++t) {
      const RowEntry e = row_entry_at(ud, u, false, t, rpt, cut.piece_all);
      const int all = e.parts & 255, last = e.parts >> 8;
      if (all > info[6] || last > info[5]) return complain(msg, "sums in flight", u, t, info[6], all);
      if (all != have_all[ud.nrow0 + t]) return complain(msg, "sums of a new row", u, t, all, have_all[ud.nrow0 + t]);
      if (own_last && last != have_last[ud.nrow0 + t]) return complain(msg, "sums of a new row, last layer", u, t, last, have_last[ud.nrow0 + t]);
      if (cut.parts_all && all != cut.parts_all) return complain(msg, "sums of every new row", u, t, all, cut.parts_all);
      if (cut.parts_last && own_last && last != cut.parts_last) return complain(msg, "sums of every new row, last layer", u, t, last, cut.parts_last);
    }
  }
  return 0;
}

// Pieces of a cached user's first row tile in a ranking of cached users: first and last key tile of each, and whether two wavefront groups share it.
extern "C" int user_pieces(int n, const int32_t* L, const int32_t* S, const int32_t* M, int user, int softmax, int heads, int dh, int n_cus, int32_t* out) {
  std::vector<UserDesc> users(n);
  int nrow = 0;
  for (int u = 0; u < n; ++u) {
    UserDesc& ud = users[u];
    memset(&ud, 0, sizeof(ud));
    ud.L = L[u]; ud.S = S[u]; ud.M = M[u]; ud.prow0 = -1; ud.nrow0 = nrow;
    nrow += ud.S + ud.M;
  }
  const int nq = attn_row_blocks(users, heads, dh);
  std::vector<AttnTile> rows_new, rows_prefix;
  attn_row_tiles(users, 128 * nq, rows_new, rows_prefix);
  AttnCut cut;
  cut_attention(rows_new, rows_prefix, heads, dh, 128 * nq, n_cus, cut, [&](const AttnCut& k) { return k.nsplit <= kMaxPieces; });
  const int least = attn_shared_tiles(softmax != 0, heads, dh, !rows_prefix.empty(), cut, n_cus);
  int count = 0;
  for (const AttnTile& a : cut.all)
    if (a.user == user && a.pos0 == 0) {
      const int32_t piece[3] = {a.t0, a.t1, a.t1 - a.t0 >= least};
      memcpy(out + 3 * a.part, piece, sizeof(piece));
      ++count;
    }
  return count;
}

extern "C" int tail_rows_of(int d, int rows) { return tail_rows(d, rows); }
extern "C" int f1_tile_of(int d, int nblk, int rows, int n_cus) { return (int)f1_tile(d, nblk, rows, n_cus); }
