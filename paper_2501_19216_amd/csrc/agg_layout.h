// Layout of the fused aggregation (fused.hip), shared by its kernel and by
// the host code that builds its coupling tables.  For one receiver and 16
// channels t the aggregation forms
//   G[be][q][t] = sum_j alpha_ij R_be(r_i - r_j) h_j[q][t]
// on 16 x 16 matrix-core tiles, be (component of the harmonics) along the
// rows and the channels of one component q along the columns, and couples
//   y[o][t] = sum_{be, q} K[o][be][q] G[be][q][t]
// from the accumulators.  K is zero unless the classes of the three
// components match: a rotation by pi about x, y or z maps every real solid
// harmonic to itself up to a sign, so the components fall into four classes
// (agg_class, an element of Z2 x Z2 in two bits) and a product of classes x
// and z lies in class x ^ z alone.  The layout sorts rows and columns by
// class (or by one of the two bits, or not at all, wherever the output
// components that are left fit one tile), so that one coupling step, four
// rows be of one class against one column tile, reaches only the output
// components of one class.
#pragma once

#include "e2f_internal.h"

namespace e2f {

constexpr int kAggMaxNk = (kMaxL + 1) * (kMaxL + 1);

// class of component k = l*l + l + m: bit 0 the parity of m, bit 1 the parity
// of l, flipped for the sine components (m < 0)
constexpr int agg_class(int k) {
  int l = 0;
  while ((l + 1) * (l + 1) <= k) ++l;
  const int m = k - l * l - l;
  return (((l + (m < 0 ? 1 : 0)) & 1) << 1) | ((m < 0 ? -m : m) & 1);
}

// Channels a lane loads at once (a float2 or a float), so agg_vec column tiles
// a component, and the waves per (receiver, column group): as many as keep a
// wave's accumulators (4 registers per row tile and column tile) within about
// 120 registers, so that two waves share a SIMD.  Measured: L = 2, 1,517 atoms
// 46 us with two channels a lane against 61 with the narrow groups of one
// head; L = 3, 10,000 atoms with 32 neighbours 493 us with one channel and one
// wave, 533 with two and two; L = 4, 2,000 atoms 356 us with one channel and
// two waves, 369 with two and four (5,001 atoms 771 and 744, 20,000 alike).
constexpr int agg_vec(int L) { return L <= 2 || L == 5 ? 2 : 1; }
constexpr int agg_waves(int L) { return L <= 3 ? 1 : L == 4 ? 2 : 8; }

struct AggMap {
  int nk;
  int keys;                // 1, 2 or 4: how far components are told apart
  int mt;                  // row tiles
  int ng;                  // groups of four rows with components (group g: tile g / 4, rows 4 k4 + g % 4)
  int nw, tw;              // waves, components (slots) per wave
  int pos[kAggMaxNk];      // row of component be
  int gkey[16];            // key of a group
  int gbe[16][4];          // its components (-1: none)
  int skey[32];            // key of slot i, to be xored with the wave's
  int wkey[8];             // key of a wave
  int slotq[8][32];        // component q of (wave, slot), -1: none
  int rows[4][17];         // component of (key, index), -1: none
  int kkey[kAggMaxNk];     // key and index of output component k
  int kidx[kAggMaxNk];
};

constexpr AggMap agg_map(int L) {
  AggMap a{};
  a.nk = (L + 1) * (L + 1);
  a.mt = (a.nk + 15) / 16;
  a.nw = agg_waves(L);
  int size4[4] = {0, 0, 0, 0};
  for (int k = 0; k < a.nk; ++k) ++size4[agg_class(k)];
  int s2 = 0;
  for (int b = 0; b < 2; ++b) s2 = size4[2 * b] + size4[2 * b + 1] > s2 ? size4[2 * b] + size4[2 * b + 1] : s2;
  a.keys = a.nk <= 16 ? 1 : (s2 <= 16 ? 2 : 4);
  int list[4][kAggMaxNk] = {}, size[4] = {0, 0, 0, 0};
  for (int k = 0; k < a.nk; ++k) {
    const int key = a.keys == 1 ? 0 : (a.keys == 2 ? agg_class(k) >> 1 : agg_class(k));
    a.kkey[k] = key;
    a.kidx[k] = size[key];
    list[key][size[key]++] = k;
  }
  for (int x = 0; x < 4; ++x)
    for (int i = 0; i < 17; ++i) a.rows[x][i] = x < a.keys && i < size[x] ? list[x][i] : -1;
  for (int x = 0; x < a.keys; ++x)
    for (int i = 0; i < size[x]; i += 4, ++a.ng) {
      a.gkey[a.ng] = x;
      for (int j = 0; j < 4; ++j) {
        a.gbe[a.ng][j] = i + j < size[x] ? list[x][i + j] : -1;
        if (i + j < size[x]) a.pos[list[x][i + j]] = 16 * (a.ng / 4) + 4 * j + a.ng % 4;
      }
    }
  // slots: the components of a key dealt to the waves (a wave holds keys / nw
  // keys, or nw / keys waves share one)
  const int kpw = a.keys >= a.nw ? a.keys / a.nw : 1, wpk = a.nw > a.keys ? a.nw / a.keys : 1;
  for (int w = 0; w < 8; ++w)
    for (int i = 0; i < 32; ++i) a.slotq[w][i] = -1;
  for (int lk = 0; lk < kpw; ++lk) {
    int comps = 0;
    for (int x = lk; x < a.keys; x += kpw) comps = size[x] > comps ? size[x] : comps;
    const int slots = (comps + wpk - 1) / wpk;
    for (int i = 0; i < slots; ++i) {
      a.skey[a.tw + i] = lk;
      for (int w = 0; w < a.nw; ++w) {
        a.wkey[w] = wpk > 1 ? w / wpk : w * kpw;
        const int key = a.wkey[w] ^ lk, at = (wpk > 1 ? w % wpk : 0) * slots + i;
        if (at < size[key]) a.slotq[w][a.tw + i] = list[key][at];
      }
    }
    a.tw += slots;
  }
  return a;
}

// Coupling table: one float per lane for the coupling step of group g of a
// slot; four steps to a float4: entry ((w tw + slot) agg_quads + g / 4) * 64 +
// lane, element g % 4.
constexpr int agg_quads(int L) { return (agg_map(L).ng + 3) / 4; }
constexpr int agg_table_floats(int L) { return agg_map(L).nw * agg_map(L).tw * agg_quads(L) * 256; }
// Index table: the row of component be (nk ints), the component of (wave,
// slot) (a missing one repeats the wave's first, its coupling is zero), then
// for each output component key * 16 + index.
constexpr int agg_index_ints(int L) { return 2 * agg_map(L).nk + agg_map(L).nw * agg_map(L).tw; }

static_assert(agg_map(4).keys == 2 && agg_map(4).ng == 7 && agg_map(4).tw == 13,
              "L = 4: two key sets of 13 and 12 components");
static_assert(agg_map(6).tw == 7 && agg_map(6).ng == 13 && agg_map(5).tw == 5 && agg_map(3).tw == 16, "slots per wave");
constexpr bool agg_fits(int L) { return agg_map(L).ng <= 4 * agg_map(L).mt; }
static_assert(agg_fits(0) && agg_fits(1) && agg_fits(2) && agg_fits(3) && agg_fits(4) && agg_fits(5) && agg_fits(6),
              "the groups of rows must fit the row tiles");

// Host: the index and coupling tables for the path weights w (tables.cpp).
struct AggTables {
  std::vector<int> index;
  std::vector<float> coef;
};
AggTables agg_tables(const LayerTables& t, const std::vector<double>& w);
// The coupling as the backward's per-edge products read it (edge_grad.hip):
// element (q ng + g) * 64 + lane of agg_map(L)'s groups and keys, K[o][be][q]
// for o = member lane / 16 of group g and be = member lane % 16 of key gkey[g]
// ^ key(q).
std::vector<float> grad_table(const LayerTables& t, const std::vector<double>& w);

}  // namespace e2f
