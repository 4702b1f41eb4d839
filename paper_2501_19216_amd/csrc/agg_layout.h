// Layout of the fused aggregation (fused.hip), shared by its kernel and by
// the host code that builds its coupling tables.  For one receiver and DH =
// 16 / P channels of a head the aggregation forms
//   G[be][q][t] = sum_j alpha_ij R_be(r_i - r_j) h_j[q][t]
// on 16 x 16 matrix-core tiles, be (component of the harmonics) along the
// rows and P components q x DH channels t along the columns, and couples
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

// waves per (receiver, column group): as many as keep a wave's accumulators
// (4 registers per row tile and slot) within about 120 registers, so that two
// waves share a SIMD
constexpr int agg_waves(int L, int P) {
  return L == 4 ? (P == 1 ? 2 : 1) : L == 5 ? (P == 4 ? 2 : 4) : L == 6 ? (P == 1 ? 8 : 4) : 1;
}

struct AggMap {
  int nk, dh;
  int keys;                // 1, 2 or 4: how far components are told apart
  int rb;                  // output components of a key per row block of dh: rb blocks
  int mt;                  // row tiles
  int ng;                  // groups of four rows with components (group g: tile g / 4, rows 4 k4 + g % 4)
  int nw, tw;              // waves, column tiles (slots) per wave
  int pos[kAggMaxNk];      // row of component be
  int gkey[16];            // key of a group
  int gbe[16][4];          // its components (-1: none)
  int skey[32];            // key of slot i, to be xored with the wave's
  int wkey[8];             // key of a wave
  int slotq[8][32][4];     // component q of (wave, slot, p), -1: none
  int rows[4][64];         // output component of (key, index), -1: none
  int kkey[kAggMaxNk];     // key and index of output component k
  int kidx[kAggMaxNk];
};

constexpr AggMap agg_map(int L, int P) {
  AggMap a{};
  a.nk = (L + 1) * (L + 1);
  a.dh = 16 / P;
  a.mt = (a.nk + 15) / 16;
  a.nw = agg_waves(L, P);
  int size4[4] = {0, 0, 0, 0};
  for (int k = 0; k < a.nk; ++k) ++size4[agg_class(k)];
  int s2 = 0;
  for (int b = 0; b < 2; ++b) s2 = size4[2 * b] + size4[2 * b + 1] > s2 ? size4[2 * b] + size4[2 * b + 1] : s2;
  a.keys = a.nk <= a.dh ? 1 : (s2 <= a.dh ? 2 : 4);
  int list[4][kAggMaxNk] = {}, size[4] = {0, 0, 0, 0};
  for (int k = 0; k < a.nk; ++k) {
    const int key = a.keys == 1 ? 0 : (a.keys == 2 ? agg_class(k) >> 1 : agg_class(k));
    a.kkey[k] = key;
    a.kidx[k] = size[key];
    list[key][size[key]++] = k;
  }
  int most = 0;
  for (int x = 0; x < a.keys; ++x) most = size[x] > most ? size[x] : most;
  a.rb = (most + a.dh - 1) / a.dh;
  for (int x = 0; x < 4; ++x)
    for (int i = 0; i < 64; ++i) a.rows[x][i] = x < a.keys && i < size[x] ? list[x][i] : -1;
  for (int x = 0; x < a.keys; ++x)
    for (int i = 0; i < size[x]; i += 4, ++a.ng) {
      a.gkey[a.ng] = x;
      for (int j = 0; j < 4; ++j) {
        a.gbe[a.ng][j] = i + j < size[x] ? list[x][i + j] : -1;
        if (i + j < size[x]) a.pos[list[x][i + j]] = 16 * (a.ng / 4) + 4 * j + a.ng % 4;
      }
    }
  // column tiles: the components of a key, P at a time, dealt to the waves
  // (a wave holds keys / nw keys, or nw / keys waves share one)
  const int kpw = a.keys >= a.nw ? a.keys / a.nw : 1, wpk = a.nw > a.keys ? a.nw / a.keys : 1;
  for (int w = 0; w < 8; ++w)
    for (int i = 0; i < 32; ++i)
      for (int p = 0; p < 4; ++p) a.slotq[w][i][p] = -1;
  for (int lk = 0; lk < kpw; ++lk) {
    int tiles = 0;
    for (int x = lk; x < a.keys; x += kpw) tiles = (size[x] + P - 1) / P > tiles ? (size[x] + P - 1) / P : tiles;
    const int slots = (tiles + wpk - 1) / wpk;
    for (int i = 0; i < slots; ++i) {
      a.skey[a.tw + i] = lk;
      for (int w = 0; w < a.nw; ++w) {
        a.wkey[w] = wpk > 1 ? w / wpk : w * kpw;
        const int key = a.wkey[w] ^ lk, tile = (wpk > 1 ? w % wpk : 0) * slots + i;
        for (int p = 0; p < P; ++p)
          if (tile * P + p < size[key]) a.slotq[w][a.tw + i][p] = list[key][tile * P + p];
      }
    }
    a.tw += slots;
  }
  return a;
}

// Coupling table: one float per lane for coupling step m = group * rb + row
// block of a slot; four steps to a float4: entry ((w tw + slot) agg_quads + m
// / 4) * 64 + lane, element m % 4.
constexpr int agg_quads(int L, int P) { return (agg_map(L, P).ng * agg_map(L, P).rb + 3) / 4; }
constexpr int agg_table_floats(int L, int P) {
  return agg_map(L, P).nw * agg_map(L, P).tw * agg_quads(L, P) * 256;
}
// Index table: the row of component be (nk ints), the component of (wave,
// slot, p) (a missing one repeats the slot's first, its coupling is zero),
// then for each output component key * rb * dh + index.
constexpr int agg_index_ints(int L, int P) {
  return 2 * agg_map(L, P).nk + agg_map(L, P).nw * agg_map(L, P).tw * P;
}

static_assert(agg_map(4, 1).keys == 2 && agg_map(4, 1).rb == 1 && agg_map(4, 1).ng == 7 && agg_map(4, 1).tw == 13,
              "L = 4, 16 channels: two key sets of 13 and 12 components");
static_assert(agg_map(6, 2).tw == 7 && agg_map(6, 2).ng == 13 && agg_map(6, 2).rb == 2, "L = 6, 8 channels");
static_assert(agg_map(6, 1).tw == 7 && agg_map(6, 4).tw == 4 && agg_map(5, 1).tw == 9 && agg_map(5, 2).tw == 5 &&
                  agg_map(4, 2).tw == 13 && agg_map(4, 4).tw == 8 && agg_map(3, 1).tw == 16,
              "slots per wave");
constexpr bool agg_fits(int L, int P) { return agg_map(L, P).ng <= 4 * agg_map(L, P).mt; }
static_assert(agg_fits(0, 1) && agg_fits(1, 1) && agg_fits(2, 1) && agg_fits(3, 1) && agg_fits(4, 1) &&
                  agg_fits(5, 1) && agg_fits(6, 1) && agg_fits(0, 2) && agg_fits(1, 2) && agg_fits(2, 2) &&
                  agg_fits(3, 2) && agg_fits(4, 2) && agg_fits(5, 2) && agg_fits(6, 2) && agg_fits(0, 4) &&
                  agg_fits(1, 4) && agg_fits(2, 4) && agg_fits(3, 4) && agg_fits(4, 4) && agg_fits(5, 4) &&
                  agg_fits(6, 4),
              "the groups of rows must fit the row tiles");

// Host: the index and coupling tables for the path weights w (tables.cpp).
struct AggTables {
  std::vector<int> index;
  std::vector<float> coef;
};
AggTables agg_tables(const LayerTables& t, const std::vector<double>& w, int P);
// The coupling as the backward's per-edge products read it (edge_grad.hip):
// element (q ng + g) * 64 + lane of agg_map(L, 1)'s groups and keys, K[o][be][q]
// for o = member lane / 16 of group g and be = member lane % 16 of key gkey[g]
// ^ key(q).
std::vector<float> grad_table(const LayerTables& t, const std::vector<double>& w);

}  // namespace e2f
