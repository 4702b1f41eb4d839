// The j-side coupling and the i-side recouple of the two-kernel form composed
// into one tensor per component of the receiver's harmonics, derived from the
// library's tables by their own indices.  No kernel reads it: the host checks
// compare the fused aggregation's coupling with it (at p_i = 0) and its layouts,
// by whose rows the forward's workspace is sized, with each other.
#pragma once

#include <cmath>

#include "e2f_internal.h"

namespace e2f {

// Up to L = 4 the j-side coupling and the i-side recouple compose into one
// per-receiver matrix F_i = Q_i CG of (L+1)^2 rows k = (o, m) and (L+1)^4
// columns (be, q), be the component of R(p_j) and q that of h_j:
//     y_i[k][c] = sum_{be, q} F_i[k][be, q] G_i[be][q][c],
//     G_i[be][q][c] = sum_j alpha_ij R_be(p_j) h_j[q][c].
// F_i = sum_x R_x(p_i) K_x with fixed tensors K_x (x a component of R(p_i)),
// K_x[k][be, q] = sum over T rows r of Q_i's coefficient of R_x in entry
// (k, r) times CG[r][be, q].  F_i is stored per receiver in the order in which
// the aggregation's waves read it as the A operand of v_mfma_f32_16x16x4f32:
// per q a block of (row tile rt, K tile mt) sub-blocks, each [k4 < kc][l16 <
// rows][s < 4] holding F[16 rt + l16][be][q] at K position 4 k4 + s =
// fuse_kpos(be) of be's tile (zero at positions no component takes).  A tile
// of r components uses kc = ceil(r / 4) groups k4 and ks = ceil(r / kc)
// steps s each (component j of the tile at k4 = j / ks, s = j % ks), so where
// r <= 12 the steps s >= ks hold only zeros and F_i G_i skips them (at
// L = 4 the second tile's 9 components take s < 3).
constexpr int kFuseMaxL = 4;
constexpr int fuse_rows(int nk, int rt) { return nk - 16 * rt < 16 ? nk - 16 * rt : 16; }
constexpr int fuse_kc(int nk, int mt) { return (fuse_rows(nk, mt) + 3) / 4; }
constexpr int fuse_tiles(int nk) { return (nk + 15) / 16; }
constexpr int fuse_ks(int nk, int mt) { return (fuse_rows(nk, mt) + fuse_kc(nk, mt) - 1) / fuse_kc(nk, mt); }
// K position (0 .. 15) of component be inside its tile be / 16
constexpr int fuse_kpos(int nk, int be) {
  return 4 * ((be % 16) / fuse_ks(nk, be / 16)) + (be % 16) % fuse_ks(nk, be / 16);
}
static_assert(fuse_ks(25, 1) == 3 && fuse_kpos(25, 24) == 10 && fuse_kpos(25, 19) == 4 && fuse_kpos(25, 7) == 7 &&
                  fuse_ks(16, 0) == 4 && fuse_ks(1, 0) == 1 && fuse_ks(9, 0) == 3,
              "K positions of the fused layout");
// The K rows of F may stack several filter degrees (alpha / D^f, one pass
// over the edges for several degrees): nkr rows, in segments of (f+1)^2 rows
// per degree f, the j-side component be of degree f's segment at row
// start + be (the plain layer: one segment, nkr = nk).  Rows k stay the nk
// output components; the functions below with nk take rows k or, with nkr,
// K rows.
// offset (floats) of sub-block (rt, mt) inside a q block, rt-major
constexpr int fuse_blk(int nk, int nkr, int rt, int mt) {
  int off = 0;
  for (int a = 0; a < fuse_tiles(nk); ++a)
    for (int b = 0; b < fuse_tiles(nkr); ++b) {
      if (a == rt && b == mt) return off;
      off += 4 * fuse_kc(nkr, b) * fuse_rows(nk, a);
    }
  return off;
}
constexpr int fuse_qblock(int nk, int nkr) { return fuse_blk(nk, nkr, fuse_tiles(nk), 0); }
// floats of one receiver's F, rounded up to 64 (256-byte rows)
constexpr int fuse_stride(int nk, int nkr) { return (nk * fuse_qblock(nk, nkr) + 63) / 64 * 64; }
// position of F[k][kr][q] (kr a K row) in a receiver's row
constexpr int fuse_pos(int nk, int nkr, int k, int kr, int q) {
  return q * fuse_qblock(nk, nkr) + fuse_blk(nk, nkr, k / 16, kr / 16) +
         (fuse_kpos(nkr, kr) / 4 * fuse_rows(nk, k / 16) + k % 16) * 4 + fuse_kpos(nkr, kr) % 4;
}
// K rows of the stacked degrees degs[0 .. nd) (a degree -1: every filter
// degree in one segment of nk rows)
inline int fuse_krows(int nk, const int* degs, int nd) {
  int r = 0;
  for (int s = 0; s < nd; ++s) r += degs[s] < 0 ? nk : (degs[s] + 1) * (degs[s] + 1);
  return r;
}
// The alpha / D^f passes of the fused aggregation, each a set of filter
// degrees stacked in the K rows: below L = 4 one pass of every degree (L, L-1,
// .. 0: 30 K rows at L = 3); at L = 4 (55 rows in all) two passes within two
// K tiles, degrees 3 and 2 (25 rows), then 4, 1 and 0 (30 rows).
struct YnormPass {
  int nd;                   // segments
  int degs[kFuseMaxL + 1];  // their filter degrees
};
constexpr int kYnormMaxPasses = 2;
inline int ynorm_passes(int L, YnormPass* out) {
  if (L == 4) {
    out[0] = YnormPass{2, {3, 2, 0, 0, 0}};
    out[1] = YnormPass{3, {4, 1, 0, 0, 0}};
    return 2;
  }
  out[0] = YnormPass{L + 1, {0, 0, 0, 0, 0}};
  for (int s = 0; s <= L; ++s) out[0].degs[s] = L - s;
  return 1;
}
// K_x by position of F (CSR over the positions 0 .. fuse_stride - 1): the
// entries of position p are idx[e] (the component x) and coef[e] (float64,
// path weights w[a][f][o] included) for e in ptr[p] .. ptr[p+1] - 1.
struct FuseTable {
  std::vector<int> ptr;
  std::vector<int> idx;
  std::vector<double> coef;
};
// degs[0 .. nd): the segments of K rows (fuse_krows): a degree f >= 0 takes
// only the terms of filter degree f (the T rows of j-side degree b with the
// receiver's harmonics of degree u = f - b), for the per-degree weights
// alpha / D^f, at rows start + be of its segment; -1 takes every term (the
// plain layer).  nkr >= fuse_krows: the K rows of the layout (rows past the
// segments hold zeros), so that one degree alone can use the plain layout.
inline FuseTable fuse_table(const LayerTables& t, const std::vector<double>& w, const int* degs, int nd, int nkr) {
  const int nk = t.nk;
  FuseTable ft;
  if (t.L > kFuseMaxL || nkr < fuse_krows(nk, degs, nd)) return ft;
  // first K row of each filter degree's segment (-1: not in this table),
  // and of the segment that takes every term (the plain layer: b + u up to 2L)
  int start[kFuseMaxL + 1], start_all = -1;
  for (int f = 0; f <= kFuseMaxL; ++f) start[f] = -1;
  for (int s = 0, r = 0; s < nd; ++s) {
    if (degs[s] < 0) start_all = r;
    else start[degs[s]] = r;
    r += degs[s] < 0 ? nk : (degs[s] + 1) * (degs[s] + 1);
  }
  std::vector<int> row_b(t.dimT, 0);  // j-side degree of every T row
  for (const Block& B : t.blocks)
    for (int de = 0; de < 2 * B.d + 1; ++de) row_b[B.toff + de] = B.b;
  // dense K[pos][x], accumulated over the T rows r that link a recouple entry
  // (k, r) with a coupling entry (r, be, q)
  const int np = fuse_stride(nk, nkr);
  std::vector<double> K((size_t)np * nk, 0.0), mag((size_t)np * nk, 0.0);
  for (int o = 0; o <= t.L; ++o) {
    const int ncol = t.q_ncol[o];
    for (int m = 0; m < 2 * o + 1; ++m)
      for (int col = 0; col < ncol; ++col) {
        const int s = t.q_slotoff[o] + m * ncol + col;
        const int r = t.q_cols[t.q_coloff[o] + col];
        const int k = o * o + m;
        const int s0 = t.m_rowoff[r], s1 = t.m_rowoff[r + 1];
        const int a = (s1 - s0 - 1) / 2;
        for (int e = t.q_ptr[s]; e < t.q_ptr[s + 1]; ++e) {
          const double cq = t.q_unit[e] * w[t.q_path[e]];
          const int x = t.q_ridx[e];
          int u = 0;  // x = u^2 + gamma: the degree of the receiver's harmonic
          while ((u + 1) * (u + 1) <= x) ++u;
          const int deg = row_b[r] + u;
          int shift = start_all;  // K row of a j-side component be: shift + be
          if (shift < 0) {
            if (deg > kFuseMaxL || start[deg] < 0) continue;
            shift = start[deg];
          }
          for (int sl = s0; sl < s1; ++sl)
            for (int e2 = t.m_ptr[sl]; e2 < t.m_ptr[sl + 1]; ++e2) {
              const size_t at = (size_t)fuse_pos(nk, nkr, k, t.m_ridx[e2] + shift, a * a + sl - s0) * nk + x;
              K[at] += cq * t.m_coef[e2];
              mag[at] += std::fabs(cq * t.m_coef[e2]);
            }
        }
      }
  }
  // sums that cancel to rounding level are zeros of the exact tensor
  ft.ptr.assign(1, 0);
  for (int p = 0; p < np; ++p) {
    for (int x = 0; x < nk; ++x) {
      const double v = K[(size_t)p * nk + x];
      if (v != 0.0 && std::fabs(v) > 1e-13 * mag[(size_t)p * nk + x]) {
        ft.idx.push_back(x);
        ft.coef.push_back(v);
      }
    }
    ft.ptr.push_back((int)ft.idx.size());
  }
  return ft;
}

}  // namespace e2f
