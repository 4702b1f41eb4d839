// Host check of the fused aggregation's layout and tables (built with g++
// against the library's tables.cpp by test_agg_tables.py; no GPU).  For every
// L it walks the index and coupling tables as the kernel does, on random G, and compares y
// with the sum over the real Clebsch-Gordan tensors; every index is checked
// against its range.  For L <= 4 the coupling is also the composed recouple of
// the local expansion at p_i = 0 (the x = 0 entries of fuse_table).
// Prints two lines per L, "ok" or "FAIL", and exits 1 on a failure.
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <random>

#include "agg_layout.h"
#include "fuse_table.h"

using namespace e2f;

int main() {
  bool all = true;
  for (int L = 0; L <= kMaxL; ++L) {
    const LayerTables t = build_layer_tables(L);
    const int nk = t.nk, L1 = L + 1;
    std::mt19937 g(5 + L);
    std::uniform_real_distribution<double> U(0.2, 1.0), S(-1.0, 1.0);
    std::vector<double> w((size_t)L1 * L1 * L1), K((size_t)nk * nk * nk, 0.0);  // K[o][q][be]
    for (double& v : w) v = U(g);
    for (int a = 0; a <= L; ++a)
      for (int f = 0; f <= L; ++f)
        for (int o = std::abs(a - f); o <= std::min(a + f, L); ++o) {
          const std::vector<double> c = real_cg(a, f, o);
          for (int x = 0; x < 2 * a + 1; ++x)
            for (int y = 0; y < 2 * f + 1; ++y)
              for (int z = 0; z < 2 * o + 1; ++z)
                K[((size_t)(o * o + z) * nk + a * a + x) * nk + f * f + y] +=
                    w[((size_t)a * L1 + f) * L1 + o] * c[((size_t)x * (2 * f + 1) + y) * (2 * o + 1) + z];
        }
    double fdiff = 0.0;
    if (L <= kFuseMaxL) {
      const int every[1] = {-1};
      const FuseTable ft = fuse_table(t, w, every, 1, nk);
      for (int k = 0; k < nk; ++k)
        for (int be = 0; be < nk; ++be)
          for (int q = 0; q < nk; ++q) {
            double v = 0.0;
            const int p = fuse_pos(nk, nk, k, be, q);
            for (int e = ft.ptr[p]; e < ft.ptr[p + 1]; ++e)
              if (ft.idx[e] == 0) v += ft.coef[e];
            int f = 0;  // R_be(r_j - r_i) = (-1)^f R_be(r_i - r_j)
            while ((f + 1) * (f + 1) <= be) ++f;
            fdiff = std::max(fdiff, std::fabs((f & 1 ? -v : v) - K[((size_t)k * nk + q) * nk + be]));
          }
    }
    // the backward's table holds every K[o][be][q] once, and nothing else
    {
      const AggMap a = agg_map(L);
      const std::vector<float> tab = grad_table(t, w);
      std::vector<double> left(K);
      bool fits = tab.size() == (size_t)nk * a.ng * 64;
      for (int q = 0; q < nk && fits; ++q)
        for (int e = 0; e < a.ng * 64; ++e) {
          const int g = e / 64, o = a.gbe[g][e % 64 / 16], be = a.rows[a.gkey[g] ^ a.kkey[q]][e % 16];
          const double v = tab[(size_t)q * a.ng * 64 + e];
          if (o < 0 || be < 0) fits = fits && v == 0.0;
          else left[((size_t)o * nk + q) * nk + be] -= v;
        }
      double most = 0.0;
      for (double v : left) most = std::max(most, std::fabs(v));
      for (int x = 0; x < a.keys; ++x) fits = fits && a.rows[x][16] < 0;  // a key fits the 16 columns
      all = all && fits && most < 1e-6;
      std::printf("L=%d backward table: %s (%.1e left)\n", L, fits && most < 1e-6 ? "ok" : "FAIL", most);
    }
    const AggMap a = agg_map(L);
    const AggTables tab = agg_tables(t, w);
    const int nq = (a.ng + 3) / 4;
    bool ok = (int)tab.index.size() == agg_index_ints(L) && (int)tab.coef.size() == agg_table_floats(L) &&
              nq == agg_quads(L) && a.tw <= 32 && a.ng <= 4 * a.mt;
    std::vector<double> G((size_t)nk * nk), rowG((size_t)16 * a.mt * nk, 0.0);  // [be][q], by row
    for (double& v : G) v = S(g);
    std::vector<int> used(16 * a.mt, 0), seen(nk, 0);
    for (int be = 0; be < nk && ok; ++be) {
      const int pos = tab.index[be];
      ok = pos >= 0 && pos < 16 * a.mt && used[pos]++ == 0;
      for (int q = 0; ok && q < nk; ++q) rowG[(size_t)pos * nk + q] = G[(size_t)be * nk + q];
    }
    std::vector<double> D((size_t)a.nw * a.keys * 16, 0.0);  // [wave][key][row]
    for (int v = 0; v < a.nw && ok; ++v)
      for (int i = 0; i < a.tw; ++i) {
        const int q = tab.index[nk + v * a.tw + i];
        ok = ok && q >= 0 && q < nk;
        if (a.slotq[v][i] >= 0) ok = ok && q == a.slotq[v][i] && seen[q]++ == 0;
        for (int gr = 0; gr < a.ng && ok; ++gr) {
          const int acc = a.gkey[gr] ^ a.skey[i];
          ok = acc >= 0 && acc < a.keys;
          for (int row = 0; row < 16; ++row)
            for (int k = 0; k < 4; ++k)
              D[((size_t)v * a.keys + acc) * 16 + row] +=
                  (double)tab.coef[((size_t)((v * a.tw + i) * nq + gr / 4) * 64 + k * 16 + row) * 4 + gr % 4] *
                  rowG[(size_t)(16 * (gr / 4) + 4 * k + gr % 4) * nk + q];
        }
      }
    for (int k = 0; k < nk; ++k) ok = ok && seen[k] == 1;
    double err = 0.0, top = 0.0;
    for (int o = 0; o < nk && ok; ++o) {
      const int kk = tab.index[nk + a.nw * a.tw + o], key = kk / 16, idx = kk % 16;
      ok = kk >= 0 && key < a.keys && a.rows[key][idx] == o;
      double got = 0.0, want = 0.0;
      for (int v = 0; v < a.nw; ++v) got += D[((size_t)v * a.keys + (key ^ a.wkey[v])) * 16 + idx];
      for (int be = 0; be < nk; ++be)
        for (int q = 0; q < nk; ++q) want += K[((size_t)o * nk + q) * nk + be] * G[(size_t)be * nk + q];
      err = std::max(err, std::fabs(got - want));
      top = std::max(top, std::fabs(want));
    }
    // the table rounds K to float: 2^-24 a term
    ok = ok && top > 0.0 && err <= 1e-6 * top && fdiff <= 1e-12;
    std::printf("L=%d: %s (err %.2e of %.2e, %d slots, %d groups, composed %.1e)\n", L, ok ? "ok" : "FAIL", err, top,
                a.tw, a.ng, fdiff);
    all = all && ok;
  }
  return all ? 0 : 1;
}
