// Internal declarations shared by the host code (tables, C ABI) and the HIP
// kernels of libe2f.  Nothing here is part of the public ABI (include/e2f.h).
#pragma once

#include <cstddef>
#include <cstdint>
#include <string>
#include <vector>

namespace e2f {

constexpr int kMaxL = 6;          // largest supported degree L
constexpr double kGrid = 65536.0; // positions are compared on a 2^-16 A grid

inline int nk_of(int L) { return (L + 1) * (L + 1); }

// ---------------------------------------------------------------- host tables
// Real-basis Clebsch-Gordan tensor C[m1][m2][m3] for (l1,l2,l3), row-major,
// built from the explicit CG formula and the real change of basis (tables.cpp).
std::vector<double> real_cg(int l1, int l2, int l3);
// Recoupling weight X(a,b,u,o;d) of [A (x) [C (x) B]^(b+u)]^(o) onto
// [C (x) [A (x) B]^(d)]^(o) (Def. 2.3), closed form from the Wigner 6j symbol.
double recoupling_weight(int a, int b, int u, int o, int d);
double wigner6j(int j1, int j2, int j3, int j4, int j5, int j6);

// Structure of the factorised layer for one L: every table is independent of
// the path weights except the *_coef arrays, which the context refreshes when
// the caller's path weights change.
// Thread count of the schedules that build per-node matrices in LDS.
constexpr int kSchedThreads = 256;
// Rows of T per chunk of the recouple's per-node matrix: 192 at L <= 4 (a
// 37 KB tile, four workgroups per CU: 1.18 vs 1.20 ms with 256 rows and three),
// 128 at L = 5, 120 at L = 6 (a 38.4 KB tile: four workgroups per CU instead
// of three with 128 rows, 46.9 vs 49.7 ms at 200k atoms).
constexpr int rc_rows(int nk) { return nk > 36 ? 120 : (nk > 25 ? 128 : 192); }
// Row stride (floats) of the recouple's per-node matrix tile in LDS: the
// 16*ceil(nk/16) used columns padded to 16 mod 32, so the MFMA operand reads
// of 4 rows x 16 columns fall in distinct banks.
constexpr int rc_qstride(int nk) {
  return 16 * ((nk + 15) / 16) + (((nk + 15) / 16) % 2 == 0 ? 16 : 0);
}

// A per-node matrix built by 256 threads from a fixed schedule: in chunk c,
// thread t walks entries k = 0..k[c]-1 at index off[c] + k*256 + t, each
// adding coef * R[ridx] and, on the last entry of a slot, storing the sum to
// LDS position dest.  meta packs dest (bits 0-19), ridx (20-26), last (31).
// Monomials of degree l, and the offset of degree l's block in the dense
// solid-harmonic table (rows 2l'+1 by columns sh_monos(l') for every l' < l).
constexpr int sh_monos(int l) { return (l + 1) * (l + 2) / 2; }
constexpr int sh_dense_off(int l) { return l <= 0 ? 0 : sh_dense_off(l - 1) + (2 * l - 1) * sh_monos(l - 1); }

struct Schedule {
  std::vector<int> k, off;
  std::vector<int> meta;
  std::vector<int> path;      // path-weight index of each entry (-1: none)
  std::vector<double> unit;   // coefficient without the path weight
};

struct Block {
  int a, b, d, toff;  // T_j^(a,b,d) occupies rows toff .. toff+2d
};

struct LayerTables {
  int L = 0, nk = 0, dimT = 0;
  std::vector<Block> blocks;        // sorted by (a, b, d)
  std::vector<int> a_row_start;     // [L+2] first T row of each a
  // solid harmonics as polynomials: component k = sum_t coef_t x^ex y^ey z^ez
  std::vector<int> sh_ptr;          // [nk+1]
  std::vector<int> sh_pow;          // packed ex | ey<<4 | ez<<8
  std::vector<double> sh_coef;
  // the same polynomials dense per degree l: rows m < 2l+1, columns the
  // monomials x^ex y^ey z^(l-ex-ey) in (ex, ey) order, ex and ey ascending;
  // the block of degree l starts at sh_dense_off(l)
  std::vector<double> sh_dense;
  // j-side per-node matrix M: row r of T has (2a+1) slots starting at m_rowoff[r]
  std::vector<int> m_rowoff;        // [dimT+1]
  std::vector<int> m_ptr;           // [nslots+1] entries of each slot
  std::vector<int> m_ridx;          // index into R (l*l + l + m)
  std::vector<double> m_coef;       // CG value
  // i-side per-node matrix Q_o, (2o+1) x ncol[o], for each output degree o
  std::vector<int> q_ncol;          // [L+1]
  std::vector<int> q_coloff;        // [L+2] offset of o's column list in q_cols
  std::vector<int> q_cols;          // T row index of each column
  std::vector<int> q_slotoff;       // [L+2] offset of o's slots
  std::vector<int> q_ptr;           // [nslots+1]
  std::vector<int> q_ridx;
  std::vector<int> q_path;          // (a*(L+1)+f)*(L+1)+o of the path weight
  std::vector<double> q_unit;       // coefficient without the path weight
  // edge tensor product filter K[k][q] (dense nk x nk)
  std::vector<int> k_ptr;           // [nk*nk+1]
  std::vector<int> k_ridx;
  std::vector<int> k_path;
  std::vector<double> k_unit;
  // node TP: one chunk; the matrix of degree a is stored transposed at
  // tp_mo[a], entry (al, row) at al*tp_rs[a] + row - a_row_start[a], with
  // 2a+1 rows of tp_rs[a] floats (tp_rs = 16 mod 32)
  Schedule tp_sched;
  std::vector<int> tp_rs, tp_mo;    // [L+1], [L+2]
  Schedule rc_sched;                // recouple: chunks of rc_rows T rows, dest = row*rc_qstride + (o*o+m)
  // recouple restricted to the terms of filter degree f = b + u, one schedule
  // per f (attention weights alpha / D^f need one aggregation per f)
  std::vector<Schedule> rcf_sched;  // [L+1]
  // j-side coupling of aggregated uncoupled products: S[row] = sum over the
  // row's entries of coef * G[be][q], entries ag_ptr[row] .. ag_ptr[row+1]
  // with ag_idx = be << 6 | q (be, q < (L+1)^2)
  std::vector<int> ag_ptr, ag_idx;
  std::vector<float> ag_coef;
  int max_qslots = 0;               // largest (2o+1)*ncol[o]
  int m_slots() const { return m_rowoff.back(); }
};

LayerTables build_layer_tables(int L);

// The coupling after aggregation as a thread-balanced schedule for `groups`
// groups of threads (one thread per channel in a group): entry k of group g
// at k*groups + g; meta = gidx (bits 0-11, be << 6 | q) | row << 12 | last
// (bit 31); rows are spread over the groups by entry count.
struct CoupleSchedule {
  int groups = 0, k = 0;
  std::vector<int> meta;
  std::vector<float> coef;
  // the same entries packed for LDS when dimT <= 512 and the coefficients take
  // at most 1024 distinct values (L <= 4): pmeta = gidx | row << 12 (9 bits) |
  // coefficient index << 21 (10 bits) | last (bit 31), tab = the coefficients
  // (empty otherwise)
  std::vector<int> pmeta;
  std::vector<float> tab;
};
CoupleSchedule couple_schedule(const LayerTables& t, int groups);

int64_t node_tp_dim(int L);

// ---------------------------------------------------------------- device side
// Device copies of one LayerTables (pointers into one allocation).
struct DevTables {
  int L, nk, dimT;
  const int* a_row_start;
  const int* sh_ptr; const int* sh_pow; const double* sh_coef;
  const double* sh_dense;  // LayerTables::sh_dense
  const int* m_rowoff; const int* m_ptr; const int* m_ridx; const double* m_coef;
  const int* q_ncol; const int* q_coloff; const int* q_cols; const int* q_slotoff;
  const int* q_ptr; const int* q_ridx; const double* q_coef; // q_coef includes path weights
  const int* k_ptr; const int* k_ridx; const float* k_coef;  // k_coef includes path weights
  const int* tp_k; const int* tp_off; const int* tp_meta; const double* tp_coef;
  const int* rc_k; const int* rc_off; const int* rc_meta; const double* rc_coef;  // rc_coef includes path weights
  const int* ag_ptr; const int* ag_idx; const float* ag_coef;
  const float* w_f;  // path weights w[(a*(L+1) + f)*(L+1) + o] as float
  int max_qslots, m_slots;
  int tp_rs[kMaxL + 1], tp_mo[kMaxL + 2];
};

}  // namespace e2f
