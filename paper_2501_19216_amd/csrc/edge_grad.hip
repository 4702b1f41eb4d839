// The per-edge products of the backward: the gradients of the attention
// weights and of the positions.  The message of edge e = (i, j) is linear in
// the harmonics of r_i - r_j, so with the receiver's output gradient gy_i
//   X_h[e][be] = sum_{q, c of head h} Z_i[q][c][be] h_j[q][c],
//   Z_i[q][c][be] = sum_o gy_i[o][c] K[o][be][q],
//   galpha[e][h] = sum_be R_be(r_e) X_h[e][be],
//   gedge[e][x]  = sum_be dR_be/dx(r_e) sum_h alpha_eh X_h[e][be].
#include <hip/hip_runtime.h>

#include <algorithm>

#include "agg_layout.h"
#include "e2f_launch.h"
#include "split_bf16.h"

namespace e2f {
namespace {

// Four floats as bfloat16 pairs (split_bf16.h).
struct Parts {
  unsigned h0, h1, m0, m1, l0, l1;
};
__device__ __forceinline__ Parts split4(float x, float y, float z, float w) {
  Parts p;
  split_pair(x, y, p.h0, p.m0, p.l0);
  split_pair(z, w, p.h1, p.m1, p.l1);
  return p;
}

// Gradient of one solid harmonic from its monomials: d/dx of c x^a y^b z^e
// is c a x^(a-1) y^b z^e (no term when a = 0).
template <typename F>
__device__ __forceinline__ void sh_poly_grad(const DevTables& t, int k, F x, F y, F z, F& gx, F& gy, F& gz) {
  // per monomial one power loop per coordinate: b^(n-1) (1 for n = 0, where
  // the derivative's factor n is 0), then b^n = b^(n-1) b selected without a
  // branch
  auto pm1 = [](F b, int n) {
    F r = 1;
    for (int q = 1; q < n; ++q) r *= b;
    return r;
  };
  gx = 0, gy = 0, gz = 0;
  for (int e = t.sh_ptr[k]; e < t.sh_ptr[k + 1]; ++e) {
    const int pw = t.sh_pow[e];
    const int ex = pw & 15, ey = (pw >> 4) & 15, ez = (pw >> 8) & 15;
    const F c = (F)t.sh_coef[e];
    const F xm = pm1(x, ex), ym = pm1(y, ey), zm = pm1(z, ez);
    const F X = ex > 0 ? xm * x : (F)1, Y = ey > 0 ? ym * y : (F)1, Z = ez > 0 ? zm * z : (F)1;
    gx += c * (F)ex * xm * Y * Z;
    gy += c * (F)ey * X * ym * Z;
    gz += c * (F)ez * X * Y * zm;
  }
}

// Sum over the 16 lanes of a lane group (rotations within a row of 16 lanes).
__device__ __forceinline__ float sum16(float v) {
#define E2F_ROR(n) \
  __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x120 | n, 0xf, 0xf, true))
  v += E2F_ROR(8);
  v += E2F_ROR(4);
  v += E2F_ROR(2);
  v += E2F_ROR(1);
#undef E2F_ROR
  return v;
}

// Row tiles of 16 edges a wave holds at a time where rows average more than 32
// edges, more than 24 (medium) or fewer: X takes 4 registers per tile and key, the
// features of two steps eight per tile.  A tile past the chunk's end is loaded all
// the same (one line), so more is not better; fewer take a long row in more
// chunks, each of which couples the receiver's gradient again.
// Attention gradient, 20,000 atoms, 8 heads, C = 64, rows of half to one and a
// half times the average (where no number of tiles fits every row), with 2, 3, 4,
// 5 and 6 tiles: 28 edges on average L = 2 460, 399, 443, 488, 570 us; L = 3 901,
// 639, 603, 682, 707; L = 4 1.66, 1.20, 1.36, 1.38, 1.43 ms; 60, L = 2 742, 728,
// 806, 814, 833 us; L = 3 1.26, 1.12, 1.18, 1.28, 1.13 ms; L = 4 2.66, 2.27, 2.48,
// 2.28, 1.98; 120, L = 3 4.09, 3.82, 3.26, 2.45, 2.58; L = 4 5.87, 6.52, 4.56, 4.96,
// 5.26; one head of 16, 36, L = 5 980, 826, 736 us (2, 3, 4).  20 on average: two
// tiles take 0.90 of the time of three at L = 2, 0.92 at L = 3, 0.98 at L = 4.
constexpr int grad_tiles(int L, int W, bool medium) {
  return L <= 2 ? 3 : L <= 4 ? (medium ? 3 : 6) : L == 5 || W == 1 ? 4 : 3;
}
// Waves a workgroup, which share the coupling table in LDS: 45 KB at L = 4, 108
// and 159 KB at L = 5, 6, where one workgroup has the CU to itself; it has four
// waves there too where eight would leave half of the CUs without one.  (Read
// from L2 at L = 5, 6, each read of the table waited for the features' loads
// before it, which return in order: 20,000 atoms, 80 neighbours,
// L = 5, 8 heads, C = 64 16.1 -> 7.2 ms, C = 32 19.2 -> 6.2.)
constexpr int kGradWaves = 4;
// Where X += h Z^T runs as split bf16 products: a lane's four slots fill the K
// of three v_mfma_f32_16x16x32_bf16 (16 cycles each) a tile and key with the six
// cross products that reach 2^-24 of the product, against four
// v_mfma_f32_16x16x4f32 (32 cycles each); the features' split is shared by the
// keys, that of Z by the tiles.  Below L = 4 one key does not pay for the
// split.  Feature and weight gradients (one component a step, P = 1): 2,000
// atoms, L = 4 1.02 -> 0.87 ms, 9,001 atoms, L = 5 3.79 -> 3.02, 2,000 atoms, L =
// 6 1.58 -> 1.34.  At L = 5, 6 with narrow heads (P = 2, 4) the coupling is the
// larger part and the registers of the split slow it: 2,500 atoms, L = 5, P = 2
// 1.12 float, 1.24 split; L = 6, P = 2 2.38 and 2.43, P = 4 4.41 and 4.44.  At L = 4
// P = 2 0.74 -> 0.67, P = 4 0.90 -> 0.89.
constexpr bool grad_split(int L, int P) { return L == 4 || (L > 4 && P == 1); }

// A wave takes one head of one receiver at a time.  Both products run on
// v_mfma_f32_16x16x4f32 (the second split where grad_split says so) and the
// first feeds the second from its accumulators: for a component q
//   Z^T[(p, c)][be] = sum_o gy^T[(p, c)][o] K_q[o][be]
// comes out with column be = l16 and rows 4 k4 + v, which is the B operand of
// step v of X[e][be] += sum_{(p, c)} h[e][(p, c)] Z^T[(p, c)][be] when step v
// takes the slots 4 k4 + v; its A operand is then component v of one float4 of
// the sender's features.  The 16 slots (p, c) are P components q (of one key)
// of DH = 16 / P channels.  Columns be are the components of one key at a time
// (agg_layout.h): the outputs o of key x reach, through q of key y, be of key
// x ^ y alone, four of them a step.  K_q[o][be] comes from a table (element
// ((q NG + g) 64 + lane): o = member k4 of group g, be = member l16 of key
// gkey[g] ^ key(q)), in LDS where it fits (LT).
//
// As in the fused aggregation an XCD takes a contiguous range of items (a set
// of receivers and a head, the heads of one 128-byte line first), so that the
// lines its waves gather stay in its L2; gedge is therefore written per head
// ([H][edges][3]) and summed over the heads by k_edge_sum.
// T: grad_tiles, or 2 for graphs of short rows (more waves share a SIMD).
// W: groups of DH channels taken together, the same component of both in turn:
// 2 for heads of 32 channels and more, whose 128-byte lines hold two groups (a
// pass per group fetched each line twice: attention gradient at 20,000 atoms,
// 80 neighbours, L = 3, four heads of 32, 3.65 -> 2.04 ms).
//
// A launch covers the edges lo .. hi - 1 (a row that crosses the range gives
// its part: every edge's products are its own).  Re, Gt and gedge hold these
// edges only, galpha every edge.  range: the receivers with an edge of the
// range (first, end), over which the workgroups are dealt out anew; NULL: all
// n.  (Workgroups dealt out over all n, those without an edge leaving at once:
// the edges of a pass then fall to a few XCDs only, 512,000 edges in four
// passes 4.1 ms against 1.3 in one.)
template <int L, int P, int W, int NWV, int T>
__global__ __launch_bounds__(64 * NWV) __attribute__((amdgpu_waves_per_eu(T > 3 ? 2 : L <= 3 ? 4 : L == 4 ? 3 : 2)))
void k_edge_grad(const float* __restrict__ Re, const float* __restrict__ Gt, const float* __restrict__ feat,
                 const float* __restrict__ gy, const int64_t* __restrict__ row_ptr, const int32_t* __restrict__ col,
                 const float* __restrict__ alpha, int n, int rpw, int nset, int lg, int per_xcd, int C, int H,
                 int64_t lo, int64_t hi, const int* __restrict__ range, const float* __restrict__ coef,
                 float* __restrict__ galpha, float* __restrict__ gedge) {
  constexpr AggMap M = agg_map(L);
  constexpr int NK = M.nk, NG = M.ng, KEYS = M.keys, DH = 16 / P;
  constexpr bool LT = L >= 2;  // (a table of up to 1 KB stays in L1)
  extern __shared__ float sm[];
  const float* tab = LT ? sm : coef;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int l16 = lane & 15, k4 = lane >> 4;
  int first = 0, nrec = n;
  if (range) {  // (fewer sets than launch_edge_grad has for all n, of the same size)
    first = range[0], nrec = range[1] - first;
    nset = (nrec + NWV * rpw - 1) / (NWV * rpw);
    per_xcd = (int)(((int64_t)nset * H + 7) / 8);
    if ((int)(blockIdx.x / 8) >= per_xcd) return;
  }
  const int item = (blockIdx.x % 8) * per_xcd + blockIdx.x / 8;
  const int h = item / (nset * lg) * lg + item % lg, set = item / lg % nset;
  if (h >= H) return;
  if constexpr (LT) {
    constexpr int NV = NK * NG * 16, NT = 64 * NWV, IT = (NV + NT - 1) / NT, B = IT < 20 ? IT : 20;
#pragma unroll 1
    for (int e0 = threadIdx.x; e0 < NV; e0 += B * NT) {
      float4 v[B];  // every load in flight before the first store
#pragma unroll
      for (int x = 0; x < B; ++x) v[x] = ((const float4*)coef)[min(e0 + x * NT, NV - 1)];
#pragma unroll
      for (int x = 0; x < B; ++x)
        if (e0 + x * NT < NV) ((float4*)sm)[e0 + x * NT] = v[x];
    }
    __syncthreads();
  }
  // the lane's component o of every group, its column be of every key (-1: none)
  int go[NG], cb[KEYS];
#pragma unroll
  for (int g = 0; g < NG; ++g) {
    int o = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) o = k4 == k && M.gbe[g][k] > 0 ? M.gbe[g][k] : o;
    go[g] = o;  // (a missing one: component 0, its table entries are zero)
  }
#pragma unroll
  for (int x = 0; x < KEYS; ++x) {
    cb[x] = -1;
#pragma unroll
    for (int k = 0; k < 16; ++k) cb[x] = l16 == k ? M.rows[x][k] : cb[x];
  }
  const int dh = C / H, uph = dh / DH;
  const int pl = 4 * k4 / DH, cl = 4 * k4 % DH;  // the lane's slots 4 k4 .. + 3: component pl, channels cl ..
  // bounds of a receiver (clamped to the range; hi < 2^31), loaded while the
  // one before is worked on
  auto receiver = [&](int k, int& i, int64_t& b0, int64_t& b1) {
    i = first + min((set * rpw + min(k, rpw - 1)) * NWV + wave, nrec - 1);
    b0 = row_ptr[i], b1 = row_ptr[i + 1];
  };
  int in;
  int64_t b0, b1;
  receiver(0, in, b0, b1);
  for (int k = 0; k < rpw; ++k) {
    if ((set * rpw + k) * NWV + wave >= nrec) return;
    const int i = __builtin_amdgcn_readfirstlane(in);
    const int e0 = __builtin_amdgcn_readfirstlane((int)max(lo, min(b0, hi)));
    const int e1 = __builtin_amdgcn_readfirstlane((int)max((int64_t)e0, min(b1, hi)));
    receiver(k + 1, in, b0, b1);
    const float* gyi = gy + (size_t)i * NK * C;
    const int all = (e1 - e0 + 15) / 16;
    const int chunks = (all + T - 1) / T, per = chunks ? (all + chunks - 1) / chunks : 0;
    for (int ch = 0; ch < chunks; ++ch) {
      const int64_t c0 = e0 + ch * per * 16;
      const int nt = min(per, all - ch * per);
      const int cnt = min((int)(e1 - c0), 16 * nt);  // edges of the chunk
      const float* fj[T];
#pragma unroll
      for (int u = 0; u < T; ++u) {
        const int j = (col + c0)[(unsigned)min(16 * u + l16, cnt - 1)];
        fj[u] = feat + (size_t)((unsigned)j < (unsigned)n ? j : 0) * NK * C + cl;
      }
      v4f X[T][KEYS];
#pragma unroll
      for (int u = 0; u < T; ++u)
#pragma unroll
        for (int x = 0; x < KEYS; ++x) X[u][x] = (v4f){0.f, 0.f, 0.f, 0.f};
      for (int un = 0; un < uph; un += W) {
        const bool pair = W == 2 && un + 1 < uph;
        int hc[W];
        float ga[W][NG];
#pragma unroll
        for (int w = 0; w < W; ++w) {
          hc[w] = h * dh + (un + (pair ? w : 0)) * DH;
#pragma unroll
          for (int g = 0; g < NG; ++g) ga[w][g] = gyi[(size_t)go[g] * C + hc[w] + l16 % DH];
        }
        // (waited for here: loads return in order, and a wait inside the loop
        // would be one for the features of its next step)
#pragma unroll
        for (int w = 0; w < W; ++w)
#pragma unroll
          for (int g = 0; g < NG; ++g) asm volatile("" : "+v"(ga[w][g]));
#pragma unroll
        for (int y = 0; y < KEYS; ++y) {
          // members of key y, P at a time
          int ny = 0;
#pragma unroll
          for (int z = 0; z < 16; ++z) ny += M.rows[y][z] >= 0 ? 1 : 0;
          const int steps = (ny + P - 1) / P;
          auto member = [&](int z) {  // component z of key y (uniform or per lane)
            if constexpr (KEYS == 1 && W == 2) return z;  // (without it the wide form spills scalars at L = 3)
            int q = M.rows[y][0];
#pragma unroll
            for (int m = 1; m < 16; ++m)
              if (M.rows[y][m] >= 0) q = z == m ? M.rows[y][m] : q;
            return q;
          };
          // unconditional loads (a tile past nt repeats the chunk's last sender, one line),
          // two register sets in turn: the waits then count exactly
          float4 fa[T], fb[T];
          auto load = [&](int s, int w, float4* d) {
            const int q = member(min(s * P + pl, ny - 1));
            const unsigned off = (unsigned)(q * C + hc[w]);
#pragma unroll
            for (int u = 0; u < T; ++u) d[u] = *(const float4*)(fj[u] + off);
          };
          auto step = [&](int s, int w, const float4* f) {
            v4f z[KEYS];
#pragma unroll
            for (int x = 0; x < KEYS; ++x) z[x] = (v4f){0.f, 0.f, 0.f, 0.f};
#pragma unroll(P == 4 && L >= 5 ? 1 : P)
            for (int p = 0; p < P; ++p) {
              if (s * P + p >= ny) break;
              const float* kq = tab + (size_t)member(s * P + p) * NG * 64 + lane;
#pragma unroll
              for (int g = 0; g < NG; ++g) {
                const float a = P == 1 || l16 / DH == p ? ga[w][g] : 0.0f;
                z[M.gkey[g]] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, kq[g * 64], z[M.gkey[g]], 0, 0, 0);
              }
            }
            // (z[x] holds the columns of key x ^ y)
            if constexpr (grad_split(L, P)) {
              v4u hm[KEYS], mh[KEYS], hl[KEYS];  // the parts of z: {hi, mid}, {mid, hi}, {hi, lo}
#pragma unroll
              for (int x = 0; x < KEYS; ++x) {
                const Parts b = split4(z[x][0], z[x][1], z[x][2], z[x][3]);
                hm[x] = (v4u){b.h0, b.h1, b.m0, b.m1};
                mh[x] = (v4u){b.m0, b.m1, b.h0, b.h1};
                hl[x] = (v4u){b.h0, b.h1, b.l0, b.l1};
              }
#pragma unroll
              for (int u = 0; u < T; ++u)
                if (u < nt) {
                  const Parts a = split4(f[u].x, f[u].y, f[u].z, f[u].w);
                  const v4u lh = {a.l0, a.l1, a.h0, a.h1}, ha = {a.h0, a.h1, a.m0, a.m1};
#pragma unroll
                  for (int x = 0; x < KEYS; ++x) X[u][x ^ y] = mfma_bf16(lh, hl[x], X[u][x ^ y]);
#pragma unroll
                  for (int x = 0; x < KEYS; ++x) X[u][x ^ y] = mfma_bf16(ha, mh[x], X[u][x ^ y]);
#pragma unroll
                  for (int x = 0; x < KEYS; ++x) X[u][x ^ y] = mfma_bf16(ha, hm[x], X[u][x ^ y]);
                }
            } else {
#pragma unroll
              for (int u = 0; u < T; ++u)
                if (u < nt) {
#pragma unroll
                  for (int v = 0; v < 4; ++v)
#pragma unroll
                    for (int x = 0; x < KEYS; ++x)
                      X[u][x ^ y] =
                          __builtin_amdgcn_mfma_f32_16x16x4f32((&f[u].x)[v], z[x][v], X[u][x ^ y], 0, 0, 0);
                }
            }
          };
          load(0, 0, fa);
          const int odd = pair ? 0 : 1;  // fb: the other group's, or the next component
#pragma unroll 1
          for (int s = 0; s < steps; s += 1 + odd) {
            load(s + odd, W - 1, fb);  // (past the end: the last component again)
            step(s, 0, fa);
            load(s + 1 + odd, 0, fa);
            if (s + odd < steps) step(s + odd, W - 1, fb);
          }
        }
      }
      // lane (l16, k4) holds X of the columns be = cb[x], edges 16 u + 4 k4 + v:
      // the sums over be for galpha (with R) and gedge (with its gradients)
      const float* Rc = Re + (c0 - lo) * NK;
      const float* Gc = Gt + (c0 - lo) * 3 * NK;
      const float* ac = alpha + c0 * H + h;
      float* gc = gedge + (h * (hi - lo) + c0 - lo) * 3;
      // (a pass over the tiles per output: its loads are in flight together)
      auto edge = [&](int u, int v) { return (unsigned)min(16 * u + 4 * k4 + v, cnt - 1); };
      if (galpha) {
        float r[T][4][KEYS];
#pragma unroll
        for (int u = 0; u < T; ++u)
#pragma unroll
          for (int v = 0; v < 4; ++v)
#pragma unroll
            for (int x = 0; x < KEYS; ++x) r[u][v][x] = L == 0 ? 1.0f : Rc[edge(u, v) * NK + max(cb[x], 0)];
#pragma unroll
        for (int u = 0; u < T; ++u) {
          float p[4];
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            p[v] = 0.0f;
#pragma unroll
            for (int x = 0; x < KEYS; ++x) p[v] += cb[x] >= 0 ? r[u][v][x] * X[u][x][v] : 0.0f;
            p[v] = sum16(p[v]);
          }
          const int e = 16 * u + 4 * k4 + l16;
          const float a = l16 == 0 ? p[0] : l16 == 1 ? p[1] : l16 == 2 ? p[2] : p[3];
          if (l16 < 4 && e < cnt && u < nt) galpha[(c0 + e) * H + h] = a;
        }
      }
      if (gedge) {
        if (alpha) {
#pragma unroll
          for (int u = 0; u < T; ++u)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
              const float w = ac[edge(u, v) * H];
#pragma unroll
              for (int x = 0; x < KEYS; ++x) X[u][x][v] *= w;
            }
        }
#pragma unroll
        for (int d = 0; d < 3; ++d) {
          float g[T][4][KEYS];
#pragma unroll
          for (int u = 0; u < T; ++u)
#pragma unroll
            for (int v = 0; v < 4; ++v)
#pragma unroll
              for (int x = 0; x < KEYS; ++x) g[u][v][x] = Gc[(edge(u, v) * 3 + d) * NK + max(cb[x], 0)];
#pragma unroll
          for (int u = 0; u < T; ++u) {
            float p[4];
#pragma unroll
            for (int v = 0; v < 4; ++v) {
              p[v] = 0.0f;
#pragma unroll
              for (int x = 0; x < KEYS; ++x) p[v] += cb[x] >= 0 ? g[u][v][x] * X[u][x][v] : 0.0f;
              p[v] = sum16(p[v]);
            }
            const int e = 16 * u + 4 * k4 + l16;
            const float a = l16 == 0 ? p[0] : l16 == 1 ? p[1] : l16 == 2 ? p[2] : p[3];
            if (l16 < 4 && e < cnt && u < nt) gc[(unsigned)(3 * e + d)] = a;
          }
        }
      }
    }
  }
}

// The receivers of each pass of `pass` edges: the first that has one of its
// edges, and one past the last (the last row that starts at or before an edge
// holds it).
__global__ __launch_bounds__(256) void k_edge_ranges(const int64_t* __restrict__ row_ptr, int n, int64_t n_edges,
                                                     int64_t pass, int passes, int* __restrict__ range) {
  const int p = (blockIdx.x * 256 + threadIdx.x) / 2, last = threadIdx.x & 1;
  if (p >= passes) return;
  const int64_t e = last ? min((p + 1) * pass, n_edges) - 1 : p * pass;
  int i = 0;
  for (int hi = n; hi - i > 1;) {
    const int mid = i + (hi - i) / 2;
    if (row_ptr[mid] <= e) i = mid;
    else hi = mid;
  }
  range[2 * p + last] = i + last;
}

// gedge = the sum of the heads' parts, in order.
__global__ __launch_bounds__(256) void k_edge_sum(const float* __restrict__ part, int H, int64_t count,
                                                  float* __restrict__ gedge) {
  const int64_t q = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (q >= count) return;
  float s = 0.0f;
  for (int h = 0; h < H; ++h) s += part[h * count + q];
  gedge[q] = s;
}

// Gradients of the harmonics of every edge, Gt [E][3][NK]: 64 edges a
// workgroup, rows through LDS (odd stride) so that they leave contiguously.
__global__ __launch_bounds__(256) void k_edge_shgrad(DevTables t, const float* __restrict__ pos,
                                                     const int32_t* __restrict__ rows,
                                                     const int32_t* __restrict__ col, int n, int64_t n_edges,
                                                     float* __restrict__ Gt) {
  extern __shared__ float sm[];
  const int nk = t.nk, ld = 3 * nk | 1, lane = threadIdx.x & 63;
  const int64_t e0 = (int64_t)blockIdx.x * 64, e = e0 + lane;
  const int cnt = (int)min((int64_t)64, n_edges - e0);
  if (lane < cnt) {
    const int i = rows[e], j = col[e], jc = (unsigned)j < (unsigned)n ? j : 0;
    const float x = pos[3 * i] - pos[3 * jc], y = pos[3 * i + 1] - pos[3 * jc + 1], z = pos[3 * i + 2] - pos[3 * jc + 2];
    for (int be = threadIdx.x >> 6; be < nk; be += 4) {
      float g[3];
      sh_poly_grad<float>(t, be, x, y, z, g[0], g[1], g[2]);
      for (int d = 0; d < 3; ++d) sm[lane * ld + d * nk + be] = g[d];
    }
  }
  __syncthreads();
  for (int q = threadIdx.x; q < cnt * 3 * nk; q += 256) Gt[e0 * 3 * nk + q] = sm[q / (3 * nk) * ld + q % (3 * nk)];
}

// Per atom: the forces of the edges it receives minus those it sends (through
// the transposed graph).  A wave per atom, its lanes over the edges, summed in
// a fixed order.
__global__ __launch_bounds__(256) void k_force_gather(const int64_t* __restrict__ row_ptr,
                                                      const int64_t* __restrict__ rowT,
                                                      const int32_t* __restrict__ perm,
                                                      const float* __restrict__ gedge, int n,
                                                      float* __restrict__ gpos) {
  const int a = blockIdx.x * 4 + (int)(threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (a >= n) return;  // uniform over the wave
  float s[3] = {0.f, 0.f, 0.f};
  for (int64_t e = row_ptr[a] + lane; e < row_ptr[a + 1]; e += 64)
    for (int x = 0; x < 3; ++x) s[x] += gedge[e * 3 + x];
  for (int64_t q = rowT[a] + lane; q < rowT[a + 1]; q += 64)
    for (int x = 0; x < 3; ++x) s[x] -= gedge[(int64_t)perm[q] * 3 + x];
  for (int o = 32; o > 0; o >>= 1)
    for (int x = 0; x < 3; ++x) s[x] += __shfl_xor(s[x], o);
  if (lane < 3) gpos[(int64_t)a * 3 + lane] = lane == 0 ? s[0] : lane == 1 ? s[1] : s[2];
}

}  // namespace

hipError_t launch_edge_grad(int L, const float* Re, const float* Gt, const float* feat, const float* gy,
                            const int64_t* row_ptr, const int32_t* col, const float* alpha, int n, int C, int H,
                            int64_t n_edges, int64_t lo, int64_t hi, const int* range, const float* coef,
                            float* galpha, float* gpart, float* gedge, hipStream_t s) {
  if (n == 0 || hi <= lo || (!galpha && !gedge)) return hipSuccess;
  const int dh = C / H, P = dh % 16 == 0 ? 1 : dh % 8 == 0 ? 2 : 4;  // the widest group that divides a head
  int lg = std::max(1, std::min(32 / dh, H));  // heads of one 128-byte line
  while (H % lg) --lg;
  float* out = gedge && H > 1 ? gpart : gedge;
  const int64_t n_waves = (int64_t)n * H;
  // Receivers a wave takes one after another (they share the table): up to eight,
  // as long as every CU has work.  One where rows are long (up to L = 4): the heads
  // of a line run as workgroups side by side and share it only as long as they
  // keep in step, which they lose over several receivers.  20,000 atoms, 8 heads,
  // C = 64, one and up to eight: 200 neighbours, L = 3 0.54 of the time, L = 4 0.53; 80, L = 2
  // 0.85, L = 3 0.59, L = 4 0.55; 60, all L, heads of 4 to 32 channels 0.9 (the
  // worst, L = 2, C = 32, 1.07); 40, L = 2 0.97, L = 3 1.06, L = 4 1.04; 12, L = 1
  // 1.11, L = 3 1.09.  At L = 5, where the table takes longer to load, 80 1.02.
  const int64_t most = L <= 4 && n_edges > (int64_t)n * 56 ? 1 : 8;
  const bool few = n_edges <= (int64_t)n * 24, medium = n_edges <= (int64_t)n * 32;
  // waves that have a SIMD to themselves wait for their own chunks (up to L = 2,
  // where the others take three tiles: 600 atoms, one head of 12, L = 2, 60
  // neighbours, three tiles 1.14 of the time of six)
  const bool alone = n_waves <= 1024;
#define E2F_G(LL, PP, WW, NN, TT)                                                                                 \
  do {                                                                                                            \
    constexpr AggMap M = agg_map(LL);                                                                             \
    constexpr int nw = NN;                                                                                        \
    const int rpw = (int)std::max<int64_t>(1, std::min(most, n_waves / (256 * 16)));                              \
    const int nset = (n + nw * rpw - 1) / (nw * rpw);                                                             \
    const int64_t per = ((int64_t)nset * H + 7) / 8;                                                              \
    if (per * 8 > 0x7fffffff) return hipErrorInvalidValue;                                                        \
    k_edge_grad<LL, PP, WW, nw, TT><<<(unsigned)(8 * per), 64 * nw, LL >= 2 ? M.nk * M.ng * 256 : 0, s>>>(        \
        Re, Gt, feat, gy, row_ptr, col, alpha, n, rpw, nset, lg, (int)per, C, H, lo, hi, range, coef,      \
        galpha, out);                                                                                             \
  } while (0)
#define E2F_GT(LL, PP, WW, NN)                                                             \
  do {                                                                                     \
    constexpr int tm = grad_tiles(LL, WW, true), tl = grad_tiles(LL, WW, false);           \
    if (few) E2F_G(LL, PP, WW, NN, 2);                                                     \
    else if (LL <= 2 && alone) E2F_G(LL, PP, WW, NN, (LL <= 2 ? 6 : tm));                  \
    else if (medium) E2F_G(LL, PP, WW, NN, tm);                                            \
    else E2F_G(LL, PP, WW, NN, tl);                                                        \
  } while (0)
#define E2F_GN(LL, PP, WW)                                     \
  do {                                                         \
    if (LL <= 4 || n_waves <= 1024) E2F_GT(LL, PP, WW, kGradWaves);           \
    else E2F_GT(LL, PP, WW, (LL <= 4 ? kGradWaves : 2 * kGradWaves));         \
  } while (0)
#define E2F_GL(LL)                                             \
  case LL:                                                     \
    if (P == 1 && dh >= 32) E2F_GN(LL, 1, 2);                  \
    else if (P == 1) E2F_GN(LL, 1, 1);                         \
    else if (P == 2) E2F_GN(LL, 2, 1);                         \
    else E2F_GN(LL, 4, 1);                                     \
    break;
  switch (L) {
    E2F_GL(0) E2F_GL(1) E2F_GL(2) E2F_GL(3) E2F_GL(4) E2F_GL(5) E2F_GL(6)
    default: return hipErrorInvalidValue;
  }
#undef E2F_GL
#undef E2F_GN
#undef E2F_GT
#undef E2F_G
  if (hipError_t e = hipGetLastError(); e != hipSuccess || out == gedge) return e;
  const int64_t blocks = ((hi - lo) * 3 + 255) / 256;
  if (blocks > 0x7fffffff) return hipErrorInvalidValue;
  k_edge_sum<<<(unsigned)blocks, 256, 0, s>>>(gpart, H, (hi - lo) * 3, gedge);
  return hipGetLastError();
}

hipError_t launch_edge_ranges(const int64_t* row_ptr, int n, int64_t n_edges, int64_t pass, int passes, int* range,
                              hipStream_t s) {
  if (n == 0 || passes <= 0) return hipSuccess;
  k_edge_ranges<<<(unsigned)((2 * (int64_t)passes + 255) / 256), 256, 0, s>>>(row_ptr, n, n_edges, pass, passes, range);
  return hipGetLastError();
}

hipError_t launch_edge_shgrad(const DevTables& t, const float* pos, const int32_t* rows, const int32_t* col, int n,
                              int64_t n_edges, float* Gt, hipStream_t s) {
  if (n_edges == 0) return hipSuccess;
  const int64_t blocks = (n_edges + 63) / 64;
  if (blocks > 0x7fffffff) return hipErrorInvalidValue;
  k_edge_shgrad<<<(unsigned)blocks, 256, sizeof(float) * 64 * (3 * t.nk | 1), s>>>(t, pos, rows, col, n, n_edges, Gt);
  return hipGetLastError();
}

hipError_t launch_force_gather(const int64_t* row_ptr, const int64_t* rowT, const int32_t* perm, const float* gedge,
                               int n, float* gpos, hipStream_t s) {
  if (n == 0) return hipSuccess;
  k_force_gather<<<(unsigned)((n + 3) / 4), 256, 0, s>>>(row_ptr, rowT, perm, gedge, n, gpos);
  return hipGetLastError();
}

}  // namespace e2f
