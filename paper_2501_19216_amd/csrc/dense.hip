// Dense-graph aggregation (Sec. 4.1's dense graphs; Alg. 1 with its attention
// tensor alpha in R^{N x N x H}): per head h the einsum "ijh,jhds->ihds" is a
// dense product S_h = A_h T_h, with A_h [N x N] the attention weights of head
// h (zero diagonal) and T_h [N x W] the head's columns of the j-side node
// products (W = dimT * C/H).
//
// The product is bound by the matrix cores.  Every float is split into three
// bf16 parts on its way into LDS (x = hi + mid + lo exactly) and the six cross
// products that reach 2^-24 of the product are summed in float: three
// v_mfma_f32_16x16x32_bf16 (16 cycles each) per 16 k of a 16 x 16 tile, whose
// 32 K slots are two parts of a lane's four k, against four
// v_mfma_f32_16x16x4f32 (32 cycles each).  Dense forward at L = 3, C = 128,
// H = 8: 522 -> 353 us at 1,000 atoms and 7.1 -> 4.4 ms at 4,000; error against
// 64 bits 6.3e-7 -> 5.5e-7.  (A scheme with one k a lane and two of eight K
// slots idle took 64 instructions where this one takes 48, and did not pay.)
//
// Tiling: a workgroup of eight waves owns a 256 x 128 tile of S_h (4 x 2
// waves of 64 x 64, each 4 x 4 MFMA tiles of 16 x 16); K advances 16 at a
// time through double-buffered LDS, the next K slab loaded into registers
// while the current one is multiplied.  128 VGPRs and 75 KB of LDS: two
// workgroups share a CU, one's splits beside the other's products.  A is stored
// by the alpha kernel with rows padded to a multiple of 32 (zeros), so K needs
// no tail handling.  Workgroups of one XCD take a contiguous range of (head,
// row block) tiles with every column block, so A's row slabs and T's column
// slabs in flight on an XCD are shared through its L2.
#include <hip/hip_runtime.h>

#include "e2f_launch.h"
#include "split_bf16.h"

namespace e2f {
namespace {

typedef unsigned v2u __attribute__((ext_vector_type(2)));

__device__ __forceinline__ void split4(float x, float y, float z, float w, v2u& hi, v2u& mid, v2u& lo) {
  unsigned h, m, l;
  split_pair(x, y, h, m, l);
  hi.x = h, mid.x = m, lo.x = l;
  split_pair(z, w, h, m, l);
  hi.y = h, mid.y = m, lo.y = l;
}

// A[h][i][j] = alpha[i][j][h] (1 if alpha is NULL), 0 for i == j and for the
// padding columns j >= n of rows of lda floats; order[i] = i (the recouple's
// receivers).  Bound by memory: a workgroup takes kPadCols columns of a row and
// kPadHeads heads through LDS (odd stride), so that the reads of alpha and the
// writes of A are both contiguous (a thread per element of A read alpha with a
// stride of H floats; dense forward at 1,000 atoms, L = 3: 539 -> 522 us).
constexpr int kPadCols = 256, kPadHeads = 8;
__global__ __launch_bounds__(kPadCols) void k_dense_alpha_pad(const float* __restrict__ alpha, int n, int H, int lda,
                                                              int chunks, int groups, float* __restrict__ A,
                                                              int32_t* __restrict__ order) {
  __shared__ float tile[kPadCols * (kPadHeads + 1)];
  const int c = blockIdx.x % chunks, g = blockIdx.x / chunks % groups, i = blockIdx.x / chunks / groups;
  const int j0 = c * kPadCols, h0 = g * kPadHeads, hn = min(kPadHeads, H - h0), cols = min(kPadCols, n - j0);
  const int tid = threadIdx.x;
  if (blockIdx.x % (chunks * groups) == 0 && tid == 0) order[i] = i;
  if (alpha) {
    const float* src = alpha + ((int64_t)i * n + j0) * H + h0;
    float v[kPadHeads];
#pragma unroll
    for (int u = 0; u < kPadHeads; ++u) {
      const int e = tid + u * kPadCols;
      v[u] = e < cols * hn ? src[(int64_t)(e / hn) * H + e % hn] : 0.0f;
    }
#pragma unroll
    for (int u = 0; u < kPadHeads; ++u) {
      const int e = tid + u * kPadCols;
      if (e < cols * hn) tile[e / hn * (kPadHeads + 1) + e % hn] = v[u];
    }
  }
  __syncthreads();
  const int j = j0 + tid;
  if (j >= lda) return;
  for (int h = 0; h < hn; ++h)
    A[((int64_t)(h0 + h) * n + i) * lda + j] =
        j >= n || i == j ? 0.0f : alpha ? tile[tid * (kPadHeads + 1) + h] : 1.0f;
}

// S_h[i][c] = sum_k A_h[i][k] T_h[k][c] for i < n, c < W, k < lda (A is zero
// past n; T rows past n are never read with a nonzero weight, their index is
// clamped).  T_h[k][c] = T[k * ldt + h * W + c], S likewise.  WGM x WGN waves
// of 64 x 64 outputs each; K slabs of BK.
template <int WGM, int WGN>
__global__ __launch_bounds__(64 * WGM * WGN) void k_dense_gemm(const float* __restrict__ A, int lda, int n,
                                                               const float* __restrict__ T, int64_t ldt, int W,
                                                               float* __restrict__ S, int n_ib, int n_cb, int H,
                                                               int per_xcd) {
  constexpr int BM = 64 * WGM, BN = 64 * WGN, NT = 64 * WGM * WGN, BK = 16;
  // K group q of a slab is its k = 4 q .. 4 q + 3; an entry (q, row or column)
  // holds the parts of its four values, A's {lo01, lo23, hi01, hi23} and
  // {mid01, mid23}, B's {hi01, hi23, mid01, mid23} and {lo01, lo23}.  (Groups
  // start 16 banks apart, so the four entries of a row that neighbouring
  // threads store fall in different banks.)
  constexpr int AQ = BM + 4, AP = BM + 8;
  constexpr int FA = BM * 4 / NT, FB = BN * 4 / NT;  // entries per thread
  static_assert(FA * NT == BM * 4 && FB * NT == BN * 4, "tile loads must divide evenly");
  __shared__ v4u Aw[2][4 * AQ];
  __shared__ v2u Am[2][4 * AP];
  __shared__ v4u Bw[2][4 * BN];
  __shared__ v2u Bl[2][4 * BN];
  const int tile = (blockIdx.x % 8) * per_xcd + (int)(blockIdx.x / 8);
  if (tile >= H * n_ib * n_cb) return;  // uniform over the workgroup
  const int cb = tile % n_cb, ib = (tile / n_cb) % n_ib, h = tile / (n_cb * n_ib);
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int l16 = lane & 15, k4 = lane >> 4;
  const int wm = (wave / WGN) * 64, wn = (wave % WGN) * 64;
  const float* Ah = A + (int64_t)h * n * lda;
  const float* Th = T + (int64_t)h * W;
  const int nk = lda / BK;
  // entry f of a slab: A row f / 4 (clamped to n - 1), group f % 4; B column f %
  // BN (clamped to W - 1, never stored), group f / BN, its rows clamped to n - 1
  // (A is zero there)
  const float* pa[FA];
  unsigned pb[FB];
  int qb[FB];  // (uniform over a wave: BN is a multiple of 64)
#pragma unroll
  for (int u = 0; u < FA; ++u) {
    const int f = tid + u * NT;
    pa[u] = Ah + (int64_t)min(ib * BM + f / 4, n - 1) * lda + 4 * (f % 4);
  }
#pragma unroll
  for (int u = 0; u < FB; ++u) {
    const int f = tid + u * NT;
    pb[u] = (unsigned)min(cb * BN + f % BN, W - 1);
    qb[u] = __builtin_amdgcn_readfirstlane(f / BN);
  }
  float4 ra[FA];
  float rb[FB][4];
  auto load = [&](int kt) {
#pragma unroll
    for (int u = 0; u < FA; ++u) ra[u] = *(const float4*)(pa[u] + kt * BK);
#pragma unroll
    for (int u = 0; u < FB; ++u)
#pragma unroll
      for (int x = 0; x < 4; ++x) rb[u][x] = (Th + (int64_t)min(kt * BK + 4 * qb[u] + x, n - 1) * ldt)[pb[u]];
  };
  auto store = [&](int buf) {
    v2u hi, mid, lo;
#pragma unroll
    for (int u = 0; u < FA; ++u) {
      const int f = tid + u * NT;
      split4(ra[u].x, ra[u].y, ra[u].z, ra[u].w, hi, mid, lo);
      Aw[buf][(f % 4) * AQ + f / 4] = (v4u){lo.x, lo.y, hi.x, hi.y};
      Am[buf][(f % 4) * AP + f / 4] = mid;
    }
#pragma unroll
    for (int u = 0; u < FB; ++u) {
      const int f = tid + u * NT;
      split4(rb[u][0], rb[u][1], rb[u][2], rb[u][3], hi, mid, lo);
      Bw[buf][f] = (v4u){hi.x, hi.y, mid.x, mid.y};
      Bl[buf][f] = lo;
    }
  };
  v4f acc[4][4];
#pragma unroll
  for (int mt = 0; mt < 4; ++mt)
#pragma unroll
    for (int nt = 0; nt < 4; ++nt) acc[mt][nt] = (v4f){0.f, 0.f, 0.f, 0.f};
  load(0);
  store(0);
  __syncthreads();
  for (int kt = 0; kt < nk; ++kt) {
    const int buf = kt & 1;
    load(min(kt + 1, nk - 1));  // in flight while this slab is multiplied
    v4u aw[4];
    v2u am[4];
#pragma unroll
    for (int mt = 0; mt < 4; ++mt) {
      aw[mt] = Aw[buf][k4 * AQ + wm + mt * 16 + l16];
      am[mt] = Am[buf][k4 * AP + wm + mt * 16 + l16];
    }
#pragma unroll
    for (int nt = 0; nt < 4; ++nt) {
      const v4u bw = Bw[buf][k4 * BN + wn + nt * 16 + l16];
      const v2u bl = Bl[buf][k4 * BN + wn + nt * 16 + l16];
      const v4u bmh = {bw.z, bw.w, bw.x, bw.y}, bhl = {bw.x, bw.y, bl.x, bl.y};
#pragma unroll
      for (int mt = 0; mt < 4; ++mt)  // lo hi + hi lo
        acc[mt][nt] = mfma_bf16(aw[mt], bhl, acc[mt][nt]);
#pragma unroll
      for (int mt = 0; mt < 4; ++mt)  // hi mid + mid hi
        acc[mt][nt] = mfma_bf16((v4u){aw[mt].z, aw[mt].w, am[mt].x, am[mt].y}, bmh, acc[mt][nt]);
#pragma unroll
      for (int mt = 0; mt < 4; ++mt)  // hi hi + mid mid
        acc[mt][nt] = mfma_bf16((v4u){aw[mt].z, aw[mt].w, am[mt].x, am[mt].y}, bw, acc[mt][nt]);
    }
    store(buf ^ 1);  // the other buffer was last read before the previous barrier
    __syncthreads();
  }
  // acc[mt][nt][v] = S[row wm + 16 mt + 4 k4 + v][col wn + 16 nt + l16]
  float* Sh = S + (int64_t)h * W;
#pragma unroll
  for (int mt = 0; mt < 4; ++mt)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int row = ib * BM + wm + mt * 16 + 4 * k4 + v;
      if (row >= n) continue;
#pragma unroll
      for (int nt = 0; nt < 4; ++nt) {
        const int col = cb * BN + wn + nt * 16 + l16;
        if (col < W) Sh[(int64_t)row * ldt + col] = acc[mt][nt][v];
      }
    }
}

}  // namespace

int dense_lda(int n) { return (n + 31) / 32 * 32; }  // a multiple of the K slab

hipError_t launch_dense_alpha(const float* alpha, int n, int H, float* A, int32_t* order, hipStream_t s) {
  if (n == 0) return hipSuccess;
  const int lda = dense_lda(n), chunks = (lda + kPadCols - 1) / kPadCols, groups = (H + kPadHeads - 1) / kPadHeads;
  const int64_t blocks = (int64_t)n * chunks * groups;
  if (blocks > 0x7fffffff) return hipErrorInvalidValue;
  k_dense_alpha_pad<<<(unsigned)blocks, kPadCols, 0, s>>>(alpha, n, H, lda, chunks, groups, A, order);
  return hipGetLastError();
}

hipError_t launch_dense_aggregate(const float* A, int n, const float* T, int dimT, int C, int H, float* S,
                                  hipStream_t s) {
  if (n == 0) return hipSuccess;
  const int dh = C / H, W = dimT * dh;
  if (W < 4 || W % 4) return hipErrorInvalidValue;
  constexpr int wgm = 4, wgn = 2;  // waves in M and N
  const int n_ib = (n + 64 * wgm - 1) / (64 * wgm), n_cb = (W + 64 * wgn - 1) / (64 * wgn);
  const int64_t tiles = (int64_t)H * n_ib * n_cb;
  const int64_t per_xcd = (tiles + 7) / 8;
  if (8 * per_xcd > 0x7fffffff) return hipErrorInvalidValue;
  const int64_t ldt = (int64_t)dimT * C;
  k_dense_gemm<wgm, wgn><<<(unsigned)(8 * per_xcd), 64 * wgm * wgn, 0, s>>>(A, dense_lda(n), n, T, ldt, W, S, n_ib, n_cb,
                                                                            H, (int)per_xcd);
  return hipGetLastError();
}

}  // namespace e2f
