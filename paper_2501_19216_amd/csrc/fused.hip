// The fused aggregation of the Wigner-6j convolution: products, coupling and
// output of a receiver in one kernel.  The local expansion of Thm. 3.3 is
// taken about the receiver itself, p_i = 0: of the receiver's harmonics
// R^(u)(p_i) only u = 0 is left, the recoupling weights are 1, and
//   y_i[o] = sum_{be, q} K[o][be][q] sum_j alpha_ij R_be(r_i - r_j) h_j[q]
// with K the path-weighted real Clebsch-Gordan tensors.  The sum over the
// neighbours is still taken before the coupling, which therefore costs the
// same for every row length.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "agg_layout.h"
#include "e2f_launch.h"
#include "split_bf16.h"

namespace e2f {
namespace {

// How far apart in the order the receivers of a workgroup lie (see below).  Flat
// around 64: 20,000 atoms, L = 4 3.12, 3.07, 3.09 and 3.14 ms with 1, 16, 64 and
// 256, 5,001 atoms 772, 764, 758 and 886 us, 3,000 atoms, L = 5 503, 500, 507, 590.
constexpr int kAggStride = 64;

// One workgroup: rpw receivers of one group of 16 V channels (V = agg_vec or 1),
// of any heads: the weight alpha_ij of a lane's head multiplies its features,
// and the harmonics R of an edge serve every channel.  Edges are taken 16 a
// step; edge 4 r + k4 of a step belongs to lane group k4 (r < 4).  A slot is a
// component q: V column tiles, tile v the channels V l16 + v, whose values of
// one sender a lane loads together.  G of a slot stays in its wave's
// accumulators over the whole row, and the coupling reads it there: element s
// of the accumulator of row tile mt is the B operand of the step of group 4 mt
// + s (agg_layout.h).
//
// Per step and slot a lane loads its four senders' values (a step ahead, into
// the registers just consumed), weights them and multiplies them by the step's
// harmonics, staged in LDS by all waves a step ahead.
//   SPLIT: every value is split into three bf16 parts (split_pair) and the
//   six cross products that reach 2^-24 of the product are summed in float
//   by three v_mfma_f32_16x16x32_bf16 a row tile, the four edges of a lane
//   filling their K: {mid01, mid23, hi01, hi23} x {hi, hi, hi, hi}, the same
//   x {mid, mid, mid, mid}, {hi01, hi23, lo01, lo23} x {lo, lo, hi, hi}.
//   Else: four v_mfma_f32_16x16x4f32, those of edges past the row's end
//   skipped.
// Edges past the row's end repeat its last sender with a weight of zero.
//
// OFF: unsigned where byte offsets into the features fit 32 bits.
template <int L, bool SPLIT, typename OFF, int V>
__global__ __launch_bounds__(64 * agg_waves(L)) __attribute__((amdgpu_waves_per_eu(L >= 2 ? 2 : 3)))
void k_aggregate_fused(const float* __restrict__ Re, const int64_t* __restrict__ row_ptr,
                       const int32_t* __restrict__ col, const float* __restrict__ alpha, int n_edges,
                       const float* __restrict__ feat, const int32_t* __restrict__ order, int first, int n, int rpw,
                       int nblk, int lg, int per_xcd, int C, int H, int n_nodes, const int* __restrict__ index,
                       const float4* __restrict__ coef, float* __restrict__ y) {
  constexpr AggMap M = agg_map(L);
  constexpr int NK = M.nk, MT = M.mt, NW = M.nw, TW = M.tw, NG = M.ng, KEYS = M.keys;
  constexpr int NT = 64 * NW, NQ = (NG + 3) / 4, W = 16 * V;
  constexpr bool PIPE = MT == 2;
  constexpr int NST = (4 * NK + NT - 1) / NT;  // staging passes: a thread per (component, k4)
  typedef float vec __attribute__((ext_vector_type(V)));
  __shared__ float4 la[2][MT * 64 + 1];  // R: split {lo01, lo23, hi01, hi23}, else four floats
  __shared__ uint2 lm[SPLIT ? 2 : 1][SPLIT ? MT * 64 + 1 : 1];  // {mid01, mid23} (the last entries: idle threads')
  __shared__ float red[NW > 1 ? NW * KEYS * V * 256 : 1];
  // XCD x takes a contiguous range of items; an item is a receiver set and a
  // column group, the column groups of one 128-byte line (lg of them) first,
  // then the sets, then the lines: the workgroups in flight on an XCD read the
  // same lines of neighbouring atoms, which then stay in its L2.  The rpw
  // receivers of a set are kAggStride apart, so that the kAggStride sets in
  // flight side by side move through the order together.
  const int units = (C + W - 1) / W;
  const int item = (blockIdx.x % 8) * per_xcd + blockIdx.x / 8;
  const int unit = item / (nblk * lg) * lg + item % lg, set = item / lg % nblk;
  const int r0 = set / kAggStride * (kAggStride * rpw) + set % kAggStride;
  if (unit >= units || r0 >= n) return;
  const int nrec = min(rpw, (n - 1 - r0) / kAggStride + 1);
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = NW > 1 ? __builtin_amdgcn_readfirstlane(tid >> 6) : 0;
  const int l16 = lane & 15, k4 = lane >> 4;
  // the lane's channels and head (lanes past C repeat its last channels and
  // store nothing)
  const int c0 = unit * W, cl = min(c0 + V * l16, C - V), head = cl / (C / H);
  const bool cok = c0 + V * l16 < C;
  // receivers and their edge ranges, one a lane (clamped to [0, E]: a
  // malformed graph cannot move a read outside the caller's buffers)
  int vi = 0, va = 0, vb = 0;
  if (lane < nrec) {
    vi = first + r0 + lane * kAggStride;
    if (order) vi = order[vi];
    const int64_t p0 = row_ptr[vi], p1 = row_ptr[vi + 1];
    va = (int)max((int64_t)0, min(p0, (int64_t)n_edges));
    vb = (int)max((int64_t)va, min(p1, (int64_t)n_edges));
  }
  for (unsigned long long z = __ballot(lane < nrec && va == vb); z; z &= z - 1) {  // isolated: zero rows
    const int i = __builtin_amdgcn_readlane(vi, __builtin_ctzll(z));
    for (int e = tid; e < NK * W; e += NT)
      if (c0 + e % W < C) y[((size_t)i * NK + e / W) * C + c0 + e % W] = 0.0f;
  }
  const unsigned long long live = __ballot(va < vb);
  if (!live) return;
  // the steps of the receivers with edges, in order
  struct Step {
    int r, e, end;
  };
  auto row = [&](unsigned long long m) {
    const int r = __builtin_ctzll(m);
    return Step{r, __builtin_amdgcn_readlane(va, r), __builtin_amdgcn_readlane(vb, r)};
  };
  auto next = [&](Step s) {  // past the last step: the last step again
    if (s.end - s.e > 16) return Step{s.r, s.e + 16, s.end};  // (s.e + 16 may pass 2^31 - 1)
    const unsigned long long m = live & ~((2ull << s.r) - 1);
    return m ? row(m) : s;
  };
  // byte offsets of the wave's slots
  const int* slotq = index + NK + wave * TW;
  OFF qoff[TW];
#pragma unroll
  for (int i = 0; i < TW; ++i) qoff[i] = (OFF)slotq[i] * (OFF)C * 4;
  const char* fbase = (const char*)feat;
  const OFF stride = (OFF)NK * C * 4;
  // (edge e of a step: a uniform base and a lane offset; past the row's end
  // the last edge)
  auto senders = [&](Step s, int (&j)[4]) {
    const int* cb = col + s.e;
#pragma unroll
    for (int r = 0; r < 4; ++r) j[r] = cb[(unsigned)min(4 * r + k4, s.end - s.e - 1)];
  };
  auto offsets = [&](const int (&j)[4], OFF (&o)[4]) {
#pragma unroll
    for (int r = 0; r < 4; ++r) o[r] = (OFF)((unsigned)j[r] < (unsigned)n_nodes ? j[r] : 0) * stride + (OFF)cl * 4;
  };
  auto value = [&](int i, OFF o) { return *(const vec*)(fbase + qoff[i] + o); };
  // the lane's weights of a step (zero past the row's end)
  const int wstride = alpha ? H : 0;
  auto weights = [&](Step s, float (&a)[4]) {
    const float* wb = alpha ? alpha + (size_t)s.e * H : Re;  // without weights any readable float
#pragma unroll
    for (int r = 0; r < 4; ++r)
      a[r] = wb[__umul24((unsigned)min(4 * r + k4, s.end - s.e - 1), wstride) + (alpha ? head : 0)];
  };
  auto masked = [&](Step s, float (&a)[4]) {
#pragma unroll
    for (int r = 0; r < 4; ++r) a[r] = 4 * r + k4 < s.end - s.e ? (alpha ? a[r] : 1.0f) : 0.0f;
  };
  // staging: thread (component be, lane group g) holds the step's four edges
  // 4 r + g
  int sbe[NST], sg[NST], spos[NST];
#pragma unroll
  for (int u = 0; u < NST; ++u) {
    const int t = tid + u * NT;
    const bool son = t < 4 * NK;
    sbe[u] = son ? t % NK : 0;
    sg[u] = son ? t / NK : 0;
    const int p = index[sbe[u]];
    spos[u] = son ? (p >> 4) * 64 + sg[u] * 16 + (p & 15) : MT * 64;
  }
  float sr[NST][4], pr[NST][4];
  auto fetch = [&](Step s, float (&v)[NST][4]) {
    const float* rb = Re + (size_t)s.e * NK;
#pragma unroll
    for (int u = 0; u < NST; ++u)
#pragma unroll
      for (int r = 0; r < 4; ++r) v[u][r] = rb[__umul24((unsigned)min(4 * r + sg[u], s.end - s.e - 1), NK) + sbe[u]];
  };
  auto store = [&](int b, const float (&v)[NST][4]) {
#pragma unroll
    for (int u = 0; u < NST; ++u) {
      if constexpr (SPLIT) {
        unsigned h[2], m[2], l[2];
        split_pair(v[u][0], v[u][1], h[0], m[0], l[0]);
        split_pair(v[u][2], v[u][3], h[1], m[1], l[1]);
        la[b][spos[u]] = __builtin_bit_cast(float4, (v4u){l[0], l[1], h[0], h[1]});
        lm[b][spos[u]] = make_uint2(m[0], m[1]);
      } else {
        la[b][spos[u]] = make_float4(v[u][0], v[u][1], v[u][2], v[u][3]);
      }
    }
  };
  v4f acc[TW][V][MT];
#pragma unroll
  for (int i = 0; i < TW; ++i)
#pragma unroll
    for (int v = 0; v < V; ++v)
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) acc[i][v][mt] = (v4f){0.f, 0.f, 0.f, 0.f};
  // rows without a component stay zero
  for (int q = tid; q < 2 * (MT * 64 + 1); q += NT) {
    (&la[0][0])[q] = make_float4(0.f, 0.f, 0.f, 0.f);
    if constexpr (SPLIT) (&lm[0][0])[q] = make_uint2(0, 0);
  }
  Step s0 = row(live), s1 = next(s0);
  int jn[4];
  OFF o[4];
  vec f[TW][4];
  float a0[4], a1[4];  // the weights of s0 and s1
  // (the loads in the order of the loop below, so that its waits, which have to
  // hold from here too, leave the features of the next step in flight)
  senders(s0, jn);
  fetch(s0, pr);
  weights(s0, a0);
  offsets(jn, o);
  fetch(s1, sr);
  senders(s1, jn);
#pragma unroll
  for (int i = 0; i < TW; ++i)
#pragma unroll
    for (int r = 0; r < 4; ++r) f[i][r] = value(i, o[r]);
  __syncthreads();
  store(0, pr);
  for (int b = 0;; b ^= 1) {
    __syncthreads();  // R of s0 is staged; the other buffer is free
    const Step s2 = next(s1);
    masked(s0, a0);
    offsets(jn, o);
    // (the next step's R goes to the other buffer, and the loads of the one
    // after start)
    if constexpr (SPLIT) {
      if (!PIPE) {
        store(b ^ 1, sr);
        fetch(s2, sr);
        senders(s2, jn);
        weights(s1, a1);
      }
      v4u A0[MT], A1[MT], A2[MT];
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) {
        A2[mt] = __builtin_bit_cast(v4u, la[b][mt * 64 + lane]);
        const uint2 m = lm[b][mt * 64 + lane];
        A0[mt] = (v4u){A2[mt][2], A2[mt][3], A2[mt][2], A2[mt][3]};
        A1[mt] = (v4u){m.x, m.y, m.x, m.y};
      }
      // column tile x of the step: slot x / V, channels V l16 + x % V
      unsigned h[2][2], m[2][2], l[2][2];  // the split values of two tiles
      auto split = [&](int x) {
        const int i = x / V, v = x % V, w = PIPE ? x & 1 : 0;
        split_pair(a0[0] * f[i][0][v], a0[1] * f[i][1][v], h[w][0], m[w][0], l[w][0]);
        split_pair(a0[2] * f[i][2][v], a0[3] * f[i][3][v], h[w][1], m[w][1], l[w][1]);
        if (v == V - 1) {
#pragma unroll
          for (int r = 0; r < 4; ++r) f[i][r] = value(i, o[r]);
        }
      };
      if (PIPE) split(0);
#pragma unroll
      for (int x = 0; x < TW * V; ++x) {
        const int i = x / V, v = x % V, w = PIPE ? x & 1 : 0;
        if (!PIPE) split(x);
        else if (x + 1 < TW * V) split(x + 1);
        if (PIPE && x == 1) store(b ^ 1, sr);
        if (PIPE && x == 2) fetch(s2, sr), senders(s2, jn), weights(s1, a1);
        const v4u bm = {m[w][0], m[w][1], h[w][0], h[w][1]}, bl = {h[w][0], h[w][1], l[w][0], l[w][1]};
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) acc[i][v][mt] = mfma_bf16(A0[mt], bm, acc[i][v][mt]);
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) acc[i][v][mt] = mfma_bf16(A1[mt], bm, acc[i][v][mt]);
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) acc[i][v][mt] = mfma_bf16(A2[mt], bl, acc[i][v][mt]);
        // the next tile's split and loads between this one's matrix
        // instructions: a wave issues in order, and a burst of them would
        // keep its own ALU work waiting behind the matrix core
#pragma unroll
        for (int u = 0; u < 3 * MT && PIPE; ++u) {
          __builtin_amdgcn_sched_group_barrier(0x8, 1, 0);
          __builtin_amdgcn_sched_group_barrier(0x2, 5, 0);
          if (u >= 3 * MT - 4) __builtin_amdgcn_sched_group_barrier(0x20, 1, 0);
        }
        if (PIPE) __builtin_amdgcn_sched_barrier(0);
      }
    } else {
      store(b ^ 1, sr);
      fetch(s2, sr);
      senders(s2, jn);
      weights(s1, a1);
      float4 A[MT];
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) A[mt] = la[b][mt * 64 + lane];
      const int here = s0.end - s0.e, then = s1.end - s1.e;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        if (4 * r < here) {
#pragma unroll
          for (int i = 0; i < TW; ++i)
#pragma unroll
            for (int v = 0; v < V; ++v)
#pragma unroll
              for (int mt = 0; mt < MT; ++mt)
                acc[i][v][mt] = __builtin_amdgcn_mfma_f32_16x16x4f32((&A[mt].x)[r], a0[r] * f[i][r][v],
                                                                     acc[i][v][mt], 0, 0, 0);
        }
        if (4 * r < then) {
#pragma unroll
          for (int i = 0; i < TW; ++i) f[i][r] = value(i, o[r]);
        }
      }
    }
    if (s0.end - s0.e <= 16) {  // the receiver's last step: couple
      const int i0 = __builtin_amdgcn_readlane(vi, s0.r);
      // (PARTS sums an accumulator, so that consecutive steps do not wait for
      // each other)
      constexpr int PARTS = KEYS * V == 1 ? (NG < 2 ? NG : 2) : 1;
      v4f d[KEYS][V][PARTS];
#pragma unroll
      for (int x = 0; x < KEYS * V * PARTS; ++x) (&d[0][0][0])[x] = (v4f){0.f, 0.f, 0.f, 0.f};
      const char* cw = (const char*)(coef + (size_t)wave * TW * NQ * 64);
      unsigned lo = (unsigned)lane * 16;
      asm("" : "+v"(lo));  // keeps the table's addresses out of the registers that live through the steps
      // the table is read AHEAD entries ahead (each is a read from L2; 20,000 atoms,
      // L = 4 3.11, 3.09 and 3.20 ms with 3, 6 and 12, 3,000 atoms, L = 5 505, 507 and
      // 614 us)
      constexpr int ALL = TW * NQ, AHEAD = ALL < 6 ? ALL : 6;
      float4 kk[AHEAD];
      auto entry = [&](int m) { return *(const float4*)(cw + m * 1024 + lo); };
#pragma unroll
      for (int m = 0; m < AHEAD; ++m) kk[m] = entry(m);
#pragma unroll
      for (int m = 0; m < ALL; ++m) {
        const int i = m / NQ, q = m % NQ;
        const float4 k = kk[m % AHEAD];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int g = 4 * q + u;
          if (g < NG) {
#pragma unroll
            for (int v = 0; v < V; ++v) {
              v4f& dd = d[M.gkey[g < 16 ? g : 0] ^ M.skey[i]][v][g % PARTS];
              dd = __builtin_amdgcn_mfma_f32_16x16x4f32((&k.x)[u], acc[i][v][(g / 4) % MT][g % 4], dd, 0, 0, 0);
            }
          }
        }
        if (m + AHEAD < ALL) kk[m % AHEAD] = entry(m + AHEAD);
        __builtin_amdgcn_sched_barrier(0);
      }
#pragma unroll
      for (int i = 0; i < TW; ++i)
#pragma unroll
        for (int v = 0; v < V; ++v)
#pragma unroll
          for (int mt = 0; mt < MT; ++mt) acc[i][v][mt] = (v4f){0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int x = 0; x < KEYS; ++x)
#pragma unroll
        for (int v = 0; v < V; ++v)
#pragma unroll
          for (int u = 1; u < PARTS; ++u) d[x][v][0] += d[x][v][u];
      float* yi = y + (size_t)i0 * NK * C + c0;
      if constexpr (NW == 1) {
#pragma unroll
        for (int x = 0; x < KEYS; ++x)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            // row 4 k4 + r of key x
            int k = -1;
#pragma unroll
            for (int u = 0; u < 4; ++u) k = k4 == u ? M.rows[x][4 * u + r] : k;
            vec z;
#pragma unroll
            for (int v = 0; v < V; ++v) z[v] = d[x][v][0][r];
            if (k >= 0 && cok) *(vec*)(yi + (size_t)k * C + V * l16) = z;
          }
      } else {
        // element (key, row, channel), summed over the waves (wave w holds key
        // x in accumulator x ^ its key)
#pragma unroll
        for (int x = 0; x < KEYS; ++x)
#pragma unroll
          for (int v = 0; v < V; ++v)
#pragma unroll
            for (int r = 0; r < 4; ++r) red[((wave * KEYS + x) * 4 + r) * 64 * V + lane * V + v] = d[x][v][0][r];
        __syncthreads();
        for (int e = tid; e < NK * W; e += NT) {
          const int k = e / W, t = e % W;
          const int kk = index[NK + NW * TW + k], key = kk / 16, rw = kk % 16;
          float sum = 0.0f;
#pragma unroll
          for (int w = 0; w < NW; ++w)
            sum += red[((w * KEYS + (key ^ M.wkey[w])) * 4 + rw % 4) * 64 * V + (rw / 4) * W + t];
          if (c0 + t < C) yi[(size_t)k * C + t] = sum;
        }
        // (the next store to red follows the barrier of the next step)
      }
      if (s1.r == s0.r) return;  // no receiver left (uniform over the workgroup)
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) a0[r] = a1[r];
    s0 = s1;
    s1 = s2;
  }
}

}  // namespace

hipError_t launch_aggregate_fused(int L, const float* Re, const int64_t* row_ptr, const int32_t* col,
                                  const float* alpha, int64_t n_edges, const float* feat, const int32_t* order,
                                  int first, int n, int C, int H, int n_nodes, const int* index, const float* coef,
                                  float* y, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  const bool wide = (double)n_nodes * nk_of(L) * C * 4.0 > 4.0e9;
  // One channel a lane where two would leave half of the last column group
  // empty, as long as that is dearer than the smaller groups (a group of 16 costs
  // 0.55 of one of 32: even at nine).  20,000 atoms, 80 neighbours, L = 2: C = 4
  // and 16 295 us with two channels a lane, 202 with one, C = 48 498 and 442, but
  // C = 20 296 and 315, C = 32 297 and 316, C = 128 906 and 996; L = 5, C = 16 1.64
  // and 1.00 ms, C = 48 3.12 and 2.78; 3,000 atoms, L = 5, C = 80 781 and 756 us.
  const int groups = (C + 15) / 16;
  const bool narrow = groups % 2 == 1 && groups <= 7;
#define E2F_AGG(LL, SP)                                                                                           \
  case LL:                                                                                                        \
    if (agg_vec(LL) > 1 && narrow) E2F_AGG_V(LL, SP, 1);                                                          \
    else E2F_AGG_V(LL, SP, agg_vec(LL));                                                                          \
    break;
#define E2F_AGG_V(LL, SP, VV)                                                                                     \
  do {                                                                                                            \
    constexpr int nw = agg_waves(LL), V = VV, W = 16 * V;                                                         \
    const int units = (C + W - 1) / W;                                                                            \
    int lg = std::min(32 / W, units); /* column groups of one line */                                             \
    while (units % lg) --lg;                                                                                      \
    /* receivers a workgroup: the steps of consecutive ones overlap, as long as every CU has work four times  */   \
    /* over.  One, 4, 8 and 16 at most: 20,000 atoms, L = 4 3.30, 3.06, 3.09, 3.18 ms; 10,000 atoms, L = 3 495,  */ \
    /* 446, 435, 440 us.  Work once, 4 and 16 times over: 7,680 atoms in rows of 6, L = 3 87, 91 and 110 us;    */  \
    /* 3,000 atoms, L = 5 482, 507 and 550; 1,517 atoms, L = 2 34.6, 33.3 and 33.2                              */  \
    const int64_t slots = 256 * 8 / nw;                                                                           \
    const int rpw = (int)std::max<int64_t>(1, std::min<int64_t>(8, (int64_t)n * units / (slots * 4)));            \
    const int nblk = (n + kAggStride * rpw - 1) / (kAggStride * rpw) * kAggStride;                                \
    const int64_t per = ((int64_t)nblk * units + 7) / 8;                                                          \
    if (per * 8 > 0x7fffffff) return hipErrorInvalidValue;                                                        \
    if (wide)                                                                                                     \
      k_aggregate_fused<LL, SP, uint64_t, V><<<(unsigned)(8 * per), 64 * nw, 0, s>>>(                                \
          Re, row_ptr, col, alpha, (int)n_edges, feat, order, first, n, rpw, nblk, lg, (int)per, C, H, n_nodes,   \
          index, (const float4*)coef, y);                                                                         \
    else                                                                                                          \
      k_aggregate_fused<LL, SP, uint32_t, V><<<(unsigned)(8 * per), 64 * nw, 0, s>>>(                                \
          Re, row_ptr, col, alpha, (int)n_edges, feat, order, first, n, rpw, nblk, lg, (int)per, C, H, n_nodes,   \
          index, (const float4*)coef, y);                                                                         \
    return hipGetLastError();                                                                                     \
  } while (0)
  switch (L) {
    E2F_AGG(0, false)
    E2F_AGG(1, false)
    E2F_AGG(2, false)
    E2F_AGG(3, false)
    E2F_AGG(4, true)
    E2F_AGG(5, true)
    E2F_AGG(6, true)
    default: return hipErrorInvalidValue;
  }
#undef E2F_AGG_V
#undef E2F_AGG
}

}  // namespace e2f
