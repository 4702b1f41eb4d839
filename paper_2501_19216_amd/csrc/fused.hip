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

namespace e2f {
namespace {

typedef float v4f __attribute__((ext_vector_type(4)));
typedef float v2f __attribute__((ext_vector_type(2)));
typedef __bf16 v2b __attribute__((ext_vector_type(2)));
typedef __bf16 v8b __attribute__((ext_vector_type(8)));
typedef unsigned v4u __attribute__((ext_vector_type(4)));

// Two floats as three words of bfloat16 pairs, x = hi + mid + lo exactly: hi
// and mid rounded to nearest, lo the rest (8 + 8 + 8 bits hold the 24).
__device__ __forceinline__ void split_pair(float x, float y, unsigned& hi, unsigned& mid, unsigned& lo) {
  hi = __builtin_bit_cast(unsigned, __builtin_convertvector((v2f){x, y}, v2b));
  const float rx = x - __uint_as_float(hi << 16), ry = y - __uint_as_float(hi & 0xffff0000u);
  mid = __builtin_bit_cast(unsigned, __builtin_convertvector((v2f){rx, ry}, v2b));
  const float sx = rx - __uint_as_float(mid << 16), sy = ry - __uint_as_float(mid & 0xffff0000u);
  lo = __builtin_bit_cast(unsigned, __builtin_convertvector((v2f){sx, sy}, v2b));
}

__device__ __forceinline__ v4f mfma_bf16(v4u a, v4u b, v4f c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(v8b, a), __builtin_bit_cast(v8b, b), c, 0, 0, 0);
}

constexpr int kAggStride = 64;

// One workgroup: rpw receivers of one group of DH = 16 / P channels of a head.  Edges are taken 16 a step; edge 4 r + k4 of a step
// belongs to lane group k4 (r < 4).  A slot is a column tile of P components
// q x DH channels; G of a slot stays in its wave's accumulators over the whole
// row, and the coupling reads it there: element s of the accumulator of row
// tile mt is the B operand of the step of group 4 mt + s (agg_layout.h).
//
// Per step and slot a lane loads its four senders' values (a step ahead, into
// the registers just consumed) and multiplies them by the step's weighted
// harmonics alpha R, staged in LDS by all waves a step ahead.
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
template <int L, int P, bool SPLIT, typename OFF>
__global__ __launch_bounds__(64 * agg_waves(L, P)) __attribute__((amdgpu_waves_per_eu(L >= 4 || (L == 3 && P == 1) ? 2 : 3)))
void k_aggregate_fused(const float* __restrict__ Re, const int64_t* __restrict__ row_ptr,
                       const int32_t* __restrict__ col, const float* __restrict__ alpha, int n_edges,
                       const float* __restrict__ feat, const int32_t* __restrict__ order, int first, int n, int rpw,
                       int nblk, int lg, int per_xcd, int C, int H, int uph, int n_nodes, const int* __restrict__ index,
                       const float4* __restrict__ coef, float* __restrict__ y) {
  constexpr AggMap M = agg_map(L, P);
  constexpr int NK = M.nk, DH = M.dh, MT = M.mt, NW = M.nw, TW = M.tw, NG = M.ng, RB = M.rb, KEYS = M.keys;
  constexpr int NT = 64 * NW, NACC = KEYS * RB, NQ = (NG * RB + 3) / 4;
  constexpr bool PIPE = MT == 2;
  constexpr int NST = (4 * NK + NT - 1) / NT;  // staging passes: a thread per (component, k4)
  __shared__ float4 la[2][MT * 64 + 1];  // alpha R: split {lo01, lo23, hi01, hi23}, else four floats
  __shared__ uint2 lm[SPLIT ? 2 : 1][SPLIT ? MT * 64 + 1 : 1];  // {mid01, mid23} (the last entries: idle threads')
  __shared__ float red[NW * P > 1 ? NW * NACC * 256 : 1];
  // XCD x takes a contiguous range of items; an item is a receiver set and a
  // column group, the column groups of one 128-byte line (lg of them) first,
  // then the sets, then the lines: the workgroups in flight on an XCD read the
  // same lines of neighbouring atoms, which then stay in its L2.  The rpw
  // receivers of a set are kAggStride apart, so that the kAggStride sets in
  // flight side by side move through the order together.
  const int item = (blockIdx.x % 8) * per_xcd + blockIdx.x / 8;
  const int unit = item / (nblk * lg) * lg + item % lg, set = item / lg % nblk;
  const int r0 = set / kAggStride * (kAggStride * rpw) + set % kAggStride;
  if (unit >= C / DH || r0 >= n) return;
  const int nrec = min(rpw, (n - 1 - r0) / kAggStride + 1);
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = NW > 1 ? __builtin_amdgcn_readfirstlane(tid >> 6) : 0;
  const int l16 = lane & 15, k4 = lane >> 4;
  const int c0 = unit * DH, head = unit / uph;
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
    for (int e = tid; e < NK * DH; e += NT) y[((size_t)i * NK + e / DH) * C + c0 + e % DH] = 0.0f;
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
    if (s.e + 16 < s.end) return Step{s.r, s.e + 16, s.end};
    const unsigned long long m = live & ~((2ull << s.r) - 1);
    return m ? row(m) : s;
  };
  // column offsets of the wave's slots
  const int* slotq = index + NK + wave * TW * P;
  OFF qoff[TW];
#pragma unroll
  for (int i = 0; i < TW; ++i)
    qoff[i] = (OFF)(P == 1 ? slotq[i] : slotq[i * P + l16 / DH]) * (OFF)C * 4 +
              (P == 1 ? (OFF)0 : (OFF)(l16 % DH) * 4);
  const char* fbase = (const char*)(feat + c0);
  const OFF loff = P == 1 ? (OFF)l16 * 4 : 0;
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
    for (int r = 0; r < 4; ++r) o[r] = (OFF)((unsigned)j[r] < (unsigned)n_nodes ? j[r] : 0) * stride + loff;
  };
  auto value = [&](int i, OFF o) {
    if constexpr (P == 1) return *(const float*)(fbase + qoff[i] + o);
    else return *(const float*)(fbase + (qoff[i] + o));
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
  float sr[NST][4], sw[NST][4];
  const float* wbase = alpha ? alpha + head : Re;  // without weights any readable float
  const int wstride = alpha ? H : 0;
  auto fetch = [&](Step s) {
    const float* rb = Re + (size_t)s.e * NK;
    const float* wb = wbase + (size_t)s.e * wstride;
#pragma unroll
    for (int u = 0; u < NST; ++u)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const unsigned e = min(4 * r + sg[u], s.end - s.e - 1);
        sr[u][r] = rb[__umul24(e, NK) + sbe[u]];
        sw[u][r] = wb[__umul24(e, wstride)];
      }
  };
  auto store = [&](Step s, int b) {
#pragma unroll
    for (int u = 0; u < NST; ++u) {
      float v[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) v[r] = 4 * r + sg[u] < s.end - s.e ? (alpha ? sw[u][r] : 1.0f) * sr[u][r] : 0.0f;
      if constexpr (SPLIT) {
        unsigned h[2], m[2], l[2];
        split_pair(v[0], v[1], h[0], m[0], l[0]);
        split_pair(v[2], v[3], h[1], m[1], l[1]);
        la[b][spos[u]] = __builtin_bit_cast(float4, (v4u){l[0], l[1], h[0], h[1]});
        lm[b][spos[u]] = make_uint2(m[0], m[1]);
      } else {
        la[b][spos[u]] = make_float4(v[0], v[1], v[2], v[3]);
      }
    }
  };
  v4f acc[TW][MT];
#pragma unroll
  for (int i = 0; i < TW; ++i)
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) acc[i][mt] = (v4f){0.f, 0.f, 0.f, 0.f};
  // rows without a component stay zero
  for (int q = tid; q < 2 * (MT * 64 + 1); q += NT) {
    (&la[0][0])[q] = make_float4(0.f, 0.f, 0.f, 0.f);
    if constexpr (SPLIT) (&lm[0][0])[q] = make_uint2(0, 0);
  }
  Step s0 = row(live), s1 = next(s0);
  int jn[4];
  OFF o[4];
  float f[TW][4];
  senders(s0, jn);
  fetch(s0);
  offsets(jn, o);
#pragma unroll
  for (int i = 0; i < TW; ++i)
#pragma unroll
    for (int r = 0; r < 4; ++r) f[i][r] = value(i, o[r]);
  senders(s1, jn);
  __syncthreads();
  store(s0, 0);
  fetch(s1);
  for (int b = 0;; b ^= 1) {
    __syncthreads();  // alpha R of s0 is staged; the other buffer is free
    const Step s2 = next(s1);
    offsets(jn, o);
    // the next step's alpha R goes to the other buffer, and the loads of the
    // one after start
    auto stage = [&] {
      store(s1, b ^ 1);
      fetch(s2);
      senders(s2, jn);
    };
    if constexpr (SPLIT) {
      if (!PIPE) stage();
      v4u a0[MT], a1[MT], a2[MT];
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) {
        a2[mt] = __builtin_bit_cast(v4u, la[b][mt * 64 + lane]);
        const uint2 m = lm[b][mt * 64 + lane];
        a0[mt] = (v4u){a2[mt][2], a2[mt][3], a2[mt][2], a2[mt][3]};
        a1[mt] = (v4u){m.x, m.y, m.x, m.y};
      }
      unsigned h[2][2], m[2][2], l[2][2];  // the split values of two slots
      auto split = [&](int i) {
        split_pair(f[i][0], f[i][1], h[i & 1][0], m[i & 1][0], l[i & 1][0]);
        split_pair(f[i][2], f[i][3], h[i & 1][1], m[i & 1][1], l[i & 1][1]);
#pragma unroll
        for (int r = 0; r < 4; ++r) f[i][r] = value(i, o[r]);
      };
      if (PIPE) split(0);
#pragma unroll
      for (int i = 0; i < TW; ++i) {
        if (!PIPE) split(i);
        else if (i + 1 < TW) split(i + 1);
        if (PIPE && i == TW / 2) stage();
        const int w = i & 1;
        const v4u bm = {m[w][0], m[w][1], h[w][0], h[w][1]}, bl = {h[w][0], h[w][1], l[w][0], l[w][1]};
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) acc[i][mt] = mfma_bf16(a0[mt], bm, acc[i][mt]);
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) acc[i][mt] = mfma_bf16(a1[mt], bm, acc[i][mt]);
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) acc[i][mt] = mfma_bf16(a2[mt], bl, acc[i][mt]);
        // the next slot's split and loads between this one's matrix
        // instructions: a wave issues in order, and a burst of them would
        // keep its own ALU work waiting behind the matrix core
#pragma unroll
        for (int u = 0; u < 3 * MT && PIPE; ++u) {
          __builtin_amdgcn_sched_group_barrier(0x8, 1, 0);
          __builtin_amdgcn_sched_group_barrier(0x2, (28 + (P > 1 ? 4 : 0) + 3 * MT - 1) / (3 * MT), 0);
          if (u >= 3 * MT - 4) __builtin_amdgcn_sched_group_barrier(0x20, 1, 0);
        }
      }
    } else {
      stage();
      float4 a[MT];
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) a[mt] = la[b][mt * 64 + lane];
      const int here = s0.end - s0.e, then = s1.end - s1.e;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        if (4 * r < here) {
#pragma unroll
          for (int i = 0; i < TW; ++i)
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
              acc[i][mt] = __builtin_amdgcn_mfma_f32_16x16x4f32((&a[mt].x)[r], f[i][r], acc[i][mt], 0, 0, 0);
        }
        if (4 * r < then) {
#pragma unroll
          for (int i = 0; i < TW; ++i) f[i][r] = value(i, o[r]);
        }
      }
    }
    if (s0.e + 16 >= s0.end) {  // the receiver's last step: couple
      const int i0 = __builtin_amdgcn_readlane(vi, s0.r);
      v4f d[NACC];
#pragma unroll
      for (int x = 0; x < NACC; ++x) d[x] = (v4f){0.f, 0.f, 0.f, 0.f};
      const char* cw = (const char*)(coef + (size_t)wave * TW * NQ * 64);
      unsigned lo = (unsigned)lane * 16;
      asm("" : "+v"(lo));  // keeps the table's addresses out of the registers that live through the steps
#pragma unroll
      for (int i = 0; i < TW; ++i)
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
          const float4 k = *(const float4*)(cw + (i * NQ + q) * 1024 + lo);
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            const int g = (4 * q + u) / RB, rb = (4 * q + u) % RB;
            if (g < NG) {
              v4f& dd = d[(M.gkey[g < 16 ? g : 0] ^ M.skey[i]) * RB + rb];
              dd = __builtin_amdgcn_mfma_f32_16x16x4f32((&k.x)[u], acc[i][(g / 4) % MT][g % 4], dd, 0, 0, 0);
            }
          }
        }
#pragma unroll
      for (int i = 0; i < TW; ++i)
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) acc[i][mt] = (v4f){0.f, 0.f, 0.f, 0.f};
      float* yi = y + (size_t)i0 * NK * C + c0;
      if constexpr (NW * P == 1) {
#pragma unroll
        for (int x = 0; x < NACC; ++x)
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            // row 4 k4 + v of key x
            int k = -1;
#pragma unroll
            for (int u = 0; u < 4; ++u) k = k4 == u ? M.rows[x][4 * u + v] : k;
            if (k >= 0) yi[(size_t)k * C + l16] = d[x][v];
          }
      } else {
        // element (key, index of the component, channel t) is row p DH + index
        // % DH of row block index / DH, column p DH + t, summed over p and
        // the waves (wave w holds key x in accumulator x ^ its key)
#pragma unroll
        for (int x = 0; x < NACC; ++x)
#pragma unroll
          for (int v = 0; v < 4; ++v) red[(wave * NACC + x) * 256 + v * 64 + lane] = d[x][v];
        __syncthreads();
        for (int e = tid; e < NK * DH; e += NT) {
          const int k = e / DH, t = e % DH;
          const int kk = index[NK + NW * TW * P + k];
          const int key = kk / (RB * DH), idx = kk % (RB * DH), rb = idx / DH;
          float sum = 0.0f;
#pragma unroll
          for (int w = 0; w < NW; ++w)
#pragma unroll
            for (int p = 0; p < P; ++p) {
              const int rw = p * DH + idx % DH;
              sum += red[(w * NACC + (key ^ M.wkey[w]) * RB + rb) * 256 + (rw % 4) * 64 + (rw / 4) * 16 + p * DH + t];
            }
          yi[(size_t)k * C + t] = sum;
        }
        // (the next store to red follows the barrier of the next step)
      }
      if (s1.r == s0.r) return;  // no receiver left (uniform over the workgroup)
    }
    s0 = s1;
    s1 = s2;
  }
}

}  // namespace

// Channels a column group holds: 16, 8 or 4, the widest that divides a head.
int agg_group(int C, int H) {
  const int dh = C / H;
  return dh % 16 == 0 ? 16 : dh % 8 == 0 ? 8 : 4;
}

hipError_t launch_aggregate_fused(int L, const float* Re, const int64_t* row_ptr, const int32_t* col,
                                  const float* alpha, int64_t n_edges, const float* feat, const int32_t* order,
                                  int first, int n, int C, int H, int n_nodes, const int* index, const float* coef,
                                  float* y, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  const int dh = agg_group(C, H), P = 16 / dh, units = C / dh;
  const int nk = nk_of(L);
  int lg = std::min(32 / dh, units);  // column groups of one line
  while (units % lg) --lg;
  const bool wide = (double)n_nodes * nk * C * 4.0 > 4.0e9;
#define E2F_AGG(LL, PP, SP)                                                                                        \
  if (L == LL && P == PP) {                                                                                        \
    constexpr int nw = agg_waves(LL, PP);                                                                          \
    /* receivers a workgroup: the steps of consecutive ones overlap, as long as every CU has work */              \
    const int64_t slots = 256 * (LL >= 4 ? 8 : 12) / nw;                                                           \
    const int rpw = (int)std::max<int64_t>(1, std::min<int64_t>(8, (int64_t)n * units / (slots * 4)));             \
    const int nblk = (n + kAggStride * rpw - 1) / (kAggStride * rpw) * kAggStride;                                 \
    const int64_t per = ((int64_t)nblk * units + 7) / 8;                                                           \
    if (per * 8 > 0x7fffffff) return hipErrorInvalidValue;                                                         \
    if (wide)                                                                                                      \
      k_aggregate_fused<LL, PP, SP, uint64_t><<<(unsigned)(8 * per), 64 * nw, 0, s>>>(                             \
          Re, row_ptr, col, alpha, (int)n_edges, feat, order, first, n, rpw, nblk, lg, (int)per, C, H, C / H / dh,     \
          n_nodes, index, (const float4*)coef, y);                                                                 \
    else                                                                                                           \
      k_aggregate_fused<LL, PP, SP, uint32_t><<<(unsigned)(8 * per), 64 * nw, 0, s>>>(                             \
          Re, row_ptr, col, alpha, (int)n_edges, feat, order, first, n, rpw, nblk, lg, (int)per, C, H, C / H / dh,     \
          n_nodes, index, (const float4*)coef, y);                                                                 \
    return hipGetLastError();                                                                                      \
  }
#define E2F_AGG_L(LL, SP) E2F_AGG(LL, 1, SP) E2F_AGG(LL, 2, SP) E2F_AGG(LL, 4, SP)
  E2F_AGG_L(0, false)
  E2F_AGG_L(1, false)
  E2F_AGG_L(2, false)
  E2F_AGG_L(3, false)
  E2F_AGG_L(4, true)
  E2F_AGG_L(5, true)
  E2F_AGG_L(6, true)
#undef E2F_AGG_L
#undef E2F_AGG
  return hipErrorInvalidValue;
}

}  // namespace e2f
