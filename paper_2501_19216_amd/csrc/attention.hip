// Attention weights of the layer's edges (Alg. 1 takes them as input; App. E
// computes them from the scalar features and a radial basis):
//   logit[(i,j)][h] = sum_t q[i][h][t] k[j][h][t] + sum_r w[h][r] exp(-((d - mu_r)/sigma)^2),
//   mu_r = r cutoff / (R - 1), sigma = cutoff / (R - 1), d = |r_i - r_j|,
//   alpha[(i,j)][h] = env(d) * softmax over the row of logit[.][h],
//   env(d) = (cos(pi d / cutoff) + 1) / 2 below the cutoff, 0 from it on.
// One wave per receiver row.  Distances, envelopes and radial functions belong
// to an edge, not to a head: the wave evaluates them a lane per edge, 64 edges
// at a time, into LDS.  Then lane l takes head l % Hp (Hp = H rounded up to a
// power of two) and every (64/Hp)-th edge, so a wave's accesses of alpha [E][H]
// and of a sender's k are contiguous and the per-head max and sum are
// xor-shuffle reductions over the lanes of one head (fixed order:
// deterministic).  With one head (Hp = 1) nothing is shared and a lane evaluates
// its own edge's in registers (20,000 atoms, 80 neighbours, R = 32, d_k = 4:
// through LDS 89 us, in registers 48).  The logits of rows up to 16 64/Hp edges (8 64 with one
// head) stay in registers; longer rows keep them in alpha between the passes.
#include <hip/hip_runtime.h>

#include "e2f_launch.h"

namespace e2f {
namespace {


// Orders the LDS accesses of a wave's lanes among each other: a fence over the
// wavefront (the wave barrier alone orders scheduling, not memory).
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

template <int HP>
__global__ __launch_bounds__(256) void k_attention(const float* __restrict__ pos, const float* __restrict__ q,
                                                   const float* __restrict__ kf, int n, int H, int dk,
                                                   const float* __restrict__ rbf_w, int R, float rc,
                                                   const int64_t* __restrict__ row_ptr,
                                                   const int32_t* __restrict__ col, float* __restrict__ alpha) {
  constexpr int EPI = 64 / HP;           // edges per wave iteration
  constexpr int ITER = HP == 1 ? 8 : 16;  // iterations whose logits stay in registers
  extern __shared__ float sm[];
  const int i = blockIdx.x * 4 + (int)(threadIdx.x >> 6);
  if (i >= n) return;  // uniform over the wave (no barrier below)
  const int lane = threadIdx.x & 63;
  // the wave's 64 rows: radial functions (zeros up to a multiple of 8), envelope,
  // sender (odd stride)
  const int Rp = (R + 7) & ~7, ld = (Rp + 2) | 1;
  float* rows = sm + (threadIdx.x >> 6) * 64 * ld;
  const int h = lane % HP, el = lane / HP;
  const bool hv = h < H;
  const int hc = hv ? h : 0;
  const int64_t e0 = row_ptr[i], e1 = row_ptr[i + 1];
  if (e0 == e1) return;
  float w[HP == 1 ? 1 : kAttnMaxRbf];  // (one head: read where they are used, by every lane alike)
#pragma unroll
  for (int r = 0; r < (HP == 1 ? 0 : kAttnMaxRbf); ++r) w[r] = r < R ? rbf_w[hc * R + r] : 0.0f;
  const float sigma = rc / (float)(R - 1), inv = 1.0f / sigma;
  const float xi = pos[3 * i], yi = pos[3 * i + 1], zi = pos[3 * i + 2];
  const float* qi = q + ((size_t)i * H + hc) * dk;
  // q of this lane's head in registers, as float4 (d_k a multiple of 4, up to 64)
  const bool vec = (dk & 3) == 0 && dk <= 64;
  float4 q4[16];
#pragma unroll
  for (int t = 0; t < 16; ++t)
    q4[t] = (vec && 4 * t < dk) ? ((const float4*)qi)[t] : make_float4(0.f, 0.f, 0.f, 0.f);
  const float kPi = 3.14159265358979f;
  auto distance = [&](int j) {
    const float dx = xi - pos[3 * j], dy = yi - pos[3 * j + 1], dz = zi - pos[3 * j + 2];
    return sqrtf(dx * dx + dy * dy + dz * dz);
  };
  auto envelope = [&](float d) { return d < rc ? 0.5f * (cosf(kPi * d / rc) + 1.0f) : 0.0f; };
  auto radial = [&](float d, int r) {
    const float z = (d - (float)r * sigma) * inv;
    return expf(-z * z);
  };
  // the rows of the 64 edges from c on (radial functions four at a time, read
  // eight at a time below: one by one each waits for its latency; 20,000 atoms, 80
  // neighbours, 8 heads, d_k = 8, R = 8 149 -> 104 us, 300 atoms, 16 neighbours, R =
  // 32 11.0 -> 9.4)
  auto fill = [&](int64_t c) {
    wave_sync();  // (the rows before have been read)
    const int64_t e = c + lane;
    if (e < e1) {
      const int j = col[e];
      const float d = distance(j);
      float* o = rows + lane * ld;
      for (int r = 0; r < R; r += 4) {
        float v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = radial(d, r + u);
#pragma unroll
        for (int u = 0; u < 4; ++u)
          o[r + u] = r + u < R ? v[u] : 0.0f;
      }
      if (R <= Rp - 4)
        for (int u = 0; u < 4; ++u) o[Rp - 4 + u] = 0.0f;
      o[Rp] = envelope(d);
      o[Rp + 1] = __int_as_float(j);
    }
    wave_sync();
  };
  auto dot = [&](int j) {
    const float* kj = kf + ((size_t)j * H + hc) * dk;
    float l = 0.0f;
    if (vec) {
#pragma unroll
      for (int t = 0; t < 16; ++t) {
        if (4 * t < dk) {
          const float4 kv = ((const float4*)kj)[t];
          l += q4[t].x * kv.x + q4[t].y * kv.y + q4[t].z * kv.z + q4[t].w * kv.w;
        }
      }
    } else {
      for (int t = 0; t < dk; ++t) l += qi[t] * kj[t];
    }
    return l;
  };
  // logit and envelope of edge e, whose row (more than one head) is o
  auto logit = [&](int64_t e, const float* o, float& env) {
    if constexpr (HP == 1) {
      const int j = col[e];
      const float d = distance(j);
      float l = dot(j);
#pragma unroll 4
      for (int r = 0; r < R; ++r) l += rbf_w[r] * radial(d, r);
      env = envelope(d);
      return l;
    }
    float l = dot(__float_as_int(o[Rp + 1]));
#pragma unroll
    for (int r = 0; r < kAttnMaxRbf; r += 8)  // (eight reads in flight together)
      if (r < R) {
        float v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = o[r + u];
#pragma unroll
        for (int u = 0; u < 8; ++u) l += w[HP == 1 ? 0 : r + u] * v[u];
      }
    env = o[Rp];
    return l;
  };
  float mx = -INFINITY, den = 0.0f;
  if (e1 - e0 <= ITER * EPI) {
    float l[ITER], env[ITER];
    const int deg = (int)(e1 - e0);
#pragma unroll
    for (int it = 0; it < ITER; ++it) {
      l[it] = -INFINITY, env[it] = 0.0f;
      if (it * EPI >= deg) continue;  // uniform
      if (HP > 1 && it % HP == 0) fill(e0 + it * EPI);
      const float* o = rows + (it % HP * EPI + el) * ld;
      if (it * EPI + el < deg) l[it] = logit(e0 + it * EPI + el, o, env[it]);
      mx = fmaxf(mx, l[it]);
    }
#pragma unroll
    for (int o = 32; o >= HP; o >>= 1) mx = fmaxf(mx, __shfl_xor(mx, o));
#pragma unroll
    for (int it = 0; it < ITER; ++it) {
      if (it * EPI >= deg) continue;
      l[it] = it * EPI + el < deg ? expf(l[it] - mx) : 0.0f;
      den += l[it];
    }
#pragma unroll
    for (int o = 32; o >= HP; o >>= 1) den += __shfl_xor(den, o);
    const float rden = 1.0f / den;
#pragma unroll
    for (int it = 0; it < ITER; ++it)
      if (it * EPI + el < deg && hv) alpha[(e0 + it * EPI + el) * H + h] = env[it] * l[it] * rden;
    return;
  }
  // pass 1: logits, kept in the output; pass 2: exponentials; pass 3: scale
  for (int64_t c = e0; c < e1; c += 64) {
    if (HP > 1) fill(c);
    for (int64_t e = c + el; e < min(c + 64, e1); e += EPI) {
      float env;
      const float l = logit(e, rows + (e - c) * ld, env);
      if (hv) alpha[e * H + h] = l;
      mx = fmaxf(mx, l);
    }
  }
#pragma unroll
  for (int o = 32; o >= HP; o >>= 1) mx = fmaxf(mx, __shfl_xor(mx, o));
  for (int64_t e = e0 + el; e < e1; e += EPI) {
    if (!hv) continue;
    const float ex = expf(alpha[e * H + h] - mx);
    alpha[e * H + h] = ex;
    den += ex;
  }
#pragma unroll
  for (int o = 32; o >= HP; o >>= 1) den += __shfl_xor(den, o);
  const float rden = 1.0f / den;
  for (int64_t c = e0; c < e1; c += 64) {
    if (HP > 1) fill(c);
    for (int64_t e = c + el; e < min(c + 64, e1); e += EPI)
      if (hv)
        alpha[e * H + h] = (HP == 1 ? envelope(distance(col[e])) : rows[(e - c) * ld + Rp]) * alpha[e * H + h] * rden;
  }
}

}  // namespace

hipError_t launch_attention(const float* pos, const float* q, const float* k, int n, int H, int dk,
                            const float* rbf_w, int R, float rc, const int64_t* row_ptr, const int32_t* col_idx,
                            float* alpha, hipStream_t s) {
  if (n == 0) return hipSuccess;
  int hp = 1;
  while (hp < H) hp <<= 1;
  const unsigned grid = (unsigned)((n + 3) / 4);
  const size_t lds = hp == 1 ? 0 : sizeof(float) * 4 * 64 * ((((R + 7) & ~7) + 2) | 1);  // at most 35 KB
  switch (hp) {
#define E2F_ATT(P)                                                                                     \
  case P:                                                                                              \
    k_attention<P><<<grid, 256, lds, s>>>(pos, q, k, n, H, dk, rbf_w, R, rc, row_ptr, col_idx, alpha);   \
    break;
    E2F_ATT(1) E2F_ATT(2) E2F_ATT(4) E2F_ATT(8) E2F_ATT(16) E2F_ATT(32) E2F_ATT(64)
#undef E2F_ATT
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace e2f
