// The row pass of one token (k_rowstats.hip), also run beside the router's product of a decode step.
#pragma once

#include "hero_device.h"

namespace hero {

// 256 threads per token, its row split over their four waves (8 elements per lane per pass, up to
// 8192 elements kept in registers for the normalisation), the four sums reduced across the waves
// through LDS.  Measured against four tokens per workgroup (one per wave): 26.8 against 28.4 us at
// 4096 tokens of d = 4096, 7.2 against 13.6 us at 256 tokens, where a wave per row left most CUs idle.
// A workgroup of 256 G threads takes the G tokens from t on (past the last of T: the last again,
// nothing stored); the threads of a token and so the order of its sums are the same for every G.
// Two tokens a workgroup are a decode step's few, a chain of latencies: the gain is loaded beside the
// row instead of after the sums (8B layer at 1 token 85.8 -> 85.1 us, level from 32 tokens on).
template <typename T, int G = 1>
__device__ __forceinline__ void rowstats_row(int t, int T_rows, const T* __restrict__ hbar, const T* __restrict__ prev1,
                                             const T* __restrict__ prev2, const T* __restrict__ norm_w, int d, int j,
                                             float eps_norm, float* __restrict__ rowstat, T* __restrict__ u) {
  constexpr int NT = 256;
  constexpr bool AHEAD = G == 2;
  __shared__ f32x4 parts[G][NT / 64];
  const int grp = G == 1 ? 0 : static_cast<int>(threadIdx.x) / NT;
  const bool own = t + grp < T_rows;
  t = min(t + grp, T_rows - 1);
  f32x4* part = parts[grp];
  const int tid = G == 1 ? threadIdx.x : threadIdx.x % NT, lane = tid & 63, wave = tid >> 6;
  const size_t row = static_cast<size_t>(t) * d;
  constexpr int RC = 1024 / NT;   // 8-element chunks per thread kept in registers (rows up to 8192)
  Raw8<T> h[RC], w[RC];
  float ss = 0.f, dd = 0.f, dp = 0.f, pp = 0.f;
  const bool resident = d <= RC * 8 * NT;
  for (int c0 = 0; c0 < d; c0 += RC * 8 * NT) {
    Raw8<T> a[RC], b[RC];
#pragma unroll
    for (int c = 0; c < RC; ++c) {
      const int col = c0 + 8 * (tid + NT * c);
      if (col < d) {
        h[c].load(hbar + row + col);
        if (j >= 2) a[c].load(prev1 + row + col);
        if (j >= 3) b[c].load(prev2 + row + col);
        if (AHEAD && resident) w[c].load(norm_w + col);
      }
    }
#pragma unroll
    for (int c = 0; c < RC; ++c) {
      const int col = c0 + 8 * (tid + NT * c);
      if (col >= d) continue;
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const float hv = h[c][i];
        ss += hv * hv;
        if (j >= 2) {
          const float av = a[c][i];
          const float dj = hv - av;
          dd += dj * dj;
          if (j >= 3) {
            const float dq = av - b[c][i];
            dp += dj * dq;
            pp += dq * dq;
          }
        }
      }
    }
  }
  ss = wave_sum(ss);
  dd = wave_sum(dd);
  dp = wave_sum(dp);
  pp = wave_sum(pp);
  if (lane == 0) part[wave] = f32x4{ss, dd, dp, pp};
  __syncthreads();
  f32x4 tot = part[0];
#pragma unroll
  for (int w = 1; w < NT / 64; ++w) tot += part[w];
  const float inv_rms = 1.0f / sqrtf(tot[0] / static_cast<float>(d) + eps_norm);
  if (!own) return;
  if (tid == 0) {
    f32x4 r = {inv_rms, tot[1], tot[2], tot[3]};
    *reinterpret_cast<f32x4*>(rowstat + 4 * static_cast<size_t>(t)) = r;
  }
  for (int c0 = 0; c0 < d; c0 += RC * 8 * NT) {
#pragma unroll
    for (int c = 0; c < RC; ++c) {
      const int col = c0 + 8 * (tid + NT * c);
      if (col >= d) continue;
      if (!resident) h[c].load(hbar + row + col);
      if (!AHEAD || !resident) w[c].load(norm_w + col);
      float o[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) o[i] = h[c][i] * inv_rms * w[c][i];
      st8(u + row + col, o);
    }
  }
}

}  // namespace hero
