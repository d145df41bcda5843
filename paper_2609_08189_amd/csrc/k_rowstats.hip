// Row pass over the post-attention states of a routed layer.
//
// For every token t (one workgroup per token row, HBM-streaming):
//   inv_rms = 1 / sqrt(mean(hbar^2) + eps_norm)            RMSNorm of the FFN input and of
//                                                           the router's hidden encoder
//                                                           (Sec. 3.1 eq:dense_attention, Sec. 3.2)
//   |delta_j|^2, <delta_j, delta_{j-1}>, |delta_{j-1}|^2    residual transitions
//     with delta_j = hbar_j - hbar_{j-1}                     (Sec. 3.2, eq:transition_features)
//   u = bf16/fp32(hbar * inv_rms * w)                        the FFN / adapter input
// The transition sums are only formed where the paper defines them (j >= 2, j >= 3).
#include "hero_device.h"
#include "hero_kernels.h"
#include "hero_rows.h"

namespace hero {

template <typename T>
__global__ __launch_bounds__(256) void rowstats_row_kernel(const T* __restrict__ hbar, const T* __restrict__ prev1,
                                                           const T* __restrict__ prev2, const T* __restrict__ norm_w,
                                                           int d, int j, float eps_norm, float* __restrict__ rowstat,
                                                           T* __restrict__ u) {
  rowstats_row<T>(static_cast<int>(blockIdx.x), static_cast<int>(gridDim.x), hbar, prev1, prev2, norm_w, d, j, eps_norm,
                  rowstat, u);
}

// ---------------------------------------------------------------------------
// The head of a decode step's layer (at most 256 tokens, bf16): the router's pre-activation
// product P = hbar [W_hd; psi_1]^T and the row pass read the same rows and nothing of each other,
// so one launch holds both.  The product streams 4 MiB of weights for few rows: up to 64 tokens
// here, workgroups of 16 columns x one of the kHeadSplits K-slices, then one workgroup per two token
// rows (beyond, the 64 x 128 tiles of launch_router_gemm, whose fragments go through LDS).  Waves
// are four blocks of 16 tokens by two halves of the K-slice, added through LDS; the fragments come
// straight from memory, BS k-steps of 32 in one batch.  One 8B layer at 1 token: 10.4 us for the
// tiles, the row pass beside them on a second stream, -> 4.5 us for both.
// ---------------------------------------------------------------------------
namespace {
constexpr int kHeadTokens = 64, kHeadSplits = 4, kHeadBatch = 16;

__global__ __launch_bounds__(512) void decode_head_kernel(const bf16_t* __restrict__ hbar,
                                                          const bf16_t* __restrict__ prev1,
                                                          const bf16_t* __restrict__ prev2,
                                                          const bf16_t* __restrict__ norm_w,
                                                          const bf16_t* __restrict__ w_hd,
                                                          const bf16_t* __restrict__ ps1, int T, int d, int d_e, int N,
                                                          int j, float eps_norm, float* __restrict__ P,
                                                          float* __restrict__ rowstat, bf16_t* __restrict__ u) {
  constexpr int BS = kHeadBatch;
  const int ncb = N / 16, ng = ncb * kHeadSplits;
  const int b = static_cast<int>(blockIdx.x);
  if (b >= ng) {
    rowstats_row<bf16_t, 2>(2 * (b - ng), T, hbar, prev1, prev2, norm_w, d, j, eps_norm, rowstat, u);
    return;
  }
  __shared__ f32x4 red[4][kWave];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) >> 6);
  const int rg = wave & 3, half = wave >> 2;
  const int cb = b % ncb, sl = b / ncb;
  const int kn = d / kHeadSplits / 2, k0 = sl * (d / kHeadSplits) + half * kn;
  const int kq = 8 * (lane >> 4), n = 16 * cb + (lane & 15);
  const bf16_t* brow = (n < d_e ? w_hd + static_cast<size_t>(n) * d : ps1 + static_cast<size_t>(n - d_e) * d) + k0 + kq;
  const bf16_t* arow = hbar + static_cast<size_t>(min(16 * rg + (lane & 15), T - 1)) * d + k0 + kq;
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  if (16 * rg < T)
    for (int kb = 0; kb < kn; kb += 32 * BS) {
      // steps past the slice load its last one again and are not used
      bf16x8 fb[BS], fa[BS];
#pragma unroll
      for (int i = 0; i < BS; ++i) {
        const int k = min(kb + 32 * i, kn - 32);
        fb[i] = *reinterpret_cast<const bf16x8*>(brow + k);
        fa[i] = *reinterpret_cast<const bf16x8*>(arow + k);
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = 0; i < BS; ++i)
        if (kb + 32 * i < kn) acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[i], fb[i], acc, 0, 0, 0);
    }
  if (half == 1) red[rg][lane] = acc;
  __syncthreads();
  if (half == 1) return;
  acc += red[rg][lane];
  float* out = P + static_cast<size_t>(sl) * T * N + n;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int t = 16 * rg + 4 * (lane >> 4) + r;
    if (t < T) out[static_cast<size_t>(t) * N] = acc[r];
  }
}
}  // namespace

bool decode_head_fits(int dtype, int T) { return dtype == 1 && T <= kDecodeTokens; }

hipError_t launch_decode_head(const void* hbar, const void* prev1, const void* prev2, const void* norm_w,
                              const void* w_hd, const void* ps1, int T, int d, int d_e, int d_head, int j,
                              float eps_norm, float* P, float* rowstat, void* u, hipStream_t s) {
  if (T <= 0) return hipSuccess;
  const int N = d_e + d_head;
  // what every bf16 model has (the argument checks of the calls)
  if (d % (64 * kHeadSplits) || d_e % 16 || N % 128 || router_gemm_splits(1, d, T, N) != kHeadSplits)
    return hipErrorInvalidValue;
  if (T > kHeadTokens)
    return launch_decode_head_tiles(hbar, prev1, prev2, norm_w, w_hd, ps1, T, d, d_e, d_head, j, eps_norm, P, rowstat,
                                    u, s);
  decode_head_kernel<<<N / 16 * kHeadSplits + (T + 1) / 2, 512, 0, s>>>(
      static_cast<const bf16_t*>(hbar), static_cast<const bf16_t*>(prev1), static_cast<const bf16_t*>(prev2),
      static_cast<const bf16_t*>(norm_w), static_cast<const bf16_t*>(w_hd), static_cast<const bf16_t*>(ps1), T, d, d_e,
      N, j, eps_norm, P, rowstat, static_cast<bf16_t*>(u));
  return hipGetLastError();
}

hipError_t launch_rowstats(int dtype, const void* hbar, const void* prev1, const void* prev2,
                           const void* norm_w, int T, int d, int j, float eps_norm,
                           float* rowstat, void* u, hipStream_t s) {
  if (T <= 0) return hipSuccess;
  if (dtype == 1)
    rowstats_row_kernel<bf16_t><<<T, 256, 0, s>>>(
        static_cast<const bf16_t*>(hbar), static_cast<const bf16_t*>(prev1), static_cast<const bf16_t*>(prev2),
        static_cast<const bf16_t*>(norm_w), d, j, eps_norm, rowstat, static_cast<bf16_t*>(u));
  else
    rowstats_row_kernel<float><<<T, 256, 0, s>>>(
        static_cast<const float*>(hbar), static_cast<const float*>(prev1), static_cast<const float*>(prev2),
        static_cast<const float*>(norm_w), d, j, eps_norm, rowstat, static_cast<float*>(u));
  return hipGetLastError();
}

}  // namespace hero
