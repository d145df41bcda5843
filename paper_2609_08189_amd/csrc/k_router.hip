// Router of one routed layer after the two large projections (Sec. 3.2), as three kernels (calls
// of few tokens run them as one, router_token):
//
//   router_pre   (8 tokens per workgroup, reuses each weight across them)
//     z^h = W_hu SiLU(inv_rms * W_hd hbar)                       hidden encoder (unit-gain RMSNorm)
//     x^path = [j/L_R, (L_R-j)/L_R, |delta_j|, gamma_j, p_{j-1}, m_{j-1}]   (eq:path_vector,
//                                                                 eq:transition_features)
//     z^a = W_p2 SiLU(W_p1 x^path),  s = [z^h; z^a]              (eq:router_state)
//     phi(q), phi(k), v, W_n s;  th1[:, :d_s] s (the s part of the history head's input layer)
//     b = ps2 . SiLU(psi_1 hbar)                                  local head (eq:final_gate)
//   router_mem   (one token per workgroup: a streaming read-modify-write of the memory)
//     c = phi(q)^T S / (phi(q)^T zeta + eps)                      (eq:memory_read, read first)
//     S <- rho S + phi(k) v^T,  zeta <- rho zeta + phi(k)          (eq:memory_update, same pass)
//   router_post  (8 tokens per workgroup)
//     nu = 1 - cos(W_n s, W_c c)  (0 at j = 1)
//     a = th2 . SiLU(th1 [s; c; nu]),  p = sigma(a / T_hist),  m = m_{j-1} p
//     logit = a + b (+ bias),  g = sigma(logit)
// At j = 1 the incoming state is the paper's initial value: S and zeta are not read
// (taken as zero) and p_0 = m_0 = 1.
// Router ablations (Table 3): without the position state the first four path features are
// zero; without the auxiliary state z^a = 0; without the memory read (or the whole history
// branch) router_mem is not launched, c = 0 and nu = 0 at every layer; without the history
// branch a = 0, so logit = b (+ bias), and p = m = 1 are written.
// The memory kernel moves 2 * 4 * (d_m^2 + d_m) bytes of state per token (2 * (2 d_m^2 + 4 d_m)
// with S stored in bf16) and is the HBM-bound part; keeping it free of the matrix-vector work lets many workgroups per
// CU keep HBM busy.  All arithmetic is fp32.
#include <algorithm>
#include <type_traits>

#include "hero_device.h"
#include "hero_kernels.h"

namespace hero {
namespace {

constexpr int TB = 16;    // tokens per workgroup (pre / post)
constexpr int NT = 256;   // threads per workgroup
constexpr int MAXE = 256; // max(d_e, d_head)
constexpr int KC = 32;    // weight columns staged per step of block_matmul
constexpr int MAXS = 128; // max d_s
constexpr int MAXP = 128; // max d_p
constexpr int MAXM = 256; // max d_m

struct Ident {
  __device__ __forceinline__ float operator()(float x) const { return x; }
};
struct SiLU {
  __device__ __forceinline__ float operator()(float x) const { return siluf_(x); }
};
struct Phi {
  __device__ __forceinline__ float operator()(float x) const { return phif_(x); }
};

// out[t*os + o] = act(sum_i W[o*ldw + i] * in[t*is + i]) for o < O and tokens t < nvalid.
// P lanes share one output row (power of two, within a wave) and reduce by shuffles;
// each lane takes 8 consecutive inputs per step, loaded as one 16-byte vector when
// the row pitch allows it and as 8 independent loads otherwise.
template <typename W, class Act>
__device__ __forceinline__ void matvec(const W* __restrict__ w, int ldw, int O, int I,
                                       const float* in, int is, float* out, int os, Act act,
                                       int nvalid = TB) {
  int P = 64;
  while (P > 1 && P * O > NT) P >>= 1;
  while (P > 1 && 8 * (P >> 1) >= I) P >>= 1;   // no lane without work
  const int rows_per_pass = NT / P;
  const int slice = threadIdx.x % P;
  const bool vec = (ldw % 8 == 0) && ((reinterpret_cast<uintptr_t>(w) & 15) == 0);
  for (int o0 = 0; o0 < O; o0 += rows_per_pass) {
    const int o = o0 + static_cast<int>(threadIdx.x) / P;
    float acc[TB];
#pragma unroll
    for (int t = 0; t < TB; ++t) acc[t] = 0.f;
    if (o < O) {
      const W* wr = w + static_cast<size_t>(o) * ldw;
      for (int i = 8 * slice; i < I; i += 8 * P) {
        float wv[8];
        if (vec && i + 8 <= I) {
          ld8(wr + i, wv);
        } else {
#pragma unroll
          for (int e = 0; e < 8; ++e) wv[e] = (i + e < I) ? ldf(wr + i + e) : 0.f;
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          if (i + e < I) {
#pragma unroll
            for (int t = 0; t < TB; ++t) acc[t] = fmaf(wv[e], in[t * is + i + e], acc[t]);
          }
        }
      }
    }
    for (int off = P >> 1; off > 0; off >>= 1)
#pragma unroll
      for (int t = 0; t < TB; ++t) acc[t] += __shfl_xor(acc[t], off, kWave);
    if (o < O && slice == 0)
#pragma unroll
      for (int t = 0; t < TB; ++t)
        if (t < nvalid) out[t * os + o] = act(acc[t]);
  }
}

// out[t*os + o] = act(bias[t*bs + o] + sum_i W[o*ldw + i] * X[t*ldx + i]) for o < O (<= 256) and
// tokens t < nvalid, all TB tokens computed.  Weight columns are staged KC at a time into LDS,
// transposed to [k][o] and converted to fp32, with loads that are contiguous along each
// row; each thread then accumulates a tile of RO rows x 4 tokens, reading one RO-wide weight
// vector and four broadcast inputs per k.
template <int RO, typename W, class Act>
__device__ __forceinline__ void block_matmul_ro(const W* __restrict__ w, int ldw, int O, int I,
                                                const float* X, int ldx, const float* bias, int bs,
                                                float* out, int os, Act act, float* wst, int nvalid) {
  constexpr int OPAD = 4 * 64 + 4;   // staged row pitch (floats)
  const int tid = threadIdx.x;
  const int og = tid >> 2, tg = tid & 3;   // rows og*RO.., tokens 4*tg..
  float acc[RO][4];
#pragma unroll
  for (int r = 0; r < RO; ++r)
#pragma unroll
    for (int q = 0; q < 4; ++q) acc[r][q] = 0.f;
  constexpr int U = 4 * 64 * KC / NT;   // staged elements per thread (rows <= 256)
  for (int i0 = 0; i0 < I; i0 += KC) {
    // all of this thread's loads are issued before any is used
    float tmp[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int e = tid + NT * u;
      const int o = e / KC, k = e % KC;
      tmp[u] = (o < O && i0 + k < I) ? ldf(w + static_cast<size_t>(o) * ldw + i0 + k) : 0.f;
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int e = tid + NT * u;
      const int o = e / KC, k = e % KC;
      if (o < O) wst[k * OPAD + o] = tmp[u];
    }
    __syncthreads();
    if (og * RO < O) {
      const int kn = min(KC, I - i0);
      for (int k = 0; k < kn; ++k) {
        float wv[RO];
#pragma unroll
        for (int r = 0; r < RO; ++r) wv[r] = wst[k * OPAD + og * RO + r];
        float xv[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) xv[q] = X[(4 * tg + q) * ldx + i0 + k];
#pragma unroll
        for (int r = 0; r < RO; ++r)
#pragma unroll
          for (int q = 0; q < 4; ++q) acc[r][q] = fmaf(wv[r], xv[q], acc[r][q]);
      }
    }
  }
  if (og * RO < O) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int t = 4 * tg + q;
      if (t >= nvalid) continue;
#pragma unroll
      for (int r = 0; r < RO; ++r) {
        const int o = og * RO + r;
        if (o < O) out[t * os + o] = act(acc[r][q] + (bias ? bias[t * bs + o] : 0.f));
      }
    }
  }
}

template <typename W, class Act>
__device__ __forceinline__ void block_matmul(const W* w, int ldw, int O, int I, const float* X, int ldx,
                                             const float* bias, int bs, float* out, int os, Act act,
                                             float* wst, int nvalid = TB) {
  if (O > 128)
    block_matmul_ro<4>(w, ldw, O, I, X, ldx, bias, bs, out, os, act, wst, nvalid);
  else if (O > 64)
    block_matmul_ro<2>(w, ldw, O, I, X, ldx, bias, bs, out, os, act, wst, nvalid);
  else
    block_matmul_ro<1>(w, ldw, O, I, X, ldx, bias, bs, out, os, act, wst, nvalid);
  __syncthreads();
}

// for (e = tid; e < n; e += NT) f(e, src(e)), with eight loads in flight per thread
template <class Src, class F>
__device__ __forceinline__ void batched(int n, Src src, F f) {
  for (int e0 = threadIdx.x; e0 < n; e0 += 8 * NT) {
    float v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int e = e0 + NT * u;
      v[u] = e < n ? src(e) : 0.f;
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int e = e0 + NT * u;
      if (e < n) f(e, v[u]);
    }
  }
}

#define LDS16 __shared__ __attribute__((aligned(16)))

// ---------------------------------------------------------------------------
// router_pre
// ---------------------------------------------------------------------------
template <typename W>
__global__ __launch_bounds__(NT) void router_pre_kernel(RouterTailArgs a) {
  constexpr int EP = MAXE + 4;
  LDS16 float bufA[TB][EP];     // SiLU(inv_rms W_hd hbar)
  LDS16 float bufB[TB][EP];     // SiLU(psi_1 hbar)
  LDS16 float s[TB][MAXS + 4];  // router state
  LDS16 float xp[TB][8];        // path vector
  LDS16 float zp[TB][MAXP];     // path-encoder hidden
  LDS16 float wst[KC * (4 * 64 + 4)];
  LDS16 float sc[TB];

  const int tid = threadIdx.x;
  const int t0 = blockIdx.x * TB;
  const int nvalid = min(TB, a.T - t0);
  const int j = a.j;
  const int d_e = a.d_e, d_head = a.d_head, NP = a.d_e + a.d_head, DM = a.d_m;

  if (tid < TB) {
    const int t = t0 + tid;
    float inv_rms = 0.f, dd = 0.f, dp = 0.f, pp = 0.f, pprev = 1.f, mprev = 1.f;
    if (t < a.T) {
      const f32x4 rs = *reinterpret_cast<const f32x4*>(a.rowstat + 4 * static_cast<size_t>(t));
      inv_rms = rs[0];
      dd = rs[1];
      dp = rs[2];
      pp = rs[3];
      if (j > 1) {
        pprev = a.p_hist[t];
        mprev = a.m_hist[t];
      }
    }
    const float dj = j >= 2 ? sqrtf(dd) : 0.f;
    const float gam = j >= 3 ? dp / (dj * sqrtf(pp) + a.eps) : 0.f;
    const bool pos = !(a.abl & ABL_NO_POS);
    xp[tid][0] = pos ? static_cast<float>(j) / static_cast<float>(a.L_R) : 0.f;
    xp[tid][1] = pos ? static_cast<float>(a.L_R - j) / static_cast<float>(a.L_R) : 0.f;
    xp[tid][2] = pos ? dj : 0.f;
    xp[tid][3] = pos ? gam : 0.f;
    xp[tid][4] = pprev;
    xp[tid][5] = mprev;
    sc[tid] = inv_rms;
  }
  __syncthreads();
  batched(
      TB * NP,
      [&](int e) { return a.P[static_cast<size_t>(min(t0 + e / NP, a.T - 1)) * NP + e % NP]; },
      [&](int e, float pv) {
        const int tt = e / NP, i = e % NP;
        if (i < d_e)
          bufA[tt][i] = siluf_(sc[tt] * pv);
        else
          bufB[tt][i - d_e] = siluf_(pv);
      });
  __syncthreads();
  block_matmul(static_cast<const W*>(a.w_hu), d_e, a.d_h, d_e, &bufA[0][0], EP, nullptr, 0, &s[0][0],
               MAXS + 4, Ident(), wst);
  matvec(static_cast<const W*>(a.w_p1), 6, a.d_p, 6, &xp[0][0], 8, &zp[0][0], MAXP, SiLU());
  matvec(static_cast<const W*>(a.ps2), d_head, 1, d_head, &bufB[0][0], EP, a.bvec + t0, 1, Ident(),
         nvalid);
  __syncthreads();
  if (a.abl & ABL_NO_AUX) {
    for (int e = tid; e < TB * a.d_a; e += NT) s[e / a.d_a][a.d_h + e % a.d_a] = 0.f;
  } else {
    matvec(static_cast<const W*>(a.w_p2), a.d_p, a.d_a, a.d_p, &zp[0][0], MAXP, &s[0][a.d_h], MAXS + 4,
           Ident());
  }
  __syncthreads();
  const int d_s = a.d_s;
  float* qkvn = a.qkvn + static_cast<size_t>(t0) * 4 * DM;
  const float* S0 = &s[0][0];
  block_matmul(static_cast<const W*>(a.w_q), d_s, DM, d_s, S0, MAXS + 4, nullptr, 0, qkvn, 4 * DM, Phi(),
               wst, nvalid);
  block_matmul(static_cast<const W*>(a.w_k), d_s, DM, d_s, S0, MAXS + 4, nullptr, 0, qkvn + DM, 4 * DM,
               Phi(), wst, nvalid);
  block_matmul(static_cast<const W*>(a.w_v), d_s, DM, d_s, S0, MAXS + 4, nullptr, 0, qkvn + 2 * DM, 4 * DM,
               Ident(), wst, nvalid);
  block_matmul(static_cast<const W*>(a.w_n), d_s, DM, d_s, S0, MAXS + 4, nullptr, 0, qkvn + 3 * DM, 4 * DM,
               Ident(), wst, nvalid);
  // the s columns of the history head's input layer
  block_matmul(static_cast<const W*>(a.th1), a.ld_th1, d_head, d_s, S0, MAXS + 4, nullptr, 0,
               a.hs + static_cast<size_t>(t0) * d_head, d_head, Ident(), wst, nvalid);
}

// ---------------------------------------------------------------------------
// router_mem: one token per workgroup
// ---------------------------------------------------------------------------
// 16 bytes of the state as fp32 values: four fp32, or eight bf16
template <typename ST>
struct SVec {
  static constexpr int N = 16 / static_cast<int>(sizeof(ST));
  float v[N];
  __device__ __forceinline__ void load(const ST* p) {
    if constexpr (sizeof(ST) == 4) {
      const f32x4 x = *reinterpret_cast<const f32x4*>(p);
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = x[e];
    } else {
      const u32x4 x = *reinterpret_cast<const u32x4*>(p);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        v[2 * e] = __uint_as_float(x[e] << 16);
        v[2 * e + 1] = __uint_as_float(x[e] & 0xffff0000u);
      }
    }
  }
  __device__ __forceinline__ void store(ST* p) const {
    if constexpr (sizeof(ST) == 4) {
      f32x4 x;
#pragma unroll
      for (int e = 0; e < 4; ++e) x[e] = v[e];
      *reinterpret_cast<f32x4*>(p) = x;
    } else {
      u32x4 x;
#pragma unroll
      for (int e = 0; e < 4; ++e)
        x[e] = static_cast<uint32_t>(f32_to_bf16(v[2 * e])) |
               (static_cast<uint32_t>(f32_to_bf16(v[2 * e + 1])) << 16);
      *reinterpret_cast<u32x4*>(p) = x;
    }
  }
};

// ST: storage type of S (float, or bf16_t: every written element rounded to nearest even)
template <int DM, typename ST>
__global__ __launch_bounds__(NT) void router_mem_kernel(RouterTailArgs a) {
  constexpr int VE = SVec<ST>::N;  // state elements per 16-byte vector
  constexpr int CV = DM / VE;      // vectors per S row
  constexpr int RP = NT / CV;      // S rows per pass
  constexpr int NR = DM / RP;      // S rows per thread
  static_assert(NR >= 1 && NT % CV == 0, "state layout");
  LDS16 float fq[DM];
  LDS16 float fk[DM];
  LDS16 float vv[DM];
  LDS16 float red[RP][DM];
  __shared__ float sden;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int t = blockIdx.x;
  const int j = a.j;
  const float rho = 1.0f / (1.0f + expf(-a.eta));
  const float* q = a.qkvn + static_cast<size_t>(t) * 4 * DM;
  for (int i = tid; i < 3 * DM; i += NT) {
    const float x = q[i];
    if (i < DM)
      fq[i] = x;
    else if (i < 2 * DM)
      fk[i - DM] = x;
    else
      vv[i - 2 * DM] = x;
  }
  __syncthreads();
  if (wave == 0) {
    float part = 0.f;
    float* z = a.zeta + static_cast<size_t>(t) * DM;
    for (int k = lane; k < DM; k += 64) {
      const float zv = j > 1 ? z[k] : 0.f;
      part = fmaf(fq[k], zv, part);
      z[k] = fmaf(rho, zv, fk[k]);
    }
    part = wave_sum(part);
    if (lane == 0) sden = part;
  }
  const int cq = tid % CV, rg = tid / CV;
  ST* Sp = static_cast<ST*>(a.S) + static_cast<size_t>(t) * DM * DM + VE * cq;
  float vr[VE], cacc[VE];
#pragma unroll
  for (int e = 0; e < VE; ++e) {
    vr[e] = vv[VE * cq + e];
    cacc[e] = 0.f;
  }
  if (j == 1) {
#pragma unroll 16
    for (int i = 0; i < NR; ++i) {
      const int r = rg + RP * i;
      SVec<ST> o;
#pragma unroll
      for (int e = 0; e < VE; ++e) o.v[e] = fk[r] * vr[e];
      o.store(Sp + r * DM);
    }
  } else {
    constexpr int CH = NR < 16 ? NR : 16;
    for (int i0 = 0; i0 < NR; i0 += CH) {
      SVec<ST> sv[CH];
#pragma unroll
      for (int c = 0; c < CH; ++c) sv[c].load(Sp + (rg + RP * (i0 + c)) * DM);
#pragma unroll
      for (int c = 0; c < CH; ++c) {
        const int r = rg + RP * (i0 + c);
        const float qv = fq[r], kv = fk[r];
        SVec<ST> o;
#pragma unroll
        for (int e = 0; e < VE; ++e) {
          cacc[e] = fmaf(qv, sv[c].v[e], cacc[e]);
          o.v[e] = fmaf(rho, sv[c].v[e], kv * vr[e]);
        }
        o.store(Sp + r * DM);
      }
    }
  }
#pragma unroll
  for (int e = 0; e < VE; ++e) red[rg][VE * cq + e] = cacc[e];
  __syncthreads();
  if (tid < DM) {
    float cs = 0.f;
    for (int g = 0; g < RP; ++g) cs += red[g][tid];
    a.cvec[static_cast<size_t>(t) * DM + tid] = j > 1 ? cs / (sden + a.eps) : 0.f;
  }
}

// ---------------------------------------------------------------------------
// router_post
// ---------------------------------------------------------------------------
template <typename W>
__global__ __launch_bounds__(NT) void router_post_kernel(RouterTailArgs a) {
  constexpr int CX = MAXM + 4;
  constexpr int HP = MAXE + 4;
  LDS16 float cx[TB][CX];         // [c; nu]
  LDS16 float ns[TB][MAXM];       // W_n s
  LDS16 float wc[TB][MAXM];       // W_c c
  LDS16 float hh[TB][HP];         // s part of the f_theta pre-activation, then its hidden
  LDS16 float wst[KC * (4 * 64 + 4)];
  LDS16 float sc[TB];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int t0 = blockIdx.x * TB;
  const int nvalid = min(TB, a.T - t0);
  const int j = a.j;
  const int DM = a.d_m, d_head = a.d_head, d_s = a.d_s;
  auto tok = [&](int tt) { return static_cast<size_t>(min(t0 + tt, a.T - 1)); };
  // a memory context exists after the first layer unless an ablation removes the memory
  const bool ctx = j > 1 && !(a.abl & (ABL_NO_MEMREAD | ABL_NO_HISTORY));
  batched(
      TB * DM, [&](int e) { return ctx ? a.cvec[tok(e / DM) * DM + e % DM] : 0.f; },
      [&](int e, float v) { cx[e / DM][e % DM] = v; });
  batched(
      TB * DM, [&](int e) { return a.qkvn[tok(e / DM) * 4 * DM + 3 * DM + e % DM]; },
      [&](int e, float v) { ns[e / DM][e % DM] = v; });
  batched(
      TB * d_head, [&](int e) { return a.hs[tok(e / d_head) * d_head + e % d_head]; },
      [&](int e, float v) { hh[e / d_head][e % d_head] = v; });
  __syncthreads();
  block_matmul(static_cast<const W*>(a.w_c), DM, DM, DM, &cx[0][0], CX, nullptr, 0, &wc[0][0], MAXM,
               Ident(), wst);
  for (int tt = wave; tt < TB; tt += NT / 64) {
    float nn = 0.f, cc = 0.f, nc = 0.f;
    for (int k = lane; k < DM; k += 64) {
      const float n = ns[tt][k], c = wc[tt][k];
      nn = fmaf(n, n, nn);
      cc = fmaf(c, c, cc);
      nc = fmaf(n, c, nc);
    }
    nn = wave_sum(nn);
    cc = wave_sum(cc);
    nc = wave_sum(nc);
    if (lane == 0) cx[tt][DM] = ctx ? 1.0f - nc / (sqrtf(nn) * sqrtf(cc) + a.eps) : 0.f;
  }
  __syncthreads();
  // the [c; nu] columns of the history head's input layer on top of its s part, then SiLU
  block_matmul(static_cast<const W*>(a.th1) + d_s, a.ld_th1, d_head, DM + 1, &cx[0][0], CX, &hh[0][0], HP,
               &hh[0][0], HP, SiLU(), wst);
  matvec(static_cast<const W*>(a.th2), d_head, 1, d_head, &hh[0][0], HP, &sc[0], 1, Ident());
  __syncthreads();
  if (tid < nvalid) {
    const int t = t0 + tid;
    const bool hist = !(a.abl & ABL_NO_HISTORY);
    const float av = hist ? sc[tid] : 0.f;
    const float mprev = j > 1 ? a.m_hist[t] : 1.0f;
    const float p = sigmoidf_(av / a.T_hist);
    a.p_hist[t] = hist ? p : 1.0f;
    a.m_hist[t] = hist ? mprev * p : 1.0f;
    const float l = av + a.bvec[t] + (a.beta ? a.beta[t] : 0.f);
    a.logit[t] = l;
    a.gate[t] = sigmoidf_(l);
  }
}


// ---------------------------------------------------------------------------
// bf16 weights: matrix cores.  Every product above is a contraction over a batch of
// tokens, run here on v_mfma_f32_16x16x32_bf16 with one 16-token row block per
// workgroup.  The fp32 activations are split as x = hi + lo into two bf16 values
// (|x - hi - lo| <= 2^-18 |x|) and the bf16 weights are exact, so each product
// hi*w and lo*w is exact in fp32 and only the fp32 accumulation rounds.
// A fragments live in LDS in MFMA order: entry [k-step s][lane], lane = i + 16 g,
// holds row i at k = 32 s + 8 g .. + 7.  B fragments are 16-byte loads of eight
// consecutive weights of one output row (L2-resident: every workgroup reads the
// same router weights).  Output lane i + 16 g holds rows 4 g .. 4 g + 3 of column i.
// ---------------------------------------------------------------------------
constexpr int MT = 16;            // tokens per workgroup
constexpr int MAXSPLIT = 4;       // K-slice partials of P
constexpr int KS_E = MAXE / 32;   // k-steps over d_e
constexpr int KS_S = MAXS / 32;   // k-steps over d_s
constexpr int KS_M = MAXM / 32;   // k-steps over d_m

__device__ __forceinline__ void split8(const float* x, bf16x8& hi, bf16x8& lo) {
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const __bf16 h = static_cast<__bf16>(x[e]);
    hi[e] = h;
    lo[e] = static_cast<__bf16>(x[e] - static_cast<float>(h));
  }
}

__device__ __forceinline__ f32x4 mfma_split(const bf16x8& ahi, const bf16x8& alo, const bf16x8& b,
                                            f32x4 acc) {
  acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ahi, b, acc, 0, 0, 0);
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(alo, b, acc, 0, 0, 0);
}

// Weights w[r][k0 + 8 g .. + 7] of row r = r0 + (lane & 15), g = lane >> 4, of a [nrows][ld]
// matrix (ld % 8 == 0, 16-byte aligned base); zero past nrows or past kmax (kmax % 8 == 0).
__device__ __forceinline__ bf16x8 bfrag(const bf16_t* __restrict__ w, int ld, int nrows, int r0,
                                        int k0, int kmax, int lane) {
  const int r = r0 + (lane & 15), k = k0 + 8 * (lane >> 4);
  u32x4 v = {0u, 0u, 0u, 0u};
  if (r < nrows && k < kmax) v = *reinterpret_cast<const u32x4*>(w + static_cast<size_t>(r) * ld + k);
  return __builtin_bit_cast(bf16x8, v);
}

// One 16-column output tile of the s-projections: which matrix, its row offset, destination.
struct SProj {
  const bf16_t* w;
  int ld, nrows, r0, os;
  float* out;
  bool phi;
};

// router_pre on 8 waves (16 tokens per workgroup).  Every global load of the kernel is issued
// first: the P partials, the hidden encoder's and the s-projections' weight fragments (up to
// PF2 output tiles per wave), the local head's weights and the path-vector inputs; what follows
// works from registers and LDS between four barriers.
constexpr int NTP = 512;
constexpr unsigned kCUsRouter = 256;   // compute units of an MI355X
constexpr int NWP = NTP / kWave;
constexpr int PF2 = 6;

// KSS: k-steps over d_s (ceil(d_s / 32)).  WPE: waves per SIMD the kernel is compiled for (2: one
// workgroup per CU with every weight fragment loaded up front, for launches of about one round of
// workgroups; 4: two workgroups per CU, each hiding the other's latencies, for many rounds)
// NSPL: the most K-slice partials of P the launch may have (p_splits <= NSPL); PF: output tiles
// of the s-projections per wave whose weight fragments are loaded up front
template <int KSS, int WPE = 2, int NSPL = MAXSPLIT, int PF = PF2>
__global__ __launch_bounds__(NTP, WPE) void router_pre_mfma(RouterTailArgs a) {
  LDS16 bf16x8 ax[2][KS_E][kWave];   // SiLU(inv_rms W_hd hbar): hi, lo
  LDS16 bf16x8 as[2][KS_S][kWave];   // s: hi, lo
  LDS16 float s[MT][MAXS + 4];
  LDS16 float hp[MT][MAXP + 1];      // path-encoder hidden
  __shared__ float xp[MT][8];
  __shared__ float sc[MT];
  __shared__ float bpart[MT][16];

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int t0 = blockIdx.x * MT;
  // column groups (few tokens): workgroup y of CS takes the output tiles ct = y + CS i of the
  // s-projections; every group forms s itself
  const int cs = blockIdx.y, CS = gridDim.y;
  const int nvalid = min(MT, a.T - t0);
  const int j = a.j;
  const int d_e = a.d_e, d_head = a.d_head, NP = d_e + d_head, DM = a.d_m, d_s = a.d_s;
  const int d_h = a.d_h, d_a = a.d_a, d_p = a.d_p;
  const int nq = DM / 16, nct = 4 * nq + d_head / 16;
  auto proj = [&](int ct) {
    const int m = ct / nq;
    if (m < 4) {
      const void* ws[4] = {a.w_q, a.w_k, a.w_v, a.w_n};
      return SProj{static_cast<const bf16_t*>(ws[m]), d_s, DM, 16 * (ct - m * nq), 4 * DM, a.qkvn + m * DM,
                   m < 2};
    }
    return SProj{static_cast<const bf16_t*>(a.th1), a.ld_th1, d_head, 16 * (ct - 4 * nq), d_head, a.hs, false};
  };

  // (1) P: token tt, columns [16 pc, 16 pc + 16) (NP <= 512), the K-slice partials
  const int tt = tid >> 5, pc = tid & 31;
  const bool has_p = 16 * pc < NP;
  const bool head = has_p && 16 * pc >= d_e;
  f32x4 pz[NSPL][4];
  if (has_p) {
    const float* src = a.P + static_cast<size_t>(min(t0 + tt, a.T - 1)) * NP + 16 * pc;
    const size_t zs = static_cast<size_t>(a.T) * NP;
#pragma unroll
    for (int z = 0; z < NSPL; ++z)
#pragma unroll
      for (int q = 0; q < 4; ++q)
        pz[z][q] = *reinterpret_cast<const f32x4*>(src + (z < a.p_splits ? z : 0) * zs + 4 * q);
  }
  // (2) the local head's output weights for head columns
  u32x4 wps2[2] = {{0u, 0u, 0u, 0u}, {0u, 0u, 0u, 0u}};
  if (head) {
    const bf16_t* w = static_cast<const bf16_t*>(a.ps2) + 16 * pc - d_e;
    wps2[0] = *reinterpret_cast<const u32x4*>(w);
    wps2[1] = *reinterpret_cast<const u32x4*>(w + 8);
  }
  // (3) hidden encoder: wave w computes z_h columns [16 w, 16 w + 16)
  const int ks1 = d_e / 32;
  const bool st1 = 16 * wave < d_h;
  bf16x8 b1[KS_E];
  if (st1) {
#pragma unroll
    for (int st = 0; st < KS_E; ++st)
      if (st < ks1) b1[st] = bfrag(static_cast<const bf16_t*>(a.w_hu), d_e, d_h, 16 * wave, 32 * st, d_e, lane);
  }
  // (4) s-projections: this wave's first PF output tiles ct = wave + NWP c
  bf16x8 b2[PF][KSS];
#pragma unroll
  for (int c = 0; c < PF; ++c) {
    const int ct = cs + CS * (wave + NWP * c);
    if (ct < nct) {
      const SProj p = proj(ct);
#pragma unroll
      for (int st = 0; st < KSS; ++st) b2[c][st] = bfrag(p.w, p.ld, p.nrows, p.r0, 32 * st, d_s, lane);
    }
  }
  // (5) path vector
  if (tid < MT) {
    const int t = t0 + tid;
    float inv_rms = 0.f, dd = 0.f, dp = 0.f, pp = 0.f, pprev = 1.f, mprev = 1.f;
    if (t < a.T) {
      const f32x4 rs = *reinterpret_cast<const f32x4*>(a.rowstat + 4 * static_cast<size_t>(t));
      inv_rms = rs[0];
      dd = rs[1];
      dp = rs[2];
      pp = rs[3];
      if (j > 1) {
        pprev = a.p_hist[t];
        mprev = a.m_hist[t];
      }
    }
    const float dj = j >= 2 ? sqrtf(dd) : 0.f;
    const float gam = j >= 3 ? dp / (dj * sqrtf(pp) + a.eps) : 0.f;
    const bool pos = !(a.abl & ABL_NO_POS);
    xp[tid][0] = pos ? static_cast<float>(j) / static_cast<float>(a.L_R) : 0.f;
    xp[tid][1] = pos ? static_cast<float>(a.L_R - j) / static_cast<float>(a.L_R) : 0.f;
    xp[tid][2] = pos ? dj : 0.f;
    xp[tid][3] = pos ? gam : 0.f;
    xp[tid][4] = pprev;
    xp[tid][5] = mprev;
    sc[tid] = inv_rms;
  }
  __syncthreads();

  // hidden-encoder A fragments (columns k = 16 pc + e: k-step pc/2, groups 2 (pc&1), +1),
  // local-head partial dot products, path-encoder hidden layer
  if (has_p) {
    float x[16];
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        float v = pz[0][q][e];
#pragma unroll
        for (int z = 1; z < NSPL; ++z)
          if (z < a.p_splits) v += pz[z][q][e];
        x[4 * q + e] = v;
      }
    if (!head) {
      const float ir = sc[tt];
#pragma unroll
      for (int e = 0; e < 16; ++e) x[e] = siluf_(ir * x[e]);
      const int st = pc >> 1, g0 = 2 * (pc & 1);
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        bf16x8 hi, lo;
        split8(x + 8 * h, hi, lo);
        ax[0][st][tt + 16 * (g0 + h)] = hi;
        ax[1][st][tt + 16 * (g0 + h)] = lo;
      }
    } else {
      float acc = 0.f;
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const uint32_t w = wps2[h][i];
          acc = fmaf(__uint_as_float(w << 16), siluf_(x[8 * h + 2 * i]), acc);
          acc = fmaf(__uint_as_float(w & 0xffff0000u), siluf_(x[8 * h + 2 * i + 1]), acc);
        }
      bpart[tt][pc - d_e / 16] = acc;
    }
  }
  {
    const bf16_t* w1 = static_cast<const bf16_t*>(a.w_p1);
    for (int e = tid; e < MT * d_p; e += NTP) {
      const int t = e / d_p, o = e % d_p;
      float acc = 0.f;
#pragma unroll
      for (int k = 0; k < 6; ++k) acc = fmaf(ldf(w1 + o * 6 + k), xp[t][k], acc);
      hp[t][o] = siluf_(acc);
    }
  }
  __syncthreads();

  // z_h = W_hu x on matrix cores, z_a = W_p2 hp
  if (st1) {
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int st = 0; st < KS_E; ++st)
      if (st < ks1) acc = mfma_split(ax[0][st][lane], ax[1][st][lane], b1[st], acc);
    const int o = 16 * wave + (lane & 15);
    if (o < d_h)
#pragma unroll
      for (int r = 0; r < 4; ++r) s[4 * (lane >> 4) + r][o] = acc[r];
  }
  {
    const bf16_t* w2 = static_cast<const bf16_t*>(a.w_p2);
    for (int e = tid; e < MT * d_a; e += NTP) {
      const int t = e / d_a, o = e % d_a;
      float acc = 0.f;
      if (!(a.abl & ABL_NO_AUX))
        for (int k = 0; k < d_p; ++k) acc = fmaf(ldf(w2 + o * d_p + k), hp[t][k], acc);
      s[t][d_h + o] = acc;
    }
  }
  __syncthreads();

  // s as A fragments (zero past d_s); the local-head logit b
  for (int e = tid; e < MT * 4 * KSS; e += NTP) {
    const int i = e & 15, g = (e >> 4) & 3, st = e >> 6;
    const int k0 = 32 * st + 8 * g;
    float x[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) x[q] = k0 + q < d_s ? s[i][k0 + q] : 0.f;
    split8(x, as[0][st][i + 16 * g], as[1][st][i + 16 * g]);
  }
  if (tid < nvalid && cs == 0) {
    float b = 0.f;
    for (int q = 0; q < d_head / 16; ++q) b += bpart[tid][q];
    a.bvec[t0 + tid] = b;
  }
  __syncthreads();

  // [phi(q); phi(k); v; W_n s; th1[:, :d_s] s]
  auto finish = [&](int ct, const bf16x8* bw) {
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int st = 0; st < KSS; ++st) acc = mfma_split(as[0][st][lane], as[1][st][lane], bw[st], acc);
    const SProj p = proj(ct);
    const int o = p.r0 + (lane & 15);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int t = t0 + 4 * (lane >> 4) + r;
      if (t < a.T) p.out[static_cast<size_t>(t) * p.os + o] = p.phi ? phif_(acc[r]) : acc[r];
    }
  };
#pragma unroll
  for (int c = 0; c < PF; ++c)
    if (cs + CS * (wave + NWP * c) < nct) finish(cs + CS * (wave + NWP * c), b2[c]);
  for (int ct = cs + CS * (wave + NWP * PF); ct < nct; ct += CS * NWP) {
    const SProj p = proj(ct);
    bf16x8 bw[KSS];
#pragma unroll
    for (int st = 0; st < KSS; ++st) bw[st] = bfrag(p.w, p.ld, p.nrows, p.r0, 32 * st, d_s, lane);
    finish(ct, bw);
  }
}

// router_post on 8 waves (16 tokens per workgroup), every global load issued first:
// c (as split A fragments), W_n s, the s part of f_theta's first layer, and the weight
// fragments of W_c and of f_theta's c columns for this wave's output tiles.
template <int KSM>   // k-steps over d_m (d_m / 32)
__global__ __launch_bounds__(NTP) void router_post_mfma(RouterTailArgs a) {
  constexpr int DM = 32 * KSM;
  constexpr int TWC = (DM / 16 + NWP - 1) / NWP;      // W_c output tiles per wave
  constexpr int TWH = (MAXE / 16 + NWP - 1) / NWP;    // f_theta output tiles per wave (d_head <= 256)
  LDS16 bf16x8 ac[2][KSM][kWave];   // c: hi, lo
  LDS16 float ns[MT][DM + 4];       // W_n s
  LDS16 float wc[MT][DM + 4];       // W_c c
  __shared__ float nu[MT];
  __shared__ float apart[NWP][MT];

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int t0 = blockIdx.x * MT;
  const int nvalid = min(MT, a.T - t0);
  const int j = a.j;
  const int d_head = a.d_head, d_s = a.d_s;
  const int g4 = 4 * (lane >> 4);
  auto tok = [&](int i) { return static_cast<size_t>(min(t0 + i, a.T - 1)); };
  const bf16_t* th1 = static_cast<const bf16_t*>(a.th1);
  const bf16_t* th2 = static_cast<const bf16_t*>(a.th2);
  const bf16_t* w_c = static_cast<const bf16_t*>(a.w_c);
  const int ld = a.ld_th1, nct_h = d_head / 16;

  // a memory context exists after the first layer unless an ablation removes the memory
  const bool ctx = j > 1 && !(a.abl & (ABL_NO_MEMREAD | ABL_NO_HISTORY));
  // c rows as split fragments, and W_n s
  for (int e = tid; e < MT * 4 * KSM; e += NTP) {
    const int i = e & 15, g = (e >> 4) & 3, st = e >> 6;
    const float* src = a.cvec + tok(i) * DM + 32 * st + 8 * g;
    const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
    const f32x4 lo4 = ctx ? *reinterpret_cast<const f32x4*>(src) : zero;
    const f32x4 hi4 = ctx ? *reinterpret_cast<const f32x4*>(src + 4) : zero;
    float x[8];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      x[q] = lo4[q];
      x[4 + q] = hi4[q];
    }
    split8(x, ac[0][st][i + 16 * g], ac[1][st][i + 16 * g]);
  }
  for (int e = tid; e < MT * DM / 4; e += NTP) {
    const int i = e / (DM / 4), c4 = e % (DM / 4);
    *reinterpret_cast<f32x4*>(&ns[i][4 * c4]) =
        *reinterpret_cast<const f32x4*>(a.qkvn + tok(i) * 4 * DM + 3 * DM + 4 * c4);
  }
  // weight fragments of this wave's tiles, the s part of the pre-activation, nu and th2 weights
  bf16x8 bc[TWC][KSM], bh[TWH][KSM];
  float hsv[TWH][4], wnu[TWH], w2[TWH];
#pragma unroll
  for (int c = 0; c < TWC; ++c) {
    const int ct = wave + NWP * c;
    if (16 * ct < DM)
#pragma unroll
      for (int st = 0; st < KSM; ++st) bc[c][st] = bfrag(w_c, DM, DM, 16 * ct, 32 * st, DM, lane);
  }
#pragma unroll
  for (int c = 0; c < TWH; ++c) {
    const int ct = wave + NWP * c;
    if (ct < nct_h) {
      const int o = 16 * ct + (lane & 15);
#pragma unroll
      for (int st = 0; st < KSM; ++st) bh[c][st] = bfrag(th1 + d_s, ld, d_head, 16 * ct, 32 * st, DM, lane);
#pragma unroll
      for (int r = 0; r < 4; ++r) hsv[c][r] = a.hs[tok(g4 + r) * d_head + o];
      wnu[c] = bf16_to_f32(th1[static_cast<size_t>(o) * ld + d_s + DM]);
      w2[c] = bf16_to_f32(th2[o]);
    }
  }
  __syncthreads();

  // W_c c
#pragma unroll
  for (int c = 0; c < TWC; ++c) {
    const int ct = wave + NWP * c;
    if (16 * ct < DM) {
      f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int st = 0; st < KSM; ++st) acc = mfma_split(ac[0][st][lane], ac[1][st][lane], bc[c][st], acc);
      const int o = 16 * ct + (lane & 15);
#pragma unroll
      for (int r = 0; r < 4; ++r) wc[g4 + r][o] = acc[r];
    }
  }
  __syncthreads();

  // nu = 1 - cos(W_n s, W_c c); 0 at j = 1
  for (int i = wave; i < MT; i += NWP) {
    float nn = 0.f, cc = 0.f, nc = 0.f;
    for (int k = lane; k < DM; k += kWave) {
      const float n = ns[i][k], c = wc[i][k];
      nn = fmaf(n, n, nn);
      cc = fmaf(c, c, cc);
      nc = fmaf(n, c, nc);
    }
    nn = wave_sum(nn);
    cc = wave_sum(cc);
    nc = wave_sum(nc);
    if (lane == 0) nu[i] = ctx ? 1.0f - nc / (sqrtf(nn) * sqrtf(cc) + a.eps) : 0.f;
  }
  __syncthreads();

  // a = th2 . SiLU(th1 [s; c; nu])
  float ap[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int c = 0; c < TWH; ++c) {
    const int ct = wave + NWP * c;
    if (ct < nct_h) {
      f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int st = 0; st < KSM; ++st) acc = mfma_split(ac[0][st][lane], ac[1][st][lane], bh[c][st], acc);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float pre = acc[r] + hsv[c][r] + wnu[c] * nu[g4 + r];
        ap[r] = fmaf(w2[c], siluf_(pre), ap[r]);
      }
    }
  }
#pragma unroll
  for (int r = 0; r < 4; ++r)
#pragma unroll
    for (int off = 1; off < 16; off <<= 1) ap[r] += __shfl_xor(ap[r], off, kWave);
  if ((lane & 15) == 0)
#pragma unroll
    for (int r = 0; r < 4; ++r) apart[wave][g4 + r] = ap[r];
  __syncthreads();
  if (tid < nvalid) {
    const int t = t0 + tid;
    const bool hist = !(a.abl & ABL_NO_HISTORY);
    float av = 0.f;
#pragma unroll
    for (int w = 0; w < NWP; ++w) av += apart[w][tid];
    if (!hist) av = 0.f;
    const float mprev = j > 1 ? a.m_hist[t] : 1.0f;
    const float p = sigmoidf_(av / a.T_hist);
    a.p_hist[t] = hist ? p : 1.0f;
    a.m_hist[t] = hist ? mprev * p : 1.0f;
    const float l = av + a.bvec[t] + (a.beta ? a.beta[t] : 0.f);
    a.logit[t] = l;
    a.gate[t] = sigmoidf_(l);
  }
}

// ---------------------------------------------------------------------------
// router_mem_hist: the memory read in depth-history form, one wave per token.
//   a_i = w_i phi(q) . phi(k_i),  c = sum_i a_i v_i / (sum_i a_i + eps)  over the stored
//   pairs i < j-1 (oldest first), then the layer's own (phi(k), v) stored as entry j-1.
// Each lane owns EPL consecutive elements of the d_m-vectors; the pairs are read in
// batches of HB with all of a batch's loads issued first.
// ---------------------------------------------------------------------------
template <int DM>
__global__ __launch_bounds__(NT) void router_mem_hist_kernel(RouterTailArgs a) {
  constexpr int EPL = DM >= kWave ? DM / kWave : 1;   // elements per lane
  constexpr int LANES = DM >= kWave ? kWave : DM;     // lanes holding elements
  constexpr int HB = 8;
  const int lane = threadIdx.x & 63;
  const int t = blockIdx.x * (NT / kWave) + (threadIdx.x >> 6);
  if (t >= a.T) return;
  const int n = a.j - 1;
  const bool on = lane < LANES;
  const int e0 = lane * EPL;
  const float* q = a.qkvn + static_cast<size_t>(t) * 4 * DM;
  float fq[EPL], fk[EPL], vv[EPL];
#pragma unroll
  for (int x = 0; x < EPL; ++x) {
    fq[x] = on ? q[e0 + x] : 0.f;
    fk[x] = on ? q[DM + e0 + x] : 0.f;
    vv[x] = on ? q[2 * DM + e0 + x] : 0.f;
  }
  float* H = a.kv + static_cast<size_t>(t) * a.L_R * 2 * DM;
  float c[EPL];
#pragma unroll
  for (int x = 0; x < EPL; ++x) c[x] = 0.f;
  float den = 0.f;
  for (int i0 = 0; i0 < n; i0 += HB) {
    float kk[HB][EPL], vh[HB][EPL];
#pragma unroll
    for (int u = 0; u < HB; ++u) {
      const int i = i0 + u;
      const float* hk = H + static_cast<size_t>(min(i, n - 1)) * 2 * DM + e0;
#pragma unroll
      for (int x = 0; x < EPL; ++x) {
        kk[u][x] = on ? hk[x] : 0.f;
        vh[u][x] = on ? hk[DM + x] : 0.f;
      }
    }
    float dots[HB];
#pragma unroll
    for (int u = 0; u < HB; ++u) {
      float s = 0.f;
#pragma unroll
      for (int x = 0; x < EPL; ++x) s = fmaf(fq[x], kk[u][x], s);
      dots[u] = wave_sum(s);
    }
#pragma unroll
    for (int u = 0; u < HB; ++u) {
      if (i0 + u < n) {
        const float al = a.hw[i0 + u] * dots[u];
        den += al;
#pragma unroll
        for (int x = 0; x < EPL; ++x) c[x] = fmaf(al, vh[u][x], c[x]);
      }
    }
  }
  if (on) {
    float* cv = a.cvec + static_cast<size_t>(t) * DM + e0;
    float* hn = H + static_cast<size_t>(n) * 2 * DM + e0;
#pragma unroll
    for (int x = 0; x < EPL; ++x) {
      cv[x] = n > 0 ? c[x] / (den + a.eps) : 0.f;
      hn[x] = fk[x];
      hn[DM + x] = vv[x];
    }
  }
}

// S[t][k][v] = sum_{i<n} w_i phi(k_i)[k] v_i[v], zeta[t][k] = sum_{i<n} w_i phi(k_i)[k];
// one workgroup per token, oldest pair first.
template <int DM>
__global__ __launch_bounds__(NT) void history_state_kernel(const float* __restrict__ kv, int L_R, int n,
                                                           HistWeights hw, float* __restrict__ S,
                                                           float* __restrict__ zeta) {
  const int t = blockIdx.x;
  const float* H = kv + static_cast<size_t>(t) * L_R * 2 * DM;
  float* St = S + static_cast<size_t>(t) * DM * DM;
  for (int e = threadIdx.x; e < DM * DM; e += NT) {
    const int k = e / DM, v = e % DM;
    float acc = 0.f;
    for (int i = 0; i < n; ++i) acc = fmaf(hw.w[i] * H[i * 2 * DM + k], H[i * 2 * DM + DM + v], acc);
    St[e] = acc;
  }
  for (int k = threadIdx.x; k < DM; k += NT) {
    float z = 0.f;
    for (int i = 0; i < n; ++i) z = fmaf(hw.w[i], H[i * 2 * DM + k], z);
    zeta[static_cast<size_t>(t) * DM + k] = z;
  }
}

// ---------------------------------------------------------------------------
// router_token: the whole router after its two large projections in one launch, one token per
// workgroup of 512 threads, for calls of few tokens (a decode step).
//
// With few tokens each of the three kernels above is a chain of latencies on a handful of
// workgroups: a round trip to HBM for its inputs (the router's weights have left the caches: the
// FFN weights of a layer stream through them between two layers), a few barriers, a launch.
// Here every weight of the router and the token's memory are loaded at the start, in one round
// trip, into registers (PRE: the widths where they fit); what follows works from LDS between
// barriers.  A matrix [O][I] is spread over the threads in pieces of eight inputs: thread t holds
// piece t mod PI (PI >= I / 8, a power of two) of rows t / PI, t / PI + 512 / PI, ..., so it needs
// the same eight inputs for every row, and a row's sum is formed over PI neighbouring lanes.
// Weights are widened to fp32 and every product and sum is fp32.  At 256 tokens of d_m = 128:
// 14 us for the 31 us of the three kernels (4 us until the loads are out, 1 us for them, then the
// chain of seven barriers).
// ---------------------------------------------------------------------------
constexpr int NTT = 512;                 // threads per token
constexpr int NWT = NTT / kWave;
constexpr int kTokenMaxS = 64;           // widths the thread layout covers: d_s, d_h, d_a
constexpr int kTokenMaxP = 128;          // d_p
constexpr int kHistMax = 64;             // stored pairs
// Most tokens of a call: three rounds of workgroups with bf16 weights, eight with fp32, whose three
// kernels are VALU chains.  Measured against the three kernels, a layer of d = 4096, d_ff = 14336,
// d_m = 128 (bf16): 187 -> 178 us at 300 tokens, 214 -> 205 at 512, 311 -> 307 at 768, 328 -> 330 at
// 1024; d_m = 256 at 512 tokens 256 -> 246, depth-history memory 208 -> 198.  fp32, four layers of
// d = 256, d_m = 32: 426 -> 208 us at 300 tokens, 614 -> 569 at 2048, 818 -> 989 at 4096.
constexpr int kTokenRowsBf16 = 768, kTokenRowsF32 = 2048;

template <typename W, int PI, int R>
struct TokenMat {
  Raw8<W> w[R];
  static constexpr int ROWS = NTT / PI;  // rows per pass
  // row(o): first element of row o.  Threads past the O rows or the I inputs (I % 8 == 0) load the
  // last ones instead of branching (a branch per load made the loads wait for one another)
  template <class Row>
  __device__ __forceinline__ void load(int O, int I, Row row) {
    const int sl = min(static_cast<int>(threadIdx.x) % PI, I / 8 - 1), o0 = static_cast<int>(threadIdx.x) / PI;
#pragma unroll
    for (int r = 0; r < R; ++r) w[r].load(row(min(o0 + ROWS * r, O - 1)) + 8 * sl);
  }
  // f(r, o, sum): lane l of a group gets the sums of the group's rows r = l, l + PI, ... below O, so
  // that what follows a sum runs once per lane and not once per row in every lane
  template <class F>
  __device__ __forceinline__ void dot(const float* x, int O, int I, F f) const {
    const int sl = static_cast<int>(threadIdx.x) % PI, o0 = static_cast<int>(threadIdx.x) / PI;
    const bool in = 8 * sl < I;
    float xv[8];
    *reinterpret_cast<f32x4*>(xv) = *reinterpret_cast<const f32x4*>(x + 8 * sl);
    *reinterpret_cast<f32x4*>(xv + 4) = *reinterpret_cast<const f32x4*>(x + 8 * sl + 4);
    constexpr int G = (R + PI - 1) / PI;
    float mine[G];
#pragma unroll
    for (int r = 0; r < R; ++r) {
      float acc = 0.f;
#pragma unroll
      for (int e = 0; e < 8; ++e) acc = fmaf(w[r][e], xv[e], acc);
      acc = group_sum<PI>(in ? acc : 0.f);
      mine[r / PI] = r % PI == 0 || sl == r % PI ? acc : mine[r / PI];
    }
#pragma unroll
    for (int g = 0; g < G; ++g) {
      const int r = g * PI + sl, o = o0 + ROWS * r;
      if (r < R && o < O) f(g, o, mine[g]);
    }
  }
};

// A kernel argument held in scalar registers from here on.  Pointers keep the global address space
// (through a generic pointer the accesses would be flat ones).
template <typename T>
__device__ __forceinline__ T keep_scalar(T v) {
  if constexpr (std::is_pointer<T>::value) {
    typedef __attribute__((address_space(1))) typename std::remove_pointer<T>::type* G;
    G g = (G)v;
    asm volatile("" : "+s"(g));
    return (T)g;
  } else {
    asm volatile("" : "+s"(v));
    return v;
  }
}

// HIST: the memory in depth-history form (kv, hw); otherwise the matrix S of storage type ST
template <typename W, int DM, typename ST, bool HIST, bool PRE>
__global__ __launch_bounds__(NTT, 2) void router_token_kernel(RouterTailArgs args) {
  constexpr int PM = DM / 8;                                   // pieces of a d_m-wide row
  constexpr int R_HU = kTokenMaxS * 32 / NTT, R_P2 = kTokenMaxS * 16 / NTT;
  constexpr int R_Q = 4 * DM * 8 / NTT > 0 ? 4 * DM * 8 / NTT : 1;
  constexpr int R_TS = MAXE * 8 / NTT;
  constexpr int R_C = DM * PM / NTT > 0 ? DM * PM / NTT : 1;
  constexpr int R_TC = MAXE * PM / NTT > 0 ? MAXE * PM / NTT : 1;
  constexpr int VE = 16 / static_cast<int>(sizeof(ST));        // state elements per 16 bytes
  constexpr int CV = DM / VE, RP = NTT / CV;                   // vectors per S row, rows per pass
  constexpr int NR = DM / RP > 0 ? DM / RP : 1;                // S rows per thread
  constexpr int CH = NR < 8 ? NR : 8;                          // ... per batch
  constexpr int EPL = DM >= kWave ? DM / kWave : 1;            // history: elements per lane
  constexpr int HPW = kHistMax / NWT;                          // history: pairs per wave
  constexpr int NRED = HIST ? NWT : (RP < DM ? RP : DM);
  LDS16 float xs[MAXE];           // SiLU(inv_rms W_hd hbar)
  LDS16 float hp[kTokenMaxP];     // path-encoder hidden
  LDS16 float s[kTokenMaxS];
  LDS16 float pr[4][DM];          // phi(q), phi(k), v, W_n s
  LDS16 float hs[MAXE];           // th1[:, :d_s] s
  LDS16 float cv[DM];             // c
  LDS16 float red[NRED][DM];
  __shared__ float bpart[NWT], dpart[NWT], npart[NWT][3], apart[NWT];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const size_t t = blockIdx.x;
  // the arguments into scalar registers at once (read where they are used, each group of them is a
  // round trip of its own)
#define HERO_KEEP(x) const auto a_##x = keep_scalar(args.x)
  HERO_KEEP(T); HERO_KEEP(j); HERO_KEEP(L_R); HERO_KEEP(d_s); HERO_KEEP(d_h); HERO_KEEP(d_a); HERO_KEEP(d_e);
  HERO_KEEP(d_p); HERO_KEEP(d_head); HERO_KEEP(eps); HERO_KEEP(T_hist); HERO_KEEP(eta); HERO_KEEP(P);
  HERO_KEEP(p_splits); HERO_KEEP(rowstat); HERO_KEEP(w_hu); HERO_KEEP(w_p1); HERO_KEEP(w_p2); HERO_KEEP(w_q);
  HERO_KEEP(w_k); HERO_KEEP(w_v); HERO_KEEP(w_n); HERO_KEEP(w_c); HERO_KEEP(th1); HERO_KEEP(th2); HERO_KEEP(ps2);
  HERO_KEEP(ld_th1); HERO_KEEP(beta); HERO_KEEP(abl); HERO_KEEP(S); HERO_KEEP(zeta); HERO_KEEP(p_hist);
  HERO_KEEP(m_hist); HERO_KEEP(logit); HERO_KEEP(gate); HERO_KEEP(kv); HERO_KEEP(c_read);
#undef HERO_KEEP
  const int j = a_j, d_e = a_d_e, d_head = a_d_head, NP = d_e + d_head;
  const int d_s = a_d_s, d_h = a_d_h, d_a = a_d_a, d_p = a_d_p;
  const bool mem = !(a_abl & (ABL_NO_MEMREAD | ABL_NO_HISTORY));
  const bool ctx = j > 1 && mem;

  // (1) every load of the kernel, none under a branch of its own
  float pv[MAXSPLIT];
  const int pcol = min(tid, NP - 1);
#pragma unroll
  for (int z = 0; z < MAXSPLIT; ++z)
    pv[z] = a_P[(static_cast<size_t>(min(z, a_p_splits - 1)) * a_T + t) * NP + pcol];
  const f32x4 rs = *reinterpret_cast<const f32x4*>(a_rowstat + 4 * t);
  const float pprev = j > 1 ? a_p_hist[t] : 1.f, mprev = j > 1 ? a_m_hist[t] : 1.f;
  const float beta = a_beta ? a_beta[t] : 0.f;
  W p1[6];
#pragma unroll
  for (int k = 0; k < 6; ++k) p1[k] = static_cast<const W*>(a_w_p1)[min(tid, d_p - 1) * 6 + k];
  const bool head = tid >= d_e && tid < NP;
  const W ps2 = static_cast<const W*>(a_ps2)[min(max(tid - d_e, 0), d_head - 1)];
  TokenMat<W, 32, R_HU> m_hu;
  TokenMat<W, 16, R_P2> m_p2;
  TokenMat<W, 8, R_Q> m_q;
  TokenMat<W, 8, R_TS> m_ts;
  TokenMat<W, PM, R_C> m_c;
  TokenMat<W, PM, R_TC> m_tc;
  // the history head's outputs this lane finishes (rows past the last: not used)
  constexpr int G_TC = (R_TC + PM - 1) / PM;
  W wnu[G_TC], th2[G_TC];
  auto own = [&](int g) {
    const int r = g * PM + tid % PM;
    return r < R_TC ? tid / PM + NTT / PM * r : MAXE;
  };
  auto load_hu = [&] {
    m_hu.load(d_h, d_e, [&](int o) { return static_cast<const W*>(a_w_hu) + o * d_e; });
    m_p2.load(d_a, d_p, [&](int o) { return static_cast<const W*>(a_w_p2) + o * d_p; });
  };
  auto load_s = [&] {
    m_q.load(4 * DM, d_s, [&](int o) {
      const int m = o / DM;
      const void* w = m == 0 ? a_w_q : m == 1 ? a_w_k : m == 2 ? a_w_v : a_w_n;
      return static_cast<const W*>(w) + (o - m * DM) * d_s;
    });
    m_ts.load(d_head, d_s, [&](int o) { return static_cast<const W*>(a_th1) + o * a_ld_th1; });
  };
  auto load_c = [&] {
    m_c.load(DM, DM, [&](int o) { return static_cast<const W*>(a_w_c) + o * DM; });
    m_tc.load(d_head, DM, [&](int o) { return static_cast<const W*>(a_th1) + o * a_ld_th1 + d_s; });
#pragma unroll
    for (int g = 0; g < G_TC; ++g) {
      const int o = min(own(g), d_head - 1);
      wnu[g] = static_cast<const W*>(a_th1)[o * a_ld_th1 + d_s + DM];
      th2[g] = static_cast<const W*>(a_th2)[o];
    }
  };
  // the token's memory: S rows rg, rg + RP, ... (columns VE cq ..), or the wave's pairs
  const int cq = tid % CV, rg = tid / CV;
  const bool on = rg < DM;
  ST* Sp = HIST ? nullptr : static_cast<ST*>(a_S) + t * DM * DM + VE * cq;
  u32x4 sv[HIST ? 1 : CH];
  auto load_mem = [&](int i0) {
#pragma unroll
    for (int c = 0; c < CH; ++c) sv[c] = *reinterpret_cast<const u32x4*>(Sp + (min(rg, DM - 1) + RP * (i0 + c)) * DM);
  };
  float* H = HIST ? a_kv + t * a_L_R * 2 * DM : nullptr;
  const int np = j - 1;                       // stored pairs
  const bool hl = lane * EPL < DM;
  float hk[HIST ? HPW : 1][EPL], hv[HIST ? HPW : 1][EPL];   // the last pair stands in past np, unused
  float zv = 0.f;
  auto load_pairs = [&] {
#pragma unroll
    for (int u = 0; u < (HIST ? HPW : 0); ++u) {
      const float* h = H + static_cast<size_t>(max(min(wave + NWT * u, np - 1), 0)) * 2 * DM + min(lane * EPL, DM - EPL);
#pragma unroll
      for (int x = 0; x < EPL; ++x) {
        hk[u][x] = h[x];
        hv[u][x] = h[DM + x];
      }
    }
  };
  if constexpr (HIST) {
    if (PRE && mem) load_pairs();
  } else if (ctx) {
    if constexpr (PRE && NR == CH) load_mem(0);
    zv = a_zeta[t * DM + min(tid, DM - 1)];
  }
  if constexpr (PRE) {
    load_hu();
    load_s();
    load_c();
  }

  // (2) SiLU of the pre-activations, the local head's shares, the path encoder's hidden layer
  float p = pv[0];
#pragma unroll
  for (int z = 1; z < MAXSPLIT; ++z) p += z < a_p_splits ? pv[z] : 0.f;
  if (tid < d_e) xs[tid] = siluf_(rs[0] * p);
  const float bsum = wave_sum(head ? ldf(&ps2) * siluf_(p) : 0.f);
  if (lane == 0) bpart[wave] = bsum;
  for (int e = d_e + tid; e < MAXE; e += NTT) xs[e] = 0.f;
  if (tid < kTokenMaxP) {
    float h = 0.f;
    if (tid < d_p) {
      const float dj = j >= 2 ? sqrtf(rs[1]) : 0.f;
      const float gam = j >= 3 ? rs[2] / (dj * sqrtf(rs[3]) + a_eps) : 0.f;
      const bool pos = !(a_abl & ABL_NO_POS);
      const float xp[6] = {pos ? static_cast<float>(j) / static_cast<float>(a_L_R) : 0.f,
                           pos ? static_cast<float>(a_L_R - j) / static_cast<float>(a_L_R) : 0.f,
                           pos ? dj : 0.f, pos ? gam : 0.f, pprev, mprev};
#pragma unroll
      for (int k = 0; k < 6; ++k) h = fmaf(ldf(&p1[k]), xp[k], h);
      h = siluf_(h);
    }
    hp[tid] = h;
  }
  if (tid < kTokenMaxS) s[tid] = 0.f;
  if constexpr (!PRE) load_hu();
  __syncthreads();

  // (3) s = [z_h; z_a]
  m_hu.dot(xs, d_h, d_e, [&](int, int o, float v) { s[o] = v; });
  m_p2.dot(hp, d_a, d_p, [&](int, int o, float v) { s[d_h + o] = a_abl & ABL_NO_AUX ? 0.f : v; });
  if constexpr (!PRE) load_s();
  __syncthreads();

  // (4) phi(q), phi(k), v, W_n s and the s part of the history head
  m_q.dot(s, 4 * DM, d_s, [&](int, int o, float v) {
    pr[o / DM][o % DM] = o < 2 * DM ? phif_(v) : v;
  });
  m_ts.dot(s, d_head, d_s, [&](int, int o, float v) { hs[o] = v; });
  if constexpr (!PRE) load_c();
  __syncthreads();

  // (5) memory read, then write
  if constexpr (HIST) {
    float c[EPL], den = 0.f;
#pragma unroll
    for (int x = 0; x < EPL; ++x) c[x] = 0.f;
    if (mem) {
      if (!PRE) load_pairs();
#pragma unroll
      for (int u = 0; u < HPW; ++u) {
        const int i = wave + NWT * u;
        if (i < np) {
          float d = 0.f;
#pragma unroll
          for (int x = 0; x < EPL; ++x)
            if (hl) d = fmaf(pr[0][lane * EPL + x], hk[u][x], d);
          const float al = args.hw[i] * wave_sum(d);
          den += al;
#pragma unroll
          for (int x = 0; x < EPL; ++x) c[x] = fmaf(al, hv[u][x], c[x]);
        }
      }
      for (int e = tid; e < 2 * DM; e += NTT) H[static_cast<size_t>(np) * 2 * DM + e] = pr[1 + e / DM][e % DM];
    }
    if (lane == 0) dpart[wave] = den;
    if (hl)
#pragma unroll
      for (int x = 0; x < EPL; ++x) red[wave][lane * EPL + x] = c[x];
  } else {
    const float rho = 1.0f / (1.0f + expf(-a_eta));
    float d = 0.f;
    if (mem && tid < DM) {
      d = pr[0][tid] * zv;
      a_zeta[t * DM + tid] = fmaf(rho, zv, pr[1][tid]);
    }
    d = wave_sum(d);
    if (lane == 0) dpart[wave] = d;
    float vr[VE], cacc[VE];
#pragma unroll
    for (int e = 0; e < VE; ++e) {
      vr[e] = pr[2][VE * cq + e];
      cacc[e] = 0.f;
    }
    auto store = [&](int r, const float* o) {
      u32x4 w;
      if constexpr (VE == 4) {
#pragma unroll
        for (int e = 0; e < 4; ++e) w[e] = __float_as_uint(o[e]);
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
          w[e] = static_cast<uint32_t>(f32_to_bf16(o[2 * e])) |
                 (static_cast<uint32_t>(f32_to_bf16(o[2 * e + 1])) << 16);
      }
      *reinterpret_cast<u32x4*>(Sp + r * DM) = w;
    };
    if (ctx && on) {
      for (int i0 = 0; i0 < NR; i0 += CH) {
        if (!(PRE && NR == CH)) load_mem(i0);
#pragma unroll
        for (int c = 0; c < CH; ++c) {
          const int r = rg + RP * (i0 + c);
          const float qv = pr[0][r], kv = pr[1][r];
          float o[VE];
#pragma unroll
          for (int e = 0; e < VE; ++e) {
            float x;
            if constexpr (VE == 4)
              x = __uint_as_float(sv[c][e]);
            else
              x = __uint_as_float(e & 1 ? sv[c][e >> 1] & 0xffff0000u : sv[c][e >> 1] << 16);
            cacc[e] = fmaf(qv, x, cacc[e]);
            o[e] = fmaf(rho, x, kv * vr[e]);
          }
          store(r, o);
        }
      }
    } else if (mem && on) {
      for (int i = 0; i < NR; ++i) {
        const int r = rg + RP * i;
        float o[VE];
#pragma unroll
        for (int e = 0; e < VE; ++e) o[e] = pr[1][r] * vr[e];
        store(r, o);
      }
    }
    if (on)
#pragma unroll
      for (int e = 0; e < VE; ++e) red[rg][VE * cq + e] = cacc[e];
  }
  __syncthreads();
  if (tid < DM) {
    float c = 0.f, den = 0.f;
#pragma unroll
    for (int g = 0; g < NRED; ++g) c += red[g][tid];
#pragma unroll
    for (int w = 0; w < NWT; ++w) den += dpart[w];
    c = ctx ? c / (den + a_eps) : 0.f;
    cv[tid] = c;
    if (a_c_read && mem) a_c_read[t * DM + tid] = c;
  }
  __syncthreads();

  // (6) W_c c beside W_n s for nu; the c part of the history head
  float nn = 0.f, cc = 0.f, nc = 0.f, pre[G_TC];
  m_c.dot(cv, DM, DM, [&](int, int o, float v) {
    const float n = pr[3][o];
    nn = fmaf(n, n, nn);
    cc = fmaf(v, v, cc);
    nc = fmaf(n, v, nc);
  });
#pragma unroll
  for (int g = 0; g < G_TC; ++g) pre[g] = 0.f;
  m_tc.dot(cv, d_head, DM, [&](int g, int o, float v) { pre[g] = v + hs[o]; });
  nn = wave_sum(nn);
  cc = wave_sum(cc);
  nc = wave_sum(nc);
  if (lane == 0) {
    npart[wave][0] = nn;
    npart[wave][1] = cc;
    npart[wave][2] = nc;
  }
  __syncthreads();
  float tot[3] = {0.f, 0.f, 0.f};
#pragma unroll
  for (int w = 0; w < NWT; ++w)
#pragma unroll
    for (int e = 0; e < 3; ++e) tot[e] += npart[w][e];
  const float nu = ctx ? 1.0f - tot[2] / (sqrtf(tot[0]) * sqrtf(tot[1]) + a_eps) : 0.f;
  float av = 0.f;
#pragma unroll
  for (int g = 0; g < G_TC; ++g)
    if (own(g) < d_head) av = fmaf(ldf(&th2[g]), siluf_(fmaf(ldf(&wnu[g]), nu, pre[g])), av);
  av = wave_sum(av);
  if (lane == 0) apart[wave] = av;
  __syncthreads();
  if (tid == 0) {
    const bool hist = !(a_abl & ABL_NO_HISTORY);
    float aa = 0.f, b = 0.f;
#pragma unroll
    for (int w = 0; w < NWT; ++w) {
      aa += apart[w];
      b += bpart[w];
    }
    if (!hist) aa = 0.f;
    const float ph = sigmoidf_(aa / a_T_hist);
    a_p_hist[t] = hist ? ph : 1.0f;
    a_m_hist[t] = hist ? mprev * ph : 1.0f;
    const float l = aa + b + beta;
    a_logit[t] = l;
    a_gate[t] = sigmoidf_(l);
  }
}

template <typename W, int DM>
hipError_t launch_token_dm(const RouterTailArgs& a, bool hist, hipStream_t s) {
  // the widths whose weights and memory fit the registers of two waves per SIMD
  constexpr bool PRE = sizeof(W) == 2 ? DM <= 128 : DM <= 64;
  if (hist) {
    router_token_kernel<W, DM, float, true, PRE><<<a.T, NTT, 0, s>>>(a);
  } else if (a.state_bf16) {
    if constexpr (DM >= 64)
      router_token_kernel<W, DM, bf16_t, false, PRE><<<a.T, NTT, 0, s>>>(a);
    else
      return hipErrorInvalidValue;
  } else {
    router_token_kernel<W, DM, float, false, PRE><<<a.T, NTT, 0, s>>>(a);
  }
  return hipGetLastError();
}

template <typename W>
hipError_t launch_token(const RouterTailArgs& a, bool hist, hipStream_t s) {
  switch (a.d_m) {
    case 32: return launch_token_dm<W, 32>(a, hist, s);
    case 64: return launch_token_dm<W, 64>(a, hist, s);
    case 128: return launch_token_dm<W, 128>(a, hist, s);
    case 256:
      if constexpr (sizeof(W) == 2) return launch_token_dm<W, 256>(a, hist, s);
      return hipErrorInvalidValue;
    default: return hipErrorInvalidValue;
  }
}

#undef LDS16

hipError_t launch_pre_post(const RouterTailArgs& a, bool post, hipStream_t s) {
  if (a.dtype == 1) {
    dim3 grid((a.T + MT - 1) / MT);
    if (post) {
      switch (a.d_m) {
        case 32: router_post_mfma<1><<<grid, NTP, 0, s>>>(a); break;
        case 64: router_post_mfma<2><<<grid, NTP, 0, s>>>(a); break;
        case 128: router_post_mfma<4><<<grid, NTP, 0, s>>>(a); break;
        case 256: router_post_mfma<8><<<grid, NTP, 0, s>>>(a); break;
        default: return hipErrorInvalidValue;
      }
    } else {
      // many rounds of workgroups (more than two per CU) with an unsplit P: two resident
      // workgroups per CU, weight fragments loaded as they are needed
      const bool many = grid.x > 2u * kCUsRouter && a.p_splits == 1;
      // few token groups: the s-projections' output tiles split over up to 16 column groups per
      // token group, so that the launch covers the CUs (decode, 256 tokens: 16 x 16 workgroups)
      const int nct = 4 * (a.d_m / 16) + a.d_head / 16;
      grid.y = static_cast<unsigned>(std::max(1, std::min({16, static_cast<int>(kCUsRouter / grid.x), nct})));
      switch ((a.d_s + 31) / 32) {
        case 1: many ? router_pre_mfma<1, 4, 1, 1><<<grid, NTP, 0, s>>>(a) : router_pre_mfma<1><<<grid, NTP, 0, s>>>(a); break;
        case 2: many ? router_pre_mfma<2, 4, 1, 1><<<grid, NTP, 0, s>>>(a) : router_pre_mfma<2><<<grid, NTP, 0, s>>>(a); break;
        case 3: many ? router_pre_mfma<3, 4, 1, 1><<<grid, NTP, 0, s>>>(a) : router_pre_mfma<3><<<grid, NTP, 0, s>>>(a); break;
        case 4: many ? router_pre_mfma<4, 4, 1, 1><<<grid, NTP, 0, s>>>(a) : router_pre_mfma<4><<<grid, NTP, 0, s>>>(a); break;
        default: return hipErrorInvalidValue;
      }
    }
  } else {
    dim3 grid((a.T + TB - 1) / TB), block(NT);
    if (post)
      router_post_kernel<float><<<grid, block, 0, s>>>(a);
    else
      router_pre_kernel<float><<<grid, block, 0, s>>>(a);
  }
  return hipGetLastError();
}

}  // namespace

size_t router_scratch_floats(int d_m, int d_head, int T) {
  return static_cast<size_t>(T) * (4 * d_m + d_head + d_m + 1);
}

bool router_token_fits(int dtype, int T, int d_m, int d_s, int d_h, int d_a, int d_e, int d_p, int d_head) {
  return T <= (dtype == 1 ? kTokenRowsBf16 : kTokenRowsF32) && (dtype == 1 || d_m <= 128) && d_s <= kTokenMaxS && d_h <= kTokenMaxS && d_a <= kTokenMaxS && d_p <= kTokenMaxP &&
         d_e <= MAXE && d_head <= MAXE && d_s % 8 == 0 && d_e % 8 == 0 && d_p % 8 == 0;
}

hipError_t launch_router_token(const RouterTailArgs& a, bool hist, hipStream_t s) {
  if (a.T <= 0) return hipSuccess;
  if (a.p_splits < 1 || a.p_splits > MAXSPLIT || (hist && (a.j < 1 || a.j > a.L_R || a.L_R > kHistMax)))
    return hipErrorInvalidValue;
  return a.dtype == 1 ? launch_token<bf16_t>(a, hist, s) : launch_token<float>(a, hist, s);
}

hipError_t launch_router_pre(const RouterTailArgs& a, hipStream_t s) {
  if (a.T <= 0) return hipSuccess;
  if (a.p_splits < 1 || a.p_splits > (a.dtype == 1 ? MAXSPLIT : 1)) return hipErrorInvalidValue;
  return launch_pre_post(a, false, s);
}

hipError_t launch_router_mem(const RouterTailArgs& a, hipStream_t s) {
  if (a.T <= 0) return hipSuccess;
  dim3 grid(a.T), block(NT);
  if (a.state_bf16) {
    switch (a.d_m) {
      case 64: router_mem_kernel<64, bf16_t><<<grid, block, 0, s>>>(a); break;
      case 128: router_mem_kernel<128, bf16_t><<<grid, block, 0, s>>>(a); break;
      case 256: router_mem_kernel<256, bf16_t><<<grid, block, 0, s>>>(a); break;
      default: return hipErrorInvalidValue;
    }
  } else {
    switch (a.d_m) {
      case 32: router_mem_kernel<32, float><<<grid, block, 0, s>>>(a); break;
      case 64: router_mem_kernel<64, float><<<grid, block, 0, s>>>(a); break;
      case 128: router_mem_kernel<128, float><<<grid, block, 0, s>>>(a); break;
      case 256: router_mem_kernel<256, float><<<grid, block, 0, s>>>(a); break;
      default: return hipErrorInvalidValue;
    }
  }
  return hipGetLastError();
}

hipError_t launch_router_mem_hist(const RouterTailArgs& a, hipStream_t s) {
  if (a.T <= 0) return hipSuccess;
  if (a.j < 1 || a.j > a.L_R || a.L_R > 64) return hipErrorInvalidValue;
  dim3 grid((a.T + NT / kWave - 1) / (NT / kWave)), block(NT);
  switch (a.d_m) {
    case 32: router_mem_hist_kernel<32><<<grid, block, 0, s>>>(a); break;
    case 64: router_mem_hist_kernel<64><<<grid, block, 0, s>>>(a); break;
    case 128: router_mem_hist_kernel<128><<<grid, block, 0, s>>>(a); break;
    case 256: router_mem_hist_kernel<256><<<grid, block, 0, s>>>(a); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_history_state(int d_m, int L_R, int n, int T, const float* kv, const HistWeights& w,
                                float* S, float* zeta, hipStream_t s) {
  if (T <= 0) return hipSuccess;
  if (n < 0 || n > L_R || L_R > 64) return hipErrorInvalidValue;
  dim3 grid(T), block(NT);
  switch (d_m) {
    case 32: history_state_kernel<32><<<grid, block, 0, s>>>(kv, L_R, n, w, S, zeta); break;
    case 64: history_state_kernel<64><<<grid, block, 0, s>>>(kv, L_R, n, w, S, zeta); break;
    case 128: history_state_kernel<128><<<grid, block, 0, s>>>(kv, L_R, n, w, S, zeta); break;
    case 256: history_state_kernel<256><<<grid, block, 0, s>>>(kv, L_R, n, w, S, zeta); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_router_post(const RouterTailArgs& a, hipStream_t s) {
  if (a.T <= 0) return hipSuccess;
  return launch_pre_post(a, true, s);
}

}  // namespace hero
