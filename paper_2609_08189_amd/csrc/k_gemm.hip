// Dense contractions of the routed layer.
//
//   router pre-activations   P = hbar [W_hd; psi_1]^T                 (Sec. 3.2, z^h and f_psi)
//   FFN gate/up              act = SiLU(u W_g^T) * (u W_u^T)          (frozen SwiGLU FFN)
//   FFN down + scatter       h_out[t] = hbar[t] + g_t (act W_d^T)     (Sec. 3.1, eq:ffn_route)
//   adapter down             hid = SiLU(u W_1^T)                      (Sec. 3.1, adapter)
//   adapter up + scatter     h_out[t] = hbar[t] + (1 - g_t) (hid W_2^T)
//
// bf16 path: MFMA with fp32 accumulation, three kernels.  phase_gemm (16x16x32) takes
// the large products, mfma_gemm (32x32x16) the smaller tiles of the router, the wide
// adapters and few rows with K split, skinny_gemm the decode steps.  A and B are both
// K-contiguous ("x W^T" with nn.Linear weights).  A k-tile of 64 elements
// (128 bytes per row) of A and B is staged through LDS, double buffered, with
// the 16-byte chunks of each row XOR-swizzled by (row / 2) & 7 so that the
// fragment reads of one MFMA hit distinct banks.  A rows may be gathered through
// an index list whose length lives on the device (tiles past it exit at once).
// Workgroups are mapped to tiles so that each XCD (8 per MI355X, round-robin
// dispatch) owns a contiguous run of a grouped tile order: the tiles it runs at
// once share a few row panels and a few weight panels in its L2.
//
// f32 path: small tiles on the fp32 matrix cores, 64 x 64 VALU tiles for the largest products, with
// full bounds checks.
#include <limits.h>

#include <algorithm>

#include <type_traits>

#include "hero_device.h"
#include "hero_kernels.h"
#include "hero_rows.h"

namespace hero {
namespace {

constexpr int BK = 64;     // k elements per tile
constexpr int ROWB = 128;  // bytes of one row of a bf16 k-tile

template <typename T>
struct ARows {
  const T* base;
  const int* idx;  // null: identity
  int ld;
  // products of two terms (an epilogue with kTwoTerm): the operand from k-tile `turn` on, where B
  // starts over
  const T* base2 = nullptr;
  int turn = 0;
  __device__ __forceinline__ const T* row(int m) const {
    return base + static_cast<size_t>(idx ? idx[m] : m) * ld;
  }
};

// B rows: [0, split) from b0, [split, ...) from b1 (router: W_hd then psi_1);
// for the gate/up product b0 = W_g, b1 = W_u and rows are addressed by column.
template <typename T>
struct BRows {
  const T* b0;
  const T* b1;
  int split;
  int ld;
  __device__ __forceinline__ const T* row(int n) const {
    return n < split ? b0 + static_cast<size_t>(n) * ld : b1 + static_cast<size_t>(n - split) * ld;
  }
  __device__ __forceinline__ const T* gate_row(int c) const { return b0 + static_cast<size_t>(c) * ld; }
  __device__ __forceinline__ const T* up_row(int c) const { return b1 + static_cast<size_t>(c) * ld; }
};

// ---------------------------------------------------------------------------
// epilogues
// ---------------------------------------------------------------------------

struct EpiStoreF32 {  // P[m][n] = acc; the MFMA path's K-slice z writes out + z * split_stride
  float* out;
  int ld;
  size_t split_stride;
  struct Pre {};
  __device__ __forceinline__ Pre prep(int, int) const { return {}; }
  __device__ __forceinline__ void store(int m, int n, float v) const {
    out[static_cast<size_t>(m) * ld + n] = v;
  }
  __device__ __forceinline__ void emit8(const Pre&, int m, int n, const float* v) const {
    float* o = out + blockIdx.y * split_stride + static_cast<size_t>(m) * ld + n;
    *reinterpret_cast<f32x4*>(o) = *reinterpret_cast<const f32x4*>(v);
    *reinterpret_cast<f32x4*>(o + 4) = *reinterpret_cast<const f32x4*>(v + 4);
  }
};

// EpiStoreF32 of the router's product in a decode step, whose launch also holds the row pass:
// workgroups (x >= tile_blocks, y) take token (x - tile_blocks) gridDim.y + y
struct EpiStoreF32Rows : EpiStoreF32 {
  static constexpr bool kRows = true;
  int tile_blocks, T, d, j;
  const bf16_t *hbar, *prev1, *prev2, *norm_w;
  float eps_norm;
  float* rowstat;
  bf16_t* u;
};

template <typename T>
struct EpiSwiGLU {  // act[m][c] = SiLU(gate) * up
  T* act;
  int ld;
  __device__ __forceinline__ void store2(int m, int c, float g, float u) const {
    stf(act + static_cast<size_t>(m) * ld + c, siluf_(g) * u);
  }
  // eight finished bf16 values (the MFMA path forms SiLU(gate) * up while staging)
  __device__ __forceinline__ void emit_packed(int m, int c, u32x4 v) const {
    *reinterpret_cast<u32x4*>(act + static_cast<size_t>(m) * ld + c) = v;
  }
};

template <typename T>
struct EpiSiLU {  // hid[m][n] = SiLU(acc)
  T* out;
  int ld;
  __device__ __forceinline__ void store(int m, int n, float v) const {
    stf(out + static_cast<size_t>(m) * ld + n, siluf_(v));
  }
};

template <typename T>
struct EpiStore {  // out[m][n] = acc in the storage dtype
  T* out;
  int ld;
  struct Pre {};
  __device__ __forceinline__ Pre prep(int, int) const { return {}; }
  __device__ __forceinline__ void store(int m, int n, float v) const {
    stf(out + static_cast<size_t>(m) * ld + n, v);
  }
  __device__ __forceinline__ void emit8(const Pre&, int m, int n, const float* v) const {
    st8(out + static_cast<size_t>(m) * ld + n, v);
  }
};

// Backward of the gated SwiGLU branch, on the recomputed gate/up products G = u W_g^T,
// U = u W_u^T of FFN row m (token t = idx[m]), given e = dL/dy W_d at the same (m, c) with
// dL/dy = g_t dL/dh (e itself carries no g):
//   act = SiLU(G) U,  dL/dact = g_t e,
//   dG = g_t e U SiLU'(G),  dU = g_t e SiLU(G)   -> dgu[m][c], dgu[m][d_ff + c]
//   the row's share of dL/dg_t = <dL/dh_t, y_t> = <e_m, act_m> over the tile's columns
//                                                  -> dgpart[m][part]
// The MFMA path hands this epilogue the accumulators of a finished wave tile (dual); the
// fp32 path calls store2 per element with one partial per column.
template <typename T>
struct EpiSwiGLUBwd {
  const T* e;
  int ld_e;
  const int* idx;
  const float* gate;
  T* dgu;
  int ld_dgu;
  int d_ff;
  float* dgpart;
  int n_parts;
  static constexpr bool kDualHook = true;
  __device__ __forceinline__ void store2(int m, int c, float g, float u) const {
    const int t = idx ? idx[m] : m;
    const float gt = gate ? gate[t] : 1.0f;
    const float ev = ldf(e + static_cast<size_t>(m) * ld_e + c);
    const float sg = 1.0f / (1.0f + expf(-g));
    const float act = g * sg * u, dact = gt * ev;
    stf(dgu + static_cast<size_t>(m) * ld_dgu + c, dact * u * sg * (1.0f + g * (1.0f - sg)));
    stf(dgu + static_cast<size_t>(m) * ld_dgu + d_ff + c, dact * g * sg);
    dgpart[static_cast<size_t>(m) * n_parts + c] = ev * act;
  }
};

// h_out[t][n] = hbar[t][n] + scale(g_t) * acc, t = idx[m]; FFN scales by g, adapter by 1 - g.
// Without an index list t = m, and without gates the scale is 1 (a plain residual add: the
// dense FFN of a non-routed block, the attention output projection).
// The MFMA path fetches each 8-column piece of hbar (prep) before it stages the accumulators,
// so that the loads of a whole wave tile are in flight together.
template <typename T, bool ADAPTER>
struct EpiScatter {
  const int* idx;
  const T* hbar;
  const float* gate;
  T* out;
  int ld;
  __device__ __forceinline__ void store(int m, int n, float v) const {
    const int t = idx ? idx[m] : m;
    const float g = gate ? gate[t] : (ADAPTER ? 0.0f : 1.0f);
    const float sc = ADAPTER ? 1.0f - g : g;
    const size_t o = static_cast<size_t>(t) * ld + n;
    stf(out + o, ldf(hbar + o) + sc * v);
  }
  struct Pre {
    u32x4 h;
    uint32_t row;
    float sc;
  };
  __device__ __forceinline__ Pre prep(int m, int n) const {
    const int t = idx ? idx[m] : m;
    const float g = gate ? gate[t] : (ADAPTER ? 0.0f : 1.0f);
    Pre p;
    p.row = static_cast<uint32_t>(t);
    p.sc = ADAPTER ? 1.0f - g : g;
    p.h = *reinterpret_cast<const u32x4*>(hbar + static_cast<size_t>(t) * ld + n);
    return p;
  }
  __device__ __forceinline__ void emit8(const Pre& p, int, int n, const float* v) const {
    u32x4 w;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float lo = __uint_as_float(p.h[i] << 16) + p.sc * v[2 * i];
      const float hi = __uint_as_float(p.h[i] & 0xffff0000u) + p.sc * v[2 * i + 1];
      w[i] = static_cast<uint32_t>(f32_to_bf16(lo)) | (static_cast<uint32_t>(f32_to_bf16(hi)) << 16);
    }
    *reinterpret_cast<u32x4*>(out + static_cast<size_t>(p.row) * ld + n) = w;
  }
};

// ---------------------------------------------------------------------------
// bf16 MFMA GEMM
//
// One workgroup of WM x WN waves computes a BM x BN tile; each wave owns a
// (BM/WM) x (BN/WN) block of 32 x 32 MFMA tiles with fp32 accumulators.  The larger
// tiles run 8 waves (two per SIMD), so that one wave's MFMAs cover the other's waits.
// K advances in 64-deep tiles through two LDS stages (more where a tile names them):
//   * each stage is filled by wave-wide global_load_lds_dwordx4: one instruction
//     moves 64 x 16 bytes into a contiguous 1 KiB of LDS, i.e. eight 128-byte
//     tile rows; lane L lands in row 8b + L/8 at physical chunk L%8 and so loads
//     logical chunk (L%8) ^ ((row/2)%8) of that row.  The fragment reads undo the
//     XOR; with it, the 16 lanes of one LDS read phase (16 consecutive rows, one
//     logical chunk) hit 16 distinct 16-byte slots of the 256-byte bank window;
//   * within a k-tile the fragments of the next 16-deep k-step are read while the
//     MFMAs of the current one run (two register sets), the reads interleaved one
//     by one with the MFMAs;
//   * the workgroup barrier sits before the last k-step: by then every wave has
//     read the whole stage, so the loads of tile k+2 are issued into it, one per
//     MFMA of that last k-step, together with the first fragment reads of tile k+1.
// A grid with gridDim.y = S > 1 splits K: workgroup y covers k-tiles [y n / S, (y + 1) n / S)
// of the n = K / 64 and its epilogue writes partial sums to a slice of its own (router
// pre-activations; gate/up with few rows).
// Epilogues first fetch what they combine with (hbar rows) for the whole wave tile,
// then stage fp32 results in 32-row blocks.
// ---------------------------------------------------------------------------

typedef __attribute__((address_space(3))) void lds_void;

__device__ __forceinline__ void load_lds16(const void* g, unsigned char* l) {
  __builtin_amdgcn_global_load_lds(g, (lds_void*)(l), 16, 0, 0);
}

__device__ __forceinline__ int swz(int row, int ch) { return row * ROWB + ((ch ^ ((row >> 1) & 7)) << 4); }

constexpr int GROUP_M = 8;   // row tiles per group of the tile order
constexpr int kCUs = 256;    // compute units of an MI355X

// instruction classes of __builtin_amdgcn_sched_group_barrier
constexpr int SG_MFMA = 0x008, SG_VMEM_READ = 0x020, SG_DS_READ = 0x100;

// An epilogue with kRows brings the row pass of a decode step along (EpiStoreF32Rows)
template <class E, class = void>
struct RowsHook : std::false_type {};
template <class E>
struct RowsHook<E, std::void_t<decltype(E::kRows)>> : std::true_type {};

// NS_: LDS stages of the k-loop; the loads of tile k + NS - 1 are in flight while tile k is
// consumed (2 where the operands sit in L2, more where streaming weights from HBM needs more bytes
// in flight per CU).
template <int BM_, int BN_, int WM_, int WN_, int NS_ = 2>
struct Tile {
  static constexpr int BM = BM_, BN = BN_, WM = WM_, WN = WN_;
  static constexpr int NS = NS_;
  static constexpr int KSTEP = 16;                    // k per MFMA
  static constexpr int NT = 64 * WM * WN;
  static constexpr int NW = WM * WN;
  static constexpr int WTM = BM / WM, WTN = BN / WN;
  static constexpr int TM = WTM / 32, TN = WTN / 32;
  static constexpr int STAGE = (BM + BN) * ROWB;
  static constexpr int OUT_N = BN;                    // output columns per tile
  static constexpr int OPAD = WTN + 4;                // fp32 staging row pitch (floats)
  static_assert(WTM % 32 == 0 && WTN % 32 == 0, "wave tile must be whole MFMA tiles");
  static_assert(BM % (8 * NW) == 0 && BN % (8 * NW) == 0, "loader split");
  static_assert(NW * 32 * OPAD * 4 <= 2 * STAGE, "epilogue staging must fit in the stages");
  static_assert((32 * (WTN / 8)) % 64 == 0, "epilogue pieces split evenly over the lanes");
  static_assert(NS >= 2 && NS * STAGE <= 160 * 1024, "stages fit in LDS");
};

// Lane layout of the two matrix instructions (wave64).  Operands: lane l holds 8 consecutive k of
// row (l mod MI) of its 16 x 32 (MI 16) or 32 x 16 (MI 32) block, at k-chunk l / MI.  Result:
// element r of lane l is row 4 (l / 16) + r (MI 16) or out_row32(r, l) (MI 32), column l mod MI.
__device__ __forceinline__ int out_row32(int r, int lane) { return 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3); }
template <int MI>
__device__ __forceinline__ int in_chunk(int ks, int lane) {   // 16-byte chunk of a 128-byte row
  if constexpr (MI == 32)
    return 2 * ks + (lane >> 5);
  else
    return 4 * ks + (lane >> 4);
}
__device__ __forceinline__ f32x16 mfma_op(bf16x8 a, bf16x8 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ f32x4 mfma_op(bf16x8 a, bf16x8 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// s_waitcnt vmcnt(N) lgkmcnt(0) for a compile-time N
template <int N>
__device__ __forceinline__ void wait_vm_lgkm() {
  static_assert(N >= 0 && N < 64, "vmcnt range");
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(N) : "memory");
}

template <class C, class Epi>
__global__ __launch_bounds__(C::NT) void mfma_gemm(ARows<bf16_t> A, BRows<bf16_t> B, Epi epi,
                                                  const int* __restrict__ m_count, int M_fixed,
                                                  int K, int mt_max, int n_tiles) {
  constexpr int NW = C::NW;
  constexpr int A_LD = C::BM / 8 / NW;  // wave-wide loads per k-tile, A
  constexpr int B_LD = C::BN / 8 / NW;
  constexpr int KS = BK / C::KSTEP;     // k-steps per k-tile
  constexpr int MI = 32;
  constexpr int NM = C::TM * C::TN;     // MFMAs per k-step
  constexpr int NR = C::TM + C::TN;     // fragment reads per k-step
  constexpr int NL = A_LD + B_LD;       // stage loads per k-tile
  __shared__ __attribute__((aligned(1024))) unsigned char smem[C::NS * C::STAGE];
  if constexpr (RowsHook<Epi>::value) {
    static_assert(C::NT == 256, "the row pass takes 256 threads a token");
    if (static_cast<int>(blockIdx.x) >= epi.tile_blocks) {
      const int t = (static_cast<int>(blockIdx.x) - epi.tile_blocks) * static_cast<int>(gridDim.y) +
                    static_cast<int>(blockIdx.y);
      if (t < epi.T)
        rowstats_row<bf16_t>(t, epi.T, epi.hbar, epi.prev1, epi.prev2, epi.norm_w, epi.d, epi.j, epi.eps_norm,
                                    epi.rowstat, epi.u);
      return;
    }
  }
  // Workgroups go to the 8 XCDs round-robin; XCD x takes the contiguous range
  // [x per, (x+1) per) of a grouped tile order (GROUP_M row tiles by every column tile),
  // so that the 32 tiles one XCD runs at a time share 8 row panels and 4 column panels
  // in its L2.
  // The grid is sized for M_fixed rows; the order is laid over the rows that exist (the device
  // count), so that every XCD gets an equal share however few rows there are.
  const int M = m_count ? *m_count : M_fixed;
  const int mt_act = min(mt_max, (M + C::BM - 1) / C::BM);
  const int per = (mt_act * n_tiles + 7) >> 3;
  const int q = blockIdx.x >> 3;
  if (q >= per) return;
  const int tile = (blockIdx.x & 7) * per + q;
  if (tile >= mt_act * n_tiles) return;
  const int grp = tile / (GROUP_M * n_tiles), rem = tile % (GROUP_M * n_tiles);
  const int gsz = min(GROUP_M, mt_act - grp * GROUP_M);
  const int mt = grp * GROUP_M + rem % gsz, nt = rem / gsz;
  const int m0 = mt * C::BM;
  // split K: workgroup y covers k-tiles [y nkt / S, (y+1) nkt / S) (S = gridDim.y <= nkt)
  const int nkt = K / BK;
  const int kt0 = static_cast<int>(blockIdx.y) * nkt / static_cast<int>(gridDim.y);
  const int kt1 = (static_cast<int>(blockIdx.y) + 1) * nkt / static_cast<int>(gridDim.y);

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) >> 6);
  const int wm = wave / C::WN, wn = wave % C::WN;
  const int rsub = lane >> 3;

  const unsigned char* a_base = reinterpret_cast<const unsigned char*>(A.base);
  uint32_t a_off[A_LD];
#pragma unroll
  for (int i = 0; i < A_LD; ++i) {
    const int r = 8 * (i * NW + wave) + rsub;
    const int ch = (lane & 7) ^ ((r >> 1) & 7);
    const int m = min(m0 + r, M - 1);
    const int row = A.idx ? A.idx[m] : m;
    a_off[i] = static_cast<uint32_t>(row) * static_cast<uint32_t>(A.ld * 2) + ch * 16;
  }
  const unsigned char* b_base[B_LD];
  uint32_t b_off[B_LD];
#pragma unroll
  for (int i = 0; i < B_LD; ++i) {
    const int blk = i * NW + wave;  // 8-row block, wave-uniform
    const int r = 8 * blk + rsub;
    const int ch = (lane & 7) ^ ((r >> 1) & 7);
    const bool second = nt * C::BN + 8 * blk >= B.split;
    const bf16_t* base = second ? B.b1 : B.b0;
    const int row = nt * C::BN + r - (second ? B.split : 0);
    b_base[i] = reinterpret_cast<const unsigned char*>(base);
    b_off[i] = static_cast<uint32_t>(row) * static_cast<uint32_t>(B.ld * 2) + ch * 16;
  }

  auto issue = [&](int stage, int k0) {
    unsigned char* sa = smem + stage * C::STAGE;
    const uint32_t kb = static_cast<uint32_t>(k0 + kt0 * BK) * 2;
#pragma unroll
    for (int i = 0; i < A_LD; ++i) load_lds16(a_base + a_off[i] + kb, sa + (i * NW + wave) * 1024);
#pragma unroll
    for (int i = 0; i < B_LD; ++i)
      load_lds16(b_base[i] + b_off[i] + kb, sa + C::BM * ROWB + (i * NW + wave) * 1024);
  };

  f32x16 acc[C::TM][C::TN];
#pragma unroll
  for (int a = 0; a < C::TM; ++a)
#pragma unroll
    for (int b = 0; b < C::TN; ++b)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[a][b][r] = 0.f;

  int fa_row[C::TM], fb_row[C::TN];
#pragma unroll
  for (int a = 0; a < C::TM; ++a) fa_row[a] = wm * C::WTM + a * MI + (lane & (MI - 1));
#pragma unroll
  for (int b = 0; b < C::TN; ++b) fb_row[b] = C::BM + wn * C::WTN + b * MI + (lane & (MI - 1));
  bf16x8 fa[2][C::TM], fb[2][C::TN];
  auto read_frags = [&](int buf, const unsigned char* st, int ks) {
    const int c = in_chunk<MI>(ks, lane);
#pragma unroll
    for (int a = 0; a < C::TM; ++a) fa[buf][a] = *reinterpret_cast<const bf16x8*>(st + swz(fa_row[a], c));
#pragma unroll
    for (int b = 0; b < C::TN; ++b) fb[buf][b] = *reinterpret_cast<const bf16x8*>(st + swz(fb_row[b], c));
  };
  auto mfmas = [&](int buf) {
#pragma unroll
    for (int a = 0; a < C::TM; ++a)
#pragma unroll
      for (int b = 0; b < C::TN; ++b)
        acc[a][b] = mfma_op(fa[buf][a], fb[buf][b], acc[a][b]);
  };
  // order within the current scheduling region: MFMA, then (while any remain) one stage load
  // and one fragment read after each
  auto interleave = [&](auto nl_, auto nr_) {
    constexpr int nl = decltype(nl_)::value, nr = decltype(nr_)::value;
#pragma unroll
    for (int i = 0; i < NM; ++i) {
      __builtin_amdgcn_sched_group_barrier(SG_MFMA, 1, 0);
      if (i < nl) __builtin_amdgcn_sched_group_barrier(SG_VMEM_READ, 1, 0);
      if (i < nr) __builtin_amdgcn_sched_group_barrier(SG_DS_READ, 1, 0);
    }
    if constexpr (nl > NM) __builtin_amdgcn_sched_group_barrier(SG_VMEM_READ, nl - NM, 0);
    if constexpr (nr > NM) __builtin_amdgcn_sched_group_barrier(SG_DS_READ, nr - NM, 0);
  };

  const int nk = kt1 - kt0;
  constexpr int NS = C::NS;
  // One k-tile.  MODE 2 (steady state): the loads of tile kt + NS go into the stage just
  // consumed and the first fragments of tile kt + 1 are read, both interleaved with the MFMAs
  // of the last k-step; MODE 1: no tile left to load; MODE 0: the last tile.  Each mode is its
  // own straight-line code, so that the scheduler can interleave the loads with the MFMAs
  // (a load under a run-time condition would sit in a block of its own and issue as a burst).
  auto ktile = [&](int kt, auto mode_) {
    constexpr int mode = decltype(mode_)::value;
    const unsigned char* st = smem + (kt % NS) * C::STAGE;
#pragma unroll
    for (int ks = 0; ks < KS - 1; ++ks) {
      read_frags((ks + 1) & 1, st, ks + 1);
      mfmas(ks & 1);
      interleave(std::integral_constant<int, 0>(), std::integral_constant<int, NR>());
      __builtin_amdgcn_sched_barrier(0);
    }
    // every wave has read all of stage kt and the loads of tile kt+1 have landed (tiles
    // kt+2 .. kt+NS-1 may still be in flight; near the end, fewer were issued)
    if constexpr (mode == 2)
      wait_vm_lgkm<(NS - 2) * NL>();
    else
      wait_vm_lgkm<0>();
    __syncthreads();
    if constexpr (mode == 2) issue(kt % NS, (kt + NS) * BK);
    if constexpr (mode >= 1) read_frags(KS & 1, smem + ((kt + 1) % NS) * C::STAGE, 0);
    mfmas((KS - 1) & 1);
    interleave(std::integral_constant<int, mode == 2 ? NL : 0>(), std::integral_constant<int, mode >= 1 ? NR : 0>());
    __builtin_amdgcn_sched_barrier(0);
  };

  // tiles 0 .. NS-1 into the NS stages; wait for tile 0 (the others may still be landing)
#pragma unroll
  for (int i = 0; i < NS; ++i)
    if (i < nk) issue(i, i * BK);
  if (nk >= NS)
    wait_vm_lgkm<(NS - 1) * NL>();
  else
    wait_vm_lgkm<0>();
  __syncthreads();
  read_frags(0, smem, 0);
  int kt = 0;
  for (; kt + NS < nk; ++kt) ktile(kt, std::integral_constant<int, 2>());
  for (; kt + 1 < nk; ++kt) ktile(kt, std::integral_constant<int, 1>());
  if (kt < nk) ktile(kt, std::integral_constant<int, 0>());

  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  constexpr int CPR = C::WTN / 8;                 // 8-column pieces per staged row
  constexpr int PPB = 32 * CPR / kWave;           // pieces per lane per 32-row block
  // what the epilogue combines with (hbar rows) is fetched for the whole wave tile ahead of the
  // staging, so those loads are in flight together
  typename Epi::Pre pre[C::TM][PPB];
#pragma unroll
  for (int a = 0; a < C::TM; ++a)
#pragma unroll
    for (int q = 0; q < PPB; ++q) {
      const int e = lane + kWave * q;
      const int m = m0 + wm * C::WTM + a * 32 + e / CPR;
      pre[a][q] = epi.prep(min(m, M - 1), nt * C::OUT_N + wn * C::WTN + (e % CPR) * 8);
    }
  float* stg = reinterpret_cast<float*>(smem) + wave * (32 * C::OPAD);
#pragma unroll
  for (int a = 0; a < C::TM; ++a) {
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int i = out_row32(r, lane);
#pragma unroll
      for (int b = 0; b < C::TN; ++b) stg[i * C::OPAD + b * 32 + (lane & 31)] = acc[a][b][r];
    }
#pragma unroll
    for (int q = 0; q < PPB; ++q) {
      const int e = lane + kWave * q;
      const int i = e / CPR, c8 = (e % CPR) * 8;
      const int m = m0 + wm * C::WTM + a * 32 + i;
      if (m < M) epi.emit8(pre[a][q], m, nt * C::OUT_N + wn * C::WTN + c8, stg + i * C::OPAD + c8);
    }
  }
}

// ---------------------------------------------------------------------------
// The large bf16 products: BM x 256 tiles (BM 256, 192 or 128) on v_mfma_f32_16x16x32_bf16, eight
// waves, two per SIMD, each with two 16 HM-row by two 32-column blocks: rows from either half of
// the A tile, columns from either half of the B tile (the gate/up product: W_g, then W_u).
//   * A k-tile is four products of a half by a half.  Each half is read from LDS into registers
//     one product ahead, so a half of a stage is free again half a k-tile after its k-tile began,
//     and its loads for k-tile kt + 2 are issued then: they have one to one and a half k-tiles to
//     land (half a k-tile to one with whole stages), and the waits leave the loads of one k-tile in
//     flight (8, 7 and 6 a wave at 256, 192 and 128 rows).  Two barriers a k-tile.
//   * The loads write the LDS that the fragment reads read, so the compiler keeps their order:
//     they are written in the order they shall issue in, one between two MFMAs.  Issued as a burst
//     ahead of the reads (the order of the source before), the same loop lost all of its gain.
//   * The 16 x 16 x 32 instruction: at the same nominal rate as 32 x 32 x 16 it sustains a higher
//     clock on random data under the board's power limit.
// What bounds it: the matrix cores are busy for 75 % of its cycles (counters of the 8B stack's
// gate/up and down; the loop with whole stages 67 %), at the clock that the power limit leaves on
// random operands, 1.7-1.8 GHz.  A register-only loop of the same instruction has 91-94 % at 1.87 GHz
// (on zeros 96 % at 2.32).  The other quarter is waiting, at the two barriers and for loads and fragments (25 %
// of the waves' time); the fragment reads take 29 % of the LDS's cycles, bank conflicts 0.3 %.  4096 rows of the
// Llama-3.1-8B gate/up product: 1.84 PFLOP/s on zeros (whole stages 1.57), 1.44 on random operands
// (1.38); 20047 rows 3510 -> 3390 us, its down product 1845 -> 1760 us, 2995 rows on 192-row tiles
// 550 -> 525 and 265 -> 257 us.  Four waves of 128 x 128 (a third fewer LDS reads) reached 1.39.
// Epilogues: the gate/up products finish in registers and stage bf16; the others stage 16-row
// blocks in fp32 and take 8-column pieces (emit8) or the whole block (block).
// A grid with gridDim.y = S > 1 splits K as mfma_gemm does.
// ---------------------------------------------------------------------------

// An epilogue with a block() member takes each staged block of 16 rows whole, instead of 8-column
// row pieces through emit8().
template <class E, class = void>
struct BlockEpilogue : std::false_type {};
template <class E>
struct BlockEpilogue<E, std::void_t<decltype(&E::block)>> : std::true_type {};
// A two-product epilogue with kDualHook takes the accumulators of a finished wave tile itself (the
// backward of the gated SwiGLU) instead of the forward's SiLU(gate) * up staging.
template <class E, class = void>
struct DualHook : std::false_type {};
template <class E>
struct DualHook<E, std::void_t<decltype(E::kDualHook)>> : std::true_type {};

// An epilogue with kTwoTerm ends a product of two terms, A B^T + A2 B^T (ARows::base2)
template <class E, class = void>
struct TwoTerm : std::false_type {};
template <class E>
struct TwoTerm<E, std::void_t<decltype(E::kTwoTerm)>> : std::true_type {};

template <int BM_, bool DUAL_>
struct Phase {
  static constexpr int WN = 4, NW = 8, NT = 512;
  static constexpr int HB = 2;                  // 16-column fragments per wave and half
  static constexpr int BM = BM_, BN = 256;
  static constexpr bool DUAL = DUAL_;
  static constexpr int HM = BM / 64;            // 16-row fragments per wave and half
  static constexpr int STAGE = (BM + BN) * ROWB;
  static constexpr int OUT_N = DUAL ? 128 : 256;
  static constexpr int A_LD = BM / 8 / NW;      // 1 KiB stage loads per wave: A
  static constexpr int A1 = BM / 16 / NW;       // ... of the first half alone
  static constexpr int BH = 16 / NW;            // ... of half of B
  static constexpr int L1 = A1 + BH, L2 = A_LD - A1 + BH;
  static constexpr int SPLIT = A_LD % 2;        // loads of the second group that the first half needs too
  static constexpr int ON = 32;                 // output columns per wave and half
};

template <class C, class Epi>
__device__ __forceinline__ void swiglu_bwd_tile(const Epi& epi, f32x4 (&acc)[2 * C::HM][4], unsigned char* smem, int m0,
                                                int nt, int wave, int wm, int wn, int M, int lane);

template <class C, class Epi>
__device__ __forceinline__ void phase_tile(const ARows<bf16_t>& A, const BRows<bf16_t>& B, const Epi& epi, int M,
                                           int M_max, int K, int n_tiles, unsigned char* smem) {
  constexpr int BM = C::BM, HM = C::HM, HB = C::HB, NW = C::NW, BH = C::BH;
  const int mt_max = (M_max + BM - 1) / BM;
  const int mt_act = min(mt_max, (M + BM - 1) / BM);
  const int per = (mt_act * n_tiles + 7) >> 3;
  const int q = blockIdx.x >> 3;
  if (q >= per) return;
  const int tile = (blockIdx.x & 7) * per + q;
  if (tile >= mt_act * n_tiles) return;
  const int grp = tile / (GROUP_M * n_tiles), rem = tile % (GROUP_M * n_tiles);
  const int gsz = min(GROUP_M, mt_act - grp * GROUP_M);
  const int mt = grp * GROUP_M + rem % gsz, nt = rem / gsz;
  const int m0 = mt * BM;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) >> 6);
  const int wm = wave / C::WN, wn = wave % C::WN;
  const int rsub = lane >> 3;

  const unsigned char* a_base = reinterpret_cast<const unsigned char*>(A.base);
  uint32_t a_off[C::A_LD], b_off[2 * BH];
#pragma unroll
  for (int i = 0; i < C::A_LD; ++i) {
    const int r = 8 * (i * NW + wave) + rsub;
    const int ch = (lane & 7) ^ ((r >> 1) & 7);
    const int m = min(m0 + r, M - 1);
    const int row = A.idx ? A.idx[m] : m;
    a_off[i] = static_cast<uint32_t>(row) * static_cast<uint32_t>(A.ld * 2) + ch * 16;
  }
  const unsigned char* b_base[2 * BH];
#pragma unroll
  for (int i = 0; i < 2 * BH; ++i) {
    const int blk = 8 * (i * NW + wave);   // first of eight rows, wave-uniform
    const int r = blk + rsub;
    const int ch = (lane & 7) ^ ((r >> 1) & 7);
    const bool second = C::DUAL ? blk >= 128 : nt * 256 + blk >= B.split;
    const int row = C::DUAL ? nt * 128 + (r & 127) : nt * 256 + r - (second ? B.split : 0);
    b_base[i] = reinterpret_cast<const unsigned char*>(second ? B.b1 : B.b0);
    b_off[i] = static_cast<uint32_t>(row) * static_cast<uint32_t>(B.ld * 2) + ch * 16;
  }
  // split K: workgroup y covers k-tiles [y nkt / S, (y + 1) nkt / S), at least two
  const int nkt = K / BK;
  const int kt0 = static_cast<int>(blockIdx.y) * nkt / static_cast<int>(gridDim.y);
  const int nk = (static_cast<int>(blockIdx.y) + 1) * nkt / static_cast<int>(gridDim.y) - kt0;
  const unsigned char* a_base2 = reinterpret_cast<const unsigned char*>(A.base2);
  // i-th load of the wave, k-tile kt of the slice
  auto ldA = [&](int i, int kt) {
    const int k = kt0 + kt;
    const bool two = TwoTerm<Epi>::value && k >= A.turn;
    const unsigned char* base = (two ? a_base2 : a_base) + static_cast<uint32_t>(two ? k - A.turn : k) * ROWB;
    load_lds16(base + a_off[i], smem + (kt & 1) * C::STAGE + (i * NW + wave) * 1024);
  };
  auto ldB = [&](int i, int kt) {
    const int k = kt0 + kt;
    const bool two = TwoTerm<Epi>::value && k >= A.turn;
    const unsigned char* base = b_base[i] + static_cast<uint32_t>(two ? k - A.turn : k) * ROWB;
    load_lds16(base + b_off[i], smem + (kt & 1) * C::STAGE + BM * ROWB + (i * NW + wave) * 1024);
  };
  // group 1: the first half of A and B; group 2: the rest (the piece of A that both halves share first)
  auto ld1 = [&](int i, int kt) { i < C::A1 ? ldA(i, kt) : ldB(i - C::A1, kt); };
  auto ld2 = [&](int i, int kt) {
    i < C::A_LD - C::A1 ? ldA(C::A1 + i, kt) : ldB(BH + i - (C::A_LD - C::A1), kt);
  };

  f32x4 acc[2 * HM][2 * HB];
#pragma unroll
  for (int a = 0; a < 2 * HM; ++a)
#pragma unroll
    for (int b = 0; b < 2 * HB; ++b) acc[a][b] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int l15 = lane & 15;
  bf16x8 fa0[HM][2], fa1[HM][2], fb0[HB][2], fb1[HB][2];
  // fragment addresses: the chunk swizzle only depends on the lane (the blocks start at multiples of
  // 16 rows), so a fragment is a constant away from one of four addresses in the stage
  uint32_t offA[2], offB[2];
#pragma unroll
  for (int ks = 0; ks < 2; ++ks) {
    offA[ks] = swz(wm * (BM / 4) + l15, in_chunk<16>(ks, lane));
    offB[ks] = BM * ROWB + swz(wn * 16 * HB + l15, in_chunk<16>(ks, lane));
  }
  auto rdA = [&](bf16x8 (&f)[HM][2], const unsigned char* st, int half, int i) {
    const int ks = i / HM, a = i % HM;
    f[a][ks] = *reinterpret_cast<const bf16x8*>(st + offA[ks] + (half * (BM / 2) + 16 * a) * ROWB);
  };
  auto rdB = [&](bf16x8 (&f)[HB][2], const unsigned char* st, int half, int i) {
    const int ks = i / HB, b = i % HB;
    f[b][ks] = *reinterpret_cast<const bf16x8*>(st + offB[ks] + (half * 128 + 16 * b) * ROWB);
  };
  auto mm = [&](const bf16x8 (&fa)[HM][2], const bf16x8 (&fb)[HB][2], int ha, int hb) {
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
      for (int a = 0; a < HM; ++a)
#pragma unroll
        for (int b = 0; b < HB; ++b)
          acc[ha * HM + a][hb * HB + b] = mfma_op(fa[a][ks], fb[b][ks], acc[ha * HM + a][hb * HB + b]);
  };
  // The memory operations of a phase in program order: a stage load after every EV-th fragment read (the
  // compiler keeps their order, as the loads write the LDS that the reads read), and the
  // schedule: one of them after each MFMA.
  auto mem = [&](auto nr_, auto nl_, auto ev_, auto rd, auto ld) {
    constexpr int nr = decltype(nr_)::value, nl = decltype(nl_)::value, ev = decltype(ev_)::value;
    int l = 0;
#pragma unroll
    for (int i = 0; i < nr; ++i) {
      rd(i);
      if (i % ev == ev - 1 && l < nl) ld(l++);
    }
#pragma unroll
    for (int i = 0; i < nl; ++i)
      if (i >= l) ld(i);
  };
  auto weave = [&](auto nm_, auto nr_, auto nl_, auto ev_) {
    constexpr int nm = decltype(nm_)::value, nl = decltype(nl_)::value, nr = decltype(nr_)::value,
                  ev = decltype(ev_)::value;
    int r = 0, l = 0;
#pragma unroll
    for (int i = 0; i < nm; ++i) {
      __builtin_amdgcn_sched_group_barrier(SG_MFMA, 1, 0);
      if (r < nr) {
        __builtin_amdgcn_sched_group_barrier(SG_DS_READ, 1, 0);
        ++r;
        if (r % ev == 0 && l < nl) {
          __builtin_amdgcn_sched_group_barrier(SG_VMEM_READ, 1, 0);
          ++l;
        }
      } else if (l < nl) {
        __builtin_amdgcn_sched_group_barrier(SG_VMEM_READ, 1, 0);
        ++l;
      }
    }
    __builtin_amdgcn_sched_barrier(0);
  };
#define IC(n) std::integral_constant<int, (n)>()
  constexpr int L1 = C::L1, L2 = C::L2, SP = C::SPLIT, NM = 2 * HM * HB;
  // MODE 2: tile kt + 2 is loaded; 1: the last but one; 0: the last
  auto ktile = [&](int kt, auto mode_) {
    constexpr int mode = decltype(mode_)::value;
    const unsigned char* st = smem + (kt & 1) * C::STAGE;
    const unsigned char* nx = smem + ((kt + 1) & 1) * C::STAGE;
    wait_vm_lgkm<mode == 0 ? 0 : L1 + L2>();
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    mem(IC(2 * HB + 2 * HM), IC(mode == 2 ? L1 : 0), IC(2),
        [&](int i) { i < 2 * HB ? rdB(fb1, st, 1, i) : rdA(fa1, st, 1, i - 2 * HB); }, [&](int i) { ld1(i, kt + 2); });
    mm(fa0, fb0, 0, 0);
    weave(IC(NM), IC(2 * HB + 2 * HM), IC(mode == 2 ? L1 : 0), IC(2));
    mm(fa0, fb1, 0, 1);
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (mode != 0) {
      wait_vm_lgkm<(mode == 2 ? L1 + L2 : L2) - SP>();
      __builtin_amdgcn_s_barrier();
      __builtin_amdgcn_sched_barrier(0);
      mem(IC(2 * HM), IC(mode == 2 ? L2 : 0), IC(1), [&](int i) { rdA(fa0, nx, 0, i); }, [&](int i) { ld2(i, kt + 2); });
    }
    mm(fa1, fb0, 1, 0);
    weave(IC(NM), IC(mode ? 2 * HM : 0), IC(mode == 2 ? L2 : 0), IC(1));
    if constexpr (mode != 0)
#pragma unroll
      for (int i = 0; i < 2 * HB; ++i) rdB(fb0, nx, 0, i);
    mm(fa1, fb1, 1, 1);
    weave(IC(NM), IC(mode ? 2 * HB : 0), IC(0), IC(1));
  };
#pragma unroll
  for (int t = 0; t < 2; ++t) {
#pragma unroll
    for (int i = 0; i < L1; ++i) ld1(i, t);
#pragma unroll
    for (int i = 0; i < L2; ++i) ld2(i, t);
  }
  wait_vm_lgkm<L1 + 2 * L2 - SP>();
  __builtin_amdgcn_s_barrier();
#pragma unroll
  for (int i = 0; i < 2 * HM; ++i) rdA(fa0, smem, 0, i);
#pragma unroll
  for (int i = 0; i < 2 * HB; ++i) rdB(fb0, smem, 0, i);
  int kt = 0;
  for (; kt + 2 < nk; ++kt) ktile(kt, IC(2));
  ktile(kt, IC(1));
  ktile(kt + 1, IC(0));
#undef IC
  asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
  __builtin_amdgcn_s_barrier();

  if constexpr (DualHook<Epi>::value) {
    swiglu_bwd_tile<C>(epi, acc, smem, m0, nt, wave, wm, wn, M, lane);
  } else if constexpr (C::DUAL) {
    // rows of half h: m0 + h BM/2 + wm BM/4 + ..; the wave's 32 columns of act, gate in acc[.][0..1], up in [2..3]
    constexpr int ON = 16 * HB, SP2 = ON + 8, CPR = ON / 8;
    bf16_t* stg = reinterpret_cast<bf16_t*>(smem) + wave * (32 * HM * SP2);
#pragma unroll
    for (int a = 0; a < 2 * HM; ++a)
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int b = 0; b < HB; ++b) {
          const float g = acc[a][b][r], u = acc[a][HB + b][r];
          stg[(16 * a + 4 * (lane >> 4) + r) * SP2 + 16 * b + l15] =
              f32_to_bf16(g * __builtin_amdgcn_rcpf(1.0f + __expf(-g)) * u);
        }
#pragma unroll
    for (int p = 0; p < 2 * HM * 16 * CPR / kWave; ++p) {
      const int e = lane + kWave * p, i = e / CPR, c8 = (e % CPR) * 8;
      const int h = i / (16 * HM), m = m0 + h * (BM / 2) + wm * (BM / 4) + i - h * 16 * HM;
      const u32x4 v = *reinterpret_cast<const u32x4*>(stg + i * SP2 + c8);
      if (m < M) epi.emit_packed(m, nt * 128 + wn * ON + c8, v);
    }
  } else {
    // per half of B: 32 columns; 16-row blocks staged as fp32
    constexpr int ON = 16 * HB, OP = 2 * ON + 4, CPR = ON / 4, PP = 16 * CPR / kWave;
    float* stg = reinterpret_cast<float*>(smem) + wave * (16 * OP);
    typename Epi::Pre pre[2 * HM][PP];
    // rows of fragment a, columns of the staged pair of 32-column blocks
    auto row_of = [&](int a, int i) { return m0 + (a / HM) * (BM / 2) + wm * (BM / 4) + 16 * (a % HM) + i; };
    auto col_of = [&](int c8) { return nt * 256 + (c8 / ON) * 128 + wn * ON + c8 % ON; };
    auto fetch = [&](int a) {
#pragma unroll
      for (int p = 0; p < PP; ++p) {
        const int e = lane + kWave * p;
        pre[a][p] = epi.prep(min(row_of(a, e / CPR), M - 1), col_of((e % CPR) * 8));
      }
    };
    // what the epilogue combines with (hbar rows) is fetched some fragments ahead of the staging
    constexpr int AHEAD = TwoTerm<Epi>::value ? 2 : 4;
#pragma unroll
    for (int a = 0; a < AHEAD; ++a) fetch(a);
#pragma unroll
    for (int a = 0; a < 2 * HM; ++a) {
      if (a + AHEAD < 2 * HM) fetch(a + AHEAD);
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int b = 0; b < 2 * HB; ++b) stg[(4 * (lane >> 4) + r) * OP + 16 * b + l15] = acc[a][b][r];
      if constexpr (BlockEpilogue<Epi>::value) {
        epi.block(stg, OP, ON, row_of(a, 0), col_of(0), M, lane);
        epi.block(stg + ON, OP, ON, row_of(a, 0), col_of(ON), M, lane);
      } else {
#pragma unroll
        for (int p = 0; p < PP; ++p) {
          const int e = lane + kWave * p, i = e / CPR, c8 = (e % CPR) * 8;
          const int m = row_of(a, i);
          if (m < M) epi.emit8(pre[a][p], m, col_of(c8), stg + i * OP + c8);
        }
      }
    }
  }
}


template <class C, class Epi>
__global__ __launch_bounds__(512, 2) void phase_gemm(ARows<bf16_t> A, BRows<bf16_t> B, Epi epi,
                                                     const int* __restrict__ m_count, int M_max, int K, int n_tiles) {
  __shared__ __attribute__((aligned(1024))) unsigned char smem[2 * C::STAGE];
  phase_tile<C>(A, B, epi, m_count ? *m_count : M_max, M_max, K, n_tiles, smem);
}

// Tile height for M rows: the launch's time in rounds of workgroups over the CUs, times the
// relative duration of a round (measured on the Llama-3.1-8B gate/up and down shapes at 0.4k to 20k
// rows: 54-57, 78 and 97 us for 128-, 192- and 256-row tiles at K = 4096; 187, 258 and 345 at
// 14336).  The smaller tiles move more bytes per product and only pay while their finer rounds
// leave fewer CUs idle, so beyond four (128) and eight (192) rounds they are not considered.
// SPILL: the epilogues of the two backwards, whose 256-row tiles spill 96 and 36 registers and so are
// hardly faster a row than 192-row ones.  With the weights above against these, whole calls at the 8B shape:
// block backward 1135 -> 1085 us at 2800 tokens, 5768 -> 5511 at 16000, router backward 1010 -> 962 at
// 8192; 256 rows stay where they make a single round (block backward of 700 tokens: 626, on 128 rows 636).
template <bool SPILL>
__host__ __device__ inline int phase_rows(int M, int n_tiles) {
  auto tiles = [&](int BM) { return (M + BM - 1) / BM * n_tiles; };
  auto cost = [&](int BM, int w) { return (tiles(BM) + kCUs - 1) / kCUs * w; };
  int best = 256, c = cost(256, SPILL ? 152 : 125);
  if ((SPILL || tiles(192) <= 8 * kCUs) && cost(192, 100) < c) {
    best = 192;
    c = cost(192, 100);
  }
  if (tiles(128) <= 4 * kCUs && cost(128, SPILL ? 80 : 75) < c) best = 128;
  return best;
}
template <class Epi>
constexpr bool kSpill = DualHook<Epi>::value || TwoTerm<Epi>::value;

// Threshold routing: the host only knows an upper bound of the row count, so the workgroups choose
// the tile height themselves from the count on the device.
template <bool DUAL, class Epi>
__global__ __launch_bounds__(512, 2) void phase_gemm_any(ARows<bf16_t> A, BRows<bf16_t> B, Epi epi,
                                                         const int* __restrict__ m_count, int M_max, int K,
                                                         int n_tiles) {
  __shared__ __attribute__((aligned(1024))) unsigned char smem[2 * Phase<256, DUAL>::STAGE];
  const int M = min(*m_count, M_max);
  const int bm = phase_rows<kSpill<Epi>>(M, n_tiles);
  if (bm == 256)
    phase_tile<Phase<256, DUAL>>(A, B, epi, M, M_max, K, n_tiles, smem);
  else if (bm == 192)
    phase_tile<Phase<192, DUAL>>(A, B, epi, M, M_max, K, n_tiles, smem);
  else
    phase_tile<Phase<128, DUAL>>(A, B, epi, M, M_max, K, n_tiles, smem);
}

// exact: M_max is the row count (m_count, if given, holds at most that)
template <bool DUAL, class Epi>
hipError_t run_phase(ARows<bf16_t> A, BRows<bf16_t> B, Epi epi, const int* m_count, int M_max, int N_out, int K,
                     hipStream_t s, bool exact = true) {
  const int n_tiles = N_out / Phase<256, DUAL>::OUT_N;
  if (M_max <= 0 || n_tiles <= 0) return hipSuccess;
  const auto blocks = [&](int BM) { return ((M_max + BM - 1) / BM * n_tiles + 7) / 8 * 8; };
  if constexpr (!TwoTerm<Epi>::value) {   // the products of two terms know their rows
    if (!exact && m_count) {
      // enough for any choice at any count up to M_max
      const int grid = std::max({blocks(256), kSpill<Epi> ? blocks(192) : std::min(blocks(192), 8 * kCUs),
                                 std::min(blocks(128), 4 * kCUs)});
      phase_gemm_any<DUAL, Epi><<<grid, 512, 0, s>>>(A, B, epi, m_count, M_max, K, n_tiles);
      return hipGetLastError();
    }
  }
  switch (phase_rows<kSpill<Epi>>(M_max, n_tiles)) {
    case 256: phase_gemm<Phase<256, DUAL>, Epi><<<blocks(256), 512, 0, s>>>(A, B, epi, m_count, M_max, K, n_tiles); break;
    case 192: phase_gemm<Phase<192, DUAL>, Epi><<<blocks(192), 512, 0, s>>>(A, B, epi, m_count, M_max, K, n_tiles); break;
    default: phase_gemm<Phase<128, DUAL>, Epi><<<blocks(128), 512, 0, s>>>(A, B, epi, m_count, M_max, K, n_tiles); break;
  }
  return hipGetLastError();
}

// K split S ways over 128-row tiles, for products of too few tiles to fill the CUs
template <class Epi>
hipError_t run_phase_split(ARows<bf16_t> A, BRows<bf16_t> B, Epi epi, const int* m_count, int M_max, int N_out, int K,
                           int S, hipStream_t s) {
  using C = Phase<128, false>;
  const int n_tiles = N_out / C::OUT_N;
  const dim3 grid(((M_max + 127) / 128 * n_tiles + 7) / 8 * 8, S);
  phase_gemm<C, Epi><<<grid, 512, 0, s>>>(A, B, epi, m_count, M_max, K, n_tiles);
  return hipGetLastError();
}

// Backward SwiGLU epilogue of one wave tile (EpiSwiGLUBwd on the MFMA path).  Lane l holds columns
// l & 15 (+ 16) of the wave's 32, gate in acc[a][0..1] and up in acc[a][2..3], at rows
// 16 a + 4 (l >> 4) + r of the wave's rows.  e is loaded two fragments of rows ahead, held as 16-bit
// words and widened at use (widening at the load let the compiler wait for each load in turn); a
// row's share of <e, act> is a sum over 16 lanes.  dG and dU of one half of the rows at a time are
// staged in the wave's own LDS region, whose operations complete in order, and leave as 16-byte
// row pieces.
template <class C, class Epi>
__device__ __forceinline__ void swiglu_bwd_tile(const Epi& epi, f32x4 (&acc)[2 * C::HM][4], unsigned char* smem, int m0,
                                                int nt, int wave, int wm, int wn, int M, int lane) {
  static_assert(C::DUAL, "gate/up tiles");
  constexpr int HM = C::HM, NA = 2 * HM, HR = 16 * HM, SPAD = C::ON + 8, CPR = C::ON / 8;
  static_assert(C::NW * (2 * HR * SPAD * 2 + 2 * HR * 4) <= 2 * C::STAGE, "backward staging fits in the stages");
  bf16_t* sg = reinterpret_cast<bf16_t*>(smem) + wave * 2 * HR * SPAD;
  bf16_t* su = sg + HR * SPAD;
  float* gl = reinterpret_cast<float*>(smem + C::NW * 2 * HR * SPAD * 2) + wave * 2 * HR;
  const int col0 = nt * C::OUT_N + wn * C::ON, l15 = lane & 15, g4 = 4 * (lane >> 4);
  auto row_of = [&](int h, int i) { return m0 + h * (C::BM / 2) + wm * (C::BM / 4) + i; };   // row i of half h
  for (int i = lane; i < 2 * HR; i += kWave) {
    const int m = min(row_of(i / HR, i % HR), M - 1);
    const int t = epi.idx ? epi.idx[m] : m;
    gl[i] = epi.gate ? epi.gate[t] : 1.0f;
  }
  constexpr int AHEAD = 2;
  bf16_t ev[AHEAD + 1][4][2];
  auto fetch = [&](int a) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int m = min(row_of(a / HM, 16 * (a % HM) + g4 + r), M - 1);
      const bf16_t* e = epi.e + static_cast<size_t>(m) * epi.ld_e + col0 + l15;
      ev[a % (AHEAD + 1)][r][0] = e[0];
      ev[a % (AHEAD + 1)][r][1] = e[16];
    }
  };
#pragma unroll
  for (int a = 0; a < AHEAD; ++a) fetch(a);
#pragma unroll
  for (int a = 0; a < NA; ++a) {
    const int h = a / HM;
    if (a + AHEAD < NA) fetch(a + AHEAD);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int i = 16 * (a % HM) + g4 + r;
      const float gt = gl[h * HR + i];
      float sum = 0.f;
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        const float g = acc[a][b][r], u = acc[a][2 + b][r];
        const float sg_ = __builtin_amdgcn_rcpf(1.0f + __expf(-g));
        const float ee = bf16_to_f32(ev[a % (AHEAD + 1)][r][b]);
        const float dact = gt * ee;
        sum += ee * (g * sg_ * u);
        sg[i * SPAD + 16 * b + l15] = f32_to_bf16(dact * u * sg_ * (1.0f + g * (1.0f - sg_)));
        su[i * SPAD + 16 * b + l15] = f32_to_bf16(dact * g * sg_);
      }
      sum = group_sum<16>(sum);
      const int m = row_of(h, i);
      if (l15 == 0 && m < M) epi.dgpart[static_cast<size_t>(m) * epi.n_parts + col0 / C::ON] = sum;
      __builtin_amdgcn_sched_barrier(0);   // one row at a time: the accumulators leave few registers
    }
    if (a % HM == HM - 1) {
#pragma unroll
      for (int p = 0; p < HR * CPR / kWave; ++p) {
        const int e = lane + kWave * p, i = e / CPR, c8 = (e % CPR) * 8;
        const u32x4 vg = *reinterpret_cast<const u32x4*>(sg + i * SPAD + c8);
        const u32x4 vu = *reinterpret_cast<const u32x4*>(su + i * SPAD + c8);
        const int m = row_of(h, i);
        if (m < M) {
          bf16_t* o = epi.dgu + static_cast<size_t>(m) * epi.ld_dgu + col0 + c8;
          *reinterpret_cast<u32x4*>(o) = vg;
          *reinterpret_cast<u32x4*>(o + epi.d_ff) = vu;
        }
      }
    }
  }
}

template <class C, class Epi>
hipError_t run_tile(ARows<bf16_t> A, BRows<bf16_t> B, Epi epi, const int* m_count, int M_max,
                    int N_out, int K, hipStream_t s, int splits = 1) {
  const int mt_max = (M_max + C::BM - 1) / C::BM;
  const int n_tiles = N_out / C::OUT_N;
  const int total = mt_max * n_tiles;
  if (total == 0) return hipSuccess;
  const dim3 grid((total + 7) / 8 * 8, splits);
  mfma_gemm<C, Epi><<<grid, C::NT, 0, s>>>(A, B, epi, m_count, M_max, K, mt_max, n_tiles);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// A routed decode step (at most 256 tokens) folds the branch decision and the adapter's
// down-projection into the gate/up launch, whose weight stream hides them (decode_route):
//   * every workgroup's activation producers decide the branches for themselves, one wave over up
//     to four tokens a lane, while the weight producers fill their ring; one workgroup also writes
//     the mask, the lists, the counts and lambda;
//   * the adapter's z = u W_1^T is formed for every token, so it waits for no decision: the launch
//     leaves CUs over (the busiest of ceil(nb / G) column blocks sets the time, and fewer
//     workgroups G reach the same maximum), and the first workgroups are the adapter's.
// The down product's reduction carries the adapter's up-projection the same way (decode_finish).
// Five launches on one stream instead of eleven on two, whose forks and joins cost an eager call
// about 7 us each: one 8B layer at 1 token 107 -> 85 us, 48 tokens 140 -> 102, the 7B decode stack of
// 256 tokens (a graph) 4.42 -> 3.74 ms with decode_head.
// ---------------------------------------------------------------------------
struct RouteArgs {
  SelectArgs sel;
  int na;                  // adapter workgroups (a multiple of 8): row tiles of 32 tokens x blocks of 32 tn columns
  int tn, groups, d_r;     // groups: adapter_groups(d)
  const bf16_t *u, *w1;
  float* z;                // [T][d_r]
};

struct RouteFinish {
  const float* z;
  const int *idx_ad, *idx_ffn, *counts;
  const bf16_t *w2, *hbar;
  const float* gate;
  bf16_t* out;
  int T, d, up_blocks;
  const float* part;
  int S, n_ffn_max;
  size_t stride;
};

// The branch decision of select_kernel for T <= kDecodeTokens by one wave: lane l holds tokens
// l, l + 64, ...  The n_skip-th smallest key is found bit by bit over ballots, its ties by token
// index.  list receives the FFN tokens in ascending order (kDecodeTokens ints); write: the outputs of
// SelectArgs too; adapters (may be null): the other tokens, also ascending.  Returns the FFN count.
__device__ __forceinline__ int select_wave(const SelectArgs& a, int lane, int* list, bool write,
                                           int* adapters = nullptr) {
  constexpr int Q = kDecodeTokens / kWave;
  float l[Q];
  uint32_t key[Q];
  unsigned long long valid[Q], skip[Q];
#pragma unroll
  for (int i = 0; i < Q; ++i) {
    const int t = lane + kWave * i;
    l[i] = t < a.T ? a.logit[t] : 0.f;
  }
#pragma unroll
  for (int i = 0; i < Q; ++i) {
    key[i] = order_key(l[i]);
    valid[i] = __ballot(lane + kWave * i < a.T);
    skip[i] = 0;
  }
  if (a.mode == 0) {
#pragma unroll
    for (int i = 0; i < Q; ++i) skip[i] = valid[i] & ~__ballot(l[i] >= a.thr);
  } else if (a.n_skip > 0) {
    // act: the tokens whose key agrees with the sought one in the bits taken so far; k: its rank
    // among them; skip: the tokens with smaller keys
    unsigned long long act[Q];
#pragma unroll
    for (int i = 0; i < Q; ++i) act[i] = valid[i];
    int k = a.n_skip;
    for (int bit = 31; bit >= 0; --bit) {
      unsigned long long zero[Q];
      int n = 0;
#pragma unroll
      for (int i = 0; i < Q; ++i) {
        zero[i] = act[i] & __ballot(((key[i] >> bit) & 1u) == 0u);
        n += __popcll(zero[i]);
      }
      const bool low = k <= n;
#pragma unroll
      for (int i = 0; i < Q; ++i) {
        if (!low) skip[i] |= zero[i];
        act[i] = low ? zero[i] : act[i] & ~zero[i];
      }
      if (!low) k -= n;
    }
    // the first k of the tied tokens
    int before = 0;
#pragma unroll
    for (int i = 0; i < Q; ++i) {
      const int r = before + __popcll(act[i] & ((1ull << lane) - 1ull));
      skip[i] |= __ballot(((act[i] >> lane) & 1ull) && r < k);
      before += __popcll(act[i]);
    }
  }
  int nf = 0, na = 0;
  float lmin = __builtin_inff();
#pragma unroll
  for (int i = 0; i < Q; ++i) {
    const int t = lane + kWave * i;
    const unsigned long long ffn = valid[i] & ~skip[i], ad = valid[i] & skip[i];
    const unsigned long long below = (1ull << lane) - 1ull;
    const bool f = (ffn >> lane) & 1ull;
    const int pf = nf + __popcll(ffn & below), pa = na + __popcll(ad & below);
    if (f) list[pf] = t;
    if (adapters && !f && t < a.T) adapters[pa] = t;
    if (write && t < a.T) {
      a.mask[t] = f ? 1 : 0;
      if (f)
        a.idx_ffn[pf] = t;
      else
        a.idx_ad[pa] = t;
    }
    if (f) lmin = fminf(lmin, l[i]);
    nf += __popcll(ffn);
    na += __popcll(ad);
  }
  if (write) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) lmin = fminf(lmin, __shfl_xor(lmin, off, kWave));
    if (lane == 0) {
      a.counts[0] = nf;
      a.counts[1] = na;
      a.lambda[0] = a.mode == 1 ? lmin : a.thr;
    }
  }
  return nf;
}

// z of 32 tokens against 32 TN of the d_r columns, by the eight waves of a workgroup.  The sums have
// the order of adapter_down_bf16 and adapter_up_tile, so that a token's z is the same bits at every
// call size: adapter_groups(d) K groups, each the sum of four pieces in turn, a piece a wave; eight
// pieces (two groups) a pass.  K groups on workgroups of their own left decode_finish eight partials
// to read: 8.9 for 8.1 us at 256 tokens of d = 4096.
template <int TN>
__device__ __forceinline__ void route_adapter(const RouteArgs& a, int K, int wg, unsigned char* smem) {
  constexpr int SB = 4, R = 32 * TN, RPITCH = R + 1, Q = 32 * R / 512;
  float* red = reinterpret_cast<float*>(smem);
  static_assert(8 * 32 * RPITCH * 4 <= 160 * 1024, "partials fit in LDS");
  const int T = a.sel.T, ncb = a.d_r / R;
  const int m0 = 32 * (wg / ncb), n0 = R * (wg % ncb);
  if (m0 >= T) return;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int kw = K / (4 * a.groups);   // a multiple of 16 SB (adapter_groups)
  const bf16_t* arow = a.u + static_cast<size_t>(min(m0 + (lane & 31), T - 1)) * K + 8 * (lane >> 5);
  const bf16_t* brow = a.w1 + static_cast<size_t>(n0 + (lane & 31)) * K + 8 * (lane >> 5);
  float z[Q];
#pragma unroll
  for (int q = 0; q < Q; ++q) z[q] = 0.f;
  for (int g = 0; g < a.groups; g += 2) {   // the pass's first group
    const int ng = min(2, a.groups - g);
    if (wave < 4 * ng) {
      const int kbeg = (4 * g + wave) * kw;
      f32x16 acc[TN];
#pragma unroll
      for (int b = 0; b < TN; ++b)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[b][r] = 0.f;
      for (int k = kbeg; k < kbeg + kw; k += 16 * SB) {
        bf16x8 fa[SB], fb[SB][TN];
#pragma unroll
        for (int st = 0; st < SB; ++st) {
          fa[st] = *reinterpret_cast<const bf16x8*>(arow + k + 16 * st);
#pragma unroll
          for (int b = 0; b < TN; ++b)
            fb[st][b] = *reinterpret_cast<const bf16x8*>(brow + static_cast<size_t>(32 * b) * K + k + 16 * st);
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int st = 0; st < SB; ++st)
#pragma unroll
          for (int b = 0; b < TN; ++b)
            acc[b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[st], fb[st][b], acc[b], 0, 0, 0);
      }
#pragma unroll
      for (int b = 0; b < TN; ++b)
#pragma unroll
        for (int r = 0; r < 16; ++r)
          red[(wave * 32 + out_row32(r, lane)) * RPITCH + b * 32 + (lane & 31)] = acc[b][r];
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const int e = threadIdx.x + 512 * q;
      const float* p = red + (e / R) * RPITCH + e % R;
      for (int x = 0; x < ng; ++x, p += 4 * 32 * RPITCH)
        z[q] += p[0] + p[32 * RPITCH] + p[64 * RPITCH] + p[96 * RPITCH];
    }
    __syncthreads();   // the next pass overwrites the partial tiles
  }
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    const int e = threadIdx.x + 512 * q, m = m0 + e / R;
    if (m < T) a.z[static_cast<size_t>(m) * a.d_r + n0 + e % R] = z[q];
  }
}

// ---------------------------------------------------------------------------
// Skinny products: a batch of at most 256 rows (a decode step) against weights streamed once
// from HBM.  The output columns are cut into 16-column blocks spread evenly over the workgroups
// (block group x takes the contiguous blocks [x nb / G, (x + 1) nb / G), and for the gate/up
// product the same blocks of W_u); S K-slices per block group where one workgroup per group
// would pull the activation rows through L2 too many times.
// Eight waves, one workgroup per CU.  Four consumers run the MFMAs (16 x 16 x 32), each on 16 RB
// rows against every weight block of the workgroup; four producers stage tiles into LDS, two the
// activation rows and two the weight rows, each pair into a ring of its own depth (weights come
// from HBM and need more bytes in flight than the L2-resident activations).  A producer's waits
// count only its own loads.  One barrier per k-tile, placed before the consumers' last k-step: by
// then they hold the whole stage in registers, so the producers refill it and the first
// fragments of the next tile are read while the last MFMAs run.
// What bounds it (measured on cold weights): a 64-deep k-tile takes 128 bytes from each weight
// row, and HBM serves such row-strided visits at ~3.5 TB/s (4.5 at 256 bytes, 5.3 at 512); with
// three or more row blocks the per-tile LDS traffic (DMA writes plus every consumer's fragment
// reads, ~108 KiB at 192 x 96) takes longer still, so deeper weight visits (which cost the
// activation ring its stages) and activation loads straight to registers both measured slower.
// ---------------------------------------------------------------------------
template <int NB_, int RB_, int NSA_, int NSB_, bool DUAL_>
struct Skinny {
  static constexpr int NB = NB_, RB = RB_, NSA = NSA_, NSB = NSB_;
  static constexpr bool DUAL = DUAL_;
  static constexpr int SL = DUAL ? 2 * NB : NB;   // 16-row weight blocks per stage
  static constexpr int MP = 64 * RB;              // rows covered (4 consumer waves x 16 RB)
  static constexpr int A_STAGE = MP * ROWB, B_STAGE = SL * 16 * ROWB;
  static constexpr int LDS = NSA * A_STAGE + NSB * B_STAGE;
  static constexpr int AL = MP / 16;              // 1 KiB loads per stage per A producer
  static constexpr int BL = SL;                   // 1 KiB loads per stage per B producer
  static_assert(LDS <= 160 * 1024, "stages fit in LDS");
  static_assert((NSA - 1) * AL < 64 && (NSB - 1) * BL < 64, "loads in flight within vmcnt");
  static_assert(NSA >= 2 && NSB >= 2 && RB >= 1 && RB <= 4 && NB >= 1, "shape");
};

// deepest weight ring that fits beside NSA activation stages
constexpr int skinny_nsb(int NB, int RB, bool dual, int NSA) {
  const int sl = dual ? 2 * NB : NB;
  int n = (160 * 1024 - NSA * 64 * RB * ROWB) / (sl * 16 * ROWB);
  n = n < 8 ? n : 8;
  return n < 63 / sl + 1 ? n : 63 / sl + 1;
}

template <int N>
__device__ __forceinline__ void wait_vm() {
  static_assert(N >= 0 && N < 64, "vmcnt range");
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// Epilogue: gate/up writes act[m][c] = bf16(SiLU(g) u) (out = act, ld = d_ff); otherwise the
// K-slice y writes fp32 sums to part + y split_stride (out = part, ld = N).
// tiled != 0: b0 holds the weights in the streaming order of tile_ffn_weights_kernel (16 x 64
// tiles, k-tile by k-tile, each k-tile's row of `tiled` 16-row blocks contiguous; for the
// gate/up product the W_g and W_u tiles of a block alternate) and b1, ldb are unused.  The same
// rows land in the same LDS slots either way, so the results are identical.  In the tiled order
// a workgroup's weights of one k-tile are one contiguous run of 2 KiB tiles, and the workgroups
// running the same k-tile read neighbouring runs, instead of 128-byte visits of rows 8 KiB apart.
// ROUTE: a routed decode step's gate/up product (decode_route): the first route.na workgroups are
// the adapter's, and the rows come from the decision made here instead of m_count and A.idx.
template <class C, bool ROUTE = false>
__global__ __launch_bounds__(512) void skinny_gemm(ARows<bf16_t> A, const bf16_t* __restrict__ b0,
                                                  const bf16_t* __restrict__ b1, int ldb, int tiled,
                                                  void* __restrict__ out, int ld, size_t split_stride,
                                                  const int* __restrict__ m_count, int n_max, int K,
                                                  int nb, int G, int S,
                                                  typename std::conditional<ROUTE, RouteArgs, int>::type route) {
  // a routed step's launch also holds the adapter's partial tiles (at most 129 KiB + 4 KiB)
  constexpr int kLds = ROUTE && C::LDS < 8 * 32 * 129 * 4 ? 8 * 32 * 129 * 4 : C::LDS;
  __shared__ __attribute__((aligned(1024))) unsigned char smem[kLds];
  if constexpr (ROUTE) {
    if (static_cast<int>(blockIdx.x) < route.na) {
      switch (route.tn) {
        case 1: route_adapter<1>(route, K, blockIdx.x, smem); break;
        case 2: route_adapter<2>(route, K, blockIdx.x, smem); break;
        case 3: route_adapter<3>(route, K, blockIdx.x, smem); break;
        default: route_adapter<4>(route, K, blockIdx.x, smem); break;
      }
      return;
    }
  }
  unsigned char* const sa = smem;
  unsigned char* const sb = smem + C::NSA * C::A_STAGE;
  // G block groups x S K-slices in slice-major order, laid over the 8 XCDs (round-robin dispatch)
  // in contiguous runs: the workgroups of one XCD share one or two K-slices of the activations
  // in its L2
  int id = static_cast<int>(blockIdx.x);
  if constexpr (ROUTE) id -= route.na;
  const int N = G * S;
  const int L = N % 8 == 0 ? (id & 7) * (N >> 3) + (id >> 3) : id;
  const int x = L % G, y = L / G;
  const int blk0 = x * nb / G;
  const int cnt = (x + 1) * nb / G - blk0;
  // the row count; a routed step in threshold mode counts the decisions (in budget mode n_max rows,
  // at least one, are certain)
  auto rows_of = [&]() -> int {
    if constexpr (ROUTE) {
      if (route.sel.mode != 0) return n_max;
      int n = 0;
#pragma unroll
      for (int i = 0; i < kDecodeTokens / kWave; ++i) {
        const int t = static_cast<int>(threadIdx.x & 63) + kWave * i;
        n += __popcll(__ballot(t < route.sel.T && route.sel.logit[min(t, route.sel.T - 1)] >= route.sel.thr));
      }
      return n;
    } else {
      return m_count ? min(*m_count, n_max) : n_max;
    }
  };
  const int nkt = K / BK;
  const int kt0 = y * nkt / S;
  const int nk = (y + 1) * nkt / S - kt0;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) >> 6);
  constexpr int NSA = C::NSA, NSB = C::NSB;
  const int M = ROUTE && wave >= 6 ? 1 : rows_of();   // the weight producers of a routed step count later
  if (M <= 0) {
    if constexpr (ROUTE)
      if (id == 0 && wave == 0) select_wave(route.sel, lane, reinterpret_cast<int*>(smem), true);
    return;
  }

  if (wave >= 6) {
    // weight producer: loads q = 2 i + pw, LDS rows 8q .. 8q + 7 = half (q & 1) of block slot q / 2;
    // a workgroup with fewer than NB blocks reloads its last one into the spare slots
    const int pw = wave - 6;
    const unsigned char* base[C::BL];
    uint32_t off[C::BL];
    constexpr int GU = C::DUAL ? 2 : 1;                       // matrices interleaved in a tiled block
    const uint32_t tstride = tiled ? static_cast<uint32_t>(tiled) * GU * 16 * ROWB : ROWB;  // k-tile to k-tile
#pragma unroll
    for (int i = 0; i < C::BL; ++i) {
      const int q = 2 * i + pw, slot = q >> 1;
      const int j = slot % C::NB;
      const int r = 8 * q + (lane >> 3);
      const int ch = (lane & 7) ^ ((r >> 1) & 7);
      const int blk = blk0 + min(j, cnt - 1), rr = 8 * (q & 1) + (lane >> 3);
      const int second = C::DUAL && slot >= C::NB;
      if (tiled) {
        base[i] = reinterpret_cast<const unsigned char*>(b0);
        off[i] = ((static_cast<uint32_t>(kt0) * tiled + blk) * GU + second) * (16 * ROWB) + rr * ROWB + ch * 16;
      } else {
        base[i] = reinterpret_cast<const unsigned char*>(second ? b1 : b0);
        off[i] = static_cast<uint32_t>(16 * blk + rr) * static_cast<uint32_t>(ldb * 2) + kt0 * ROWB + ch * 16;
      }
    }
    auto issue = [&](int t) {
      unsigned char* st = sb + (t % NSB) * C::B_STAGE;
#pragma unroll
      for (int i = 0; i < C::BL; ++i) load_lds16(base[i] + off[i] + t * tstride, st + (2 * i + pw) * 1024);
    };
    for (int t = 0; t < NSB; ++t)
      if (t < nk) issue(t);
    if constexpr (ROUTE) {
      // no FFN row: the other waves have left; this one leaves when its loads have landed
      if (rows_of() <= 0) {
        wait_vm<0>();
        return;
      }
    }
    // before barrier j tile j + 1 has landed; tiles up to j + NSB - 1 may be in flight
    for (int j = -1; j < nk; ++j) {
      if (j < 0) {
        if (nk >= NSB) wait_vm<(NSB - 1) * C::BL>(); else wait_vm<0>();
      } else if (j + NSB <= nk) {
        wait_vm<(NSB - 2) * C::BL>();
      } else {
        wait_vm<0>();
      }
      __syncthreads();
      if (j >= 0 && j + NSB < nk) issue(j + NSB);
    }
    return;
  }
  if (wave >= 4) {
    // activation producer: loads q = 2 i + pw, LDS rows 8q .. 8q + 7; rows past M repeat row M - 1
    const int pw = wave - 4;
    uint32_t off[C::AL];
    // the wave's own list of FFN tokens, in the 1 KiB of the first stage that only its loads fill
    const int* rows = A.idx;
    if constexpr (ROUTE) {
      static_assert(kDecodeTokens * sizeof(int) <= 1024, "the list fits the first load's KiB");
      int* list = reinterpret_cast<int*>(sa + pw * 1024);
      select_wave(route.sel, lane, list, id == 0 && pw == 0);
      rows = list;
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    }
#pragma unroll
    for (int i = 0; i < C::AL; ++i) {
      const int r = 8 * (2 * i + pw) + (lane >> 3);
      const int ch = (lane & 7) ^ ((r >> 1) & 7);
      const int m = min(r, M - 1);
      const int row = rows ? rows[m] : m;
      off[i] = static_cast<uint32_t>(row) * static_cast<uint32_t>(A.ld * 2) + kt0 * ROWB + ch * 16;
    }
    const unsigned char* abase = reinterpret_cast<const unsigned char*>(A.base);
    if constexpr (ROUTE) asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // the list is read before it is overwritten
    auto issue = [&](int t) {
      unsigned char* st = sa + (t % NSA) * C::A_STAGE;
#pragma unroll
      for (int i = 0; i < C::AL; ++i) load_lds16(abase + off[i] + t * ROWB, st + (2 * i + pw) * 1024);
    };
    for (int t = 0; t < NSA; ++t)
      if (t < nk) issue(t);
    for (int j = -1; j < nk; ++j) {
      if (j < 0) {
        if (nk >= NSA) wait_vm<(NSA - 1) * C::AL>(); else wait_vm<0>();
      } else if (j + NSA <= nk) {
        wait_vm<(NSA - 2) * C::AL>();
      } else {
        wait_vm<0>();
      }
      __syncthreads();
      if (j >= 0 && j + NSA < nk) issue(j + NSA);
    }
    return;
  }

  // consumers
  constexpr int RB = C::RB, SL = C::SL;
  f32x4 acc[RB][SL];
#pragma unroll
  for (int r = 0; r < RB; ++r)
#pragma unroll
    for (int c = 0; c < SL; ++c) acc[r][c] = f32x4{0.f, 0.f, 0.f, 0.f};
  bf16x8 fa[2][RB], fb[2][SL];
  const int arow0 = wave * 16 * RB + (lane & 15), brow0 = lane & 15;
  auto read = [&](int buf, const unsigned char* ast, const unsigned char* bst, int ks) {
    const int c = in_chunk<16>(ks, lane);
#pragma unroll
    for (int r = 0; r < RB; ++r) fa[buf][r] = *reinterpret_cast<const bf16x8*>(ast + swz(arow0 + 16 * r, c));
#pragma unroll
    for (int b = 0; b < SL; ++b) fb[buf][b] = *reinterpret_cast<const bf16x8*>(bst + swz(brow0 + 16 * b, c));
  };
  auto mfmas = [&](int buf) {
#pragma unroll
    for (int r = 0; r < RB; ++r)
#pragma unroll
      for (int b = 0; b < SL; ++b) acc[r][b] = mfma_op(fa[buf][r], fb[buf][b], acc[r][b]);
  };
  // the fragment reads of the other k-step go out one after each MFMA; the reads of tile kt + 1
  // past the last tile hit a stale stage and are never used
  auto interleave = [&]() {
#pragma unroll
    for (int i = 0; i < RB * SL; ++i) {
      __builtin_amdgcn_sched_group_barrier(SG_MFMA, 1, 0);
      if (i < RB + SL) __builtin_amdgcn_sched_group_barrier(SG_DS_READ, 1, 0);
    }
    if constexpr (RB + SL > RB * SL) __builtin_amdgcn_sched_group_barrier(SG_DS_READ, RB + SL - RB * SL, 0);
  };
  __syncthreads();                       // barrier -1: tile 0 has landed
  read(0, sa, sb, 0);
  int ia = 0, ib = 0;                    // stages of tile kt
  for (int kt = 0; kt < nk; ++kt) {
    read(1, sa + ia * C::A_STAGE, sb + ib * C::B_STAGE, 1);
    mfmas(0);
    interleave();
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __syncthreads();                     // barrier kt: stage kt is free, tile kt + 1 has landed
    ia = ia + 1 == NSA ? 0 : ia + 1;
    ib = ib + 1 == NSB ? 0 : ib + 1;
    read(0, sa + ia * C::A_STAGE, sb + ib * C::B_STAGE, 0);
    mfmas(1);
    interleave();
    __builtin_amdgcn_sched_barrier(0);
  }

  // element i of acc[r][b] in lane l: row 16 (wave RB + r) + 4 (l >> 4) + i, column l & 15
  const int col = lane & 15;
#pragma unroll
  for (int r = 0; r < RB; ++r)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int m = 16 * (wave * RB + r) + 4 * (lane >> 4) + i;
      if (m >= M) continue;
      if constexpr (C::DUAL) {
        bf16_t* o = static_cast<bf16_t*>(out) + static_cast<size_t>(m) * ld;
#pragma unroll
        for (int j = 0; j < C::NB; ++j) {
          if (j >= cnt) break;
          const float g = acc[r][j][i], u = acc[r][C::NB + j][i];
          o[16 * (blk0 + j) + col] = f32_to_bf16(g * __builtin_amdgcn_rcpf(1.0f + __expf(-g)) * u);
        }
      } else {
        float* o = static_cast<float*>(out) + y * split_stride + static_cast<size_t>(m) * ld;
#pragma unroll
        for (int j = 0; j < C::NB; ++j) {
          if (j >= cnt) break;
          o[16 * (blk0 + j) + col] = acc[r][j][i];
        }
      }
    }
}

template <class C>
hipError_t run_skinny(ARows<bf16_t> A, const bf16_t* b0, const bf16_t* b1, int ldb, int tiled, void* out, int ld,
                      size_t split_stride, const int* m_count, int n_max, int K, int nb, int G, int S,
                      hipStream_t s) {
  skinny_gemm<C><<<G * S, 512, 0, s>>>(A, b0, b1, ldb, tiled, out, ld, split_stride, m_count, n_max, K, nb, G, S, 0);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// fp32 GEMM on the fp32 matrix cores (v_mfma_f32_16x16x4f32: products and sums in fp32)
//
// A workgroup of four waves computes a 16 R x 16 R output tile; the waves take every fourth
// 16-deep k-step and their partial tiles are added in wave order through LDS.  The fragments come
// straight from memory: lane l holds k = 4 (l >> 4) .. + 3 of row l & 15 of a k-step as one 16-byte
// load, and element e of it feeds MFMA e of the step (both operands take the k in that order, so
// every k meets its own).  A batch of U steps is loaded before its products.
// The fp32 shapes are narrow, so their launches are short of workgroups and bound by the chain of
// dependent loads, not by the arithmetic: a 64 x 64 LDS tile on the VALU walked K = 688 in 43
// dependent steps on 4 workgroups at 64 rows.  Measured against it: the 4-layer stack of
// d = 256, d_ff = 688 at 64 tokens 1318 -> 508 us, 2 layers of d = 2048, d_ff = 5632 at 20 tokens
// 3460 -> 407 us and at 2048 tokens 6489 -> 4540 us.  Without LDS each tile reads its operands anew,
// so once the 64 x 64 tiles fill the chip several times over they are the faster ones
// (f32_valu_gemm).
// ---------------------------------------------------------------------------

// elements k .. k + 3 of a row, zero past K; VEC: K and both row pitches are multiples of four
template <bool VEC>
__device__ __forceinline__ f32x4 f32_frag(const float* row, int k, int K) {
  f32x4 v = {0.f, 0.f, 0.f, 0.f};
  if constexpr (VEC) {
    if (k < K) v = *reinterpret_cast<const f32x4*>(row + k);
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (k + e < K) v[e] = row[k + e];
  }
  return v;
}

template <bool DUAL, int R, bool VEC, class Epi>
__device__ __forceinline__ void f32_tile(const ARows<float>& A, const BRows<float>& B, const Epi& epi, int M, int N,
                                         int K, int bm, int bn) {
  constexpr int BT = 16 * R;                   // rows and columns of the tile
  constexpr int U = R == 1 ? 8 : 4;            // k-steps per batch of loads
  constexpr int RP = BT + 1;
  __shared__ float red[DUAL ? 2 : 1][4][BT][RP];
  const int m0 = bm * BT, n0 = bn * BT;
  if (m0 >= M) return;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) >> 6);
  const int r16 = lane & 15, k4 = 4 * (lane >> 4);
  // rows and columns past the end repeat the last one: their results are not stored
  const float *ar[R], *br[R], *ur[R];
#pragma unroll
  for (int i = 0; i < R; ++i) {
    ar[i] = A.row(min(m0 + 16 * i + r16, M - 1));
    const int n = min(n0 + 16 * i + r16, N - 1);
    if constexpr (DUAL) {
      br[i] = B.gate_row(n);
      ur[i] = B.up_row(n);
    } else {
      br[i] = B.row(n);
    }
  }
  f32x4 acc[R][R], acu[R][R];
#pragma unroll
  for (int i = 0; i < R; ++i)
#pragma unroll
    for (int j = 0; j < R; ++j) acc[i][j] = acu[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int nks = (K + 15) / 16;
  for (int s0 = wave; s0 < nks; s0 += 4 * U) {
    f32x4 fa[U][R], fb[U][R], fu[U][R];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int k = 16 * (s0 + 4 * u) + k4;    // past K in the last batch: zeros
#pragma unroll
      for (int i = 0; i < R; ++i) {
        fa[u][i] = f32_frag<VEC>(ar[i], k, K);
        fb[u][i] = f32_frag<VEC>(br[i], k, K);
        if constexpr (DUAL) fu[u][i] = f32_frag<VEC>(ur[i], k, K);
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int i = 0; i < R; ++i)
#pragma unroll
          for (int j = 0; j < R; ++j) {
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(fa[u][i][e], fb[u][j][e], acc[i][j], 0, 0, 0);
            if constexpr (DUAL)
              acu[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(fa[u][i][e], fu[u][j][e], acu[i][j], 0, 0, 0);
          }
  }
#pragma unroll
  for (int i = 0; i < R; ++i)
#pragma unroll
    for (int j = 0; j < R; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        red[0][wave][16 * i + k4 + r][16 * j + r16] = acc[i][j][r];
        if constexpr (DUAL) red[1][wave][16 * i + k4 + r][16 * j + r16] = acu[i][j][r];
      }
  __syncthreads();
  for (int e = threadIdx.x; e < BT * BT; e += 256) {
    const int i = e / BT, c = e % BT;
    if (m0 + i >= M || n0 + c >= N) continue;
    float v = 0.f, w = 0.f;
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      v += red[0][g][i][c];
      if constexpr (DUAL) w += red[1][g][i][c];
    }
    if constexpr (DUAL)
      epi.store2(m0 + i, n0 + c, v, w);
    else
      epi.store(m0 + i, n0 + c, v);
  }
}

template <bool DUAL, int R, bool VEC, class Epi>
__global__ __launch_bounds__(256) void f32_gemm(ARows<float> A, BRows<float> B, Epi epi,
                                               const int* __restrict__ m_count, int M_fixed,
                                               int N, int K) {
  f32_tile<DUAL, R, VEC>(A, B, epi, m_count ? *m_count : M_fixed, N, K, static_cast<int>(blockIdx.x),
                         static_cast<int>(blockIdx.y));
}

// Products of few tiles are bound by their launches and load latencies, so two that do not depend on
// each other share one: the row pass beside the router's product, the adapter's beside the FFN's
// (f32_pair), whose first launch also decides the branches, a wave of every workgroup for itself.
// The 4-layer stack of d = 256 at 64 tokens: 147 us with a launch each, 105 so; 2 layers of d = 2048
// at 20 tokens 407 -> 181.
template <bool VEC>
__global__ __launch_bounds__(256) void f32_head(ARows<float> A, BRows<float> B, EpiStoreF32 epi, int T, int N, int K,
                                               int mt, int tiles, const float* __restrict__ prev1,
                                               const float* __restrict__ prev2, const float* __restrict__ norm_w,
                                               int j, float eps_norm, float* __restrict__ rowstat,
                                               float* __restrict__ u) {
  const int b = static_cast<int>(blockIdx.x);
  if (b >= tiles)
    rowstats_row<float>(b - tiles, T, A.base, prev1, prev2, norm_w, K, j, eps_norm, rowstat, u);
  else
    f32_tile<false, 1, VEC>(A, B, epi, T, N, K, b % mt, b / mt);
}

template <class Epi>
struct F32Job {
  ARows<float> A;
  BRows<float> B;
  Epi epi;
  int M_max, N, K;
  bool vec() const {
    const auto al = [](const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; };
    return K % 4 == 0 && A.ld % 4 == 0 && B.ld % 4 == 0 && al(A.base) && al(B.b0) && al(B.b1);
  }
  __host__ __device__ int mt() const { return (M_max + 15) / 16; }
  int tiles() const { return mt() * ((N + 15) / 16); }
};

// ROUTE: the row lists are decided here (at most kDecodeTokens tokens); else sel.counts holds the
// row counts: [0] of the first job, [1] of the second
template <bool DUAL, bool V0, bool V1, bool ROUTE, class E0, class E1>
__global__ __launch_bounds__(256) void f32_pair(F32Job<E0> j0, F32Job<E1> j1, int tiles0, SelectArgs sel) {
  const int b = static_cast<int>(blockIdx.x);
  int nf, na;
  if constexpr (ROUTE) {
    __shared__ int lists[2][kDecodeTokens];
    __shared__ int s_nf;
    if (threadIdx.x < kWave) {
      const int n = select_wave(sel, static_cast<int>(threadIdx.x), lists[0], b == 0, lists[1]);
      if (threadIdx.x == 0) s_nf = n;
    }
    __syncthreads();
    nf = s_nf;
    na = sel.T - nf;
    j0.A.idx = lists[0];
    j1.A.idx = lists[1];
  } else {
    nf = sel.counts[0];
    na = sel.counts[1];
  }
  if (b < tiles0)
    f32_tile<DUAL, 1, V0>(j0.A, j0.B, j0.epi, nf, j0.N, j0.K, b % j0.mt(), b / j0.mt());
  else
    f32_tile<false, 1, V1>(j1.A, j1.B, j1.epi, na, j1.N, j1.K, (b - tiles0) % j1.mt(), (b - tiles0) / j1.mt());
}

template <bool DUAL, bool ROUTE, class E0, class E1>
hipError_t run_f32_pair(const F32Job<E0>& j0, const F32Job<E1>& j1, const SelectArgs& sel, hipStream_t s) {
  const int t0 = j0.tiles(), blocks = t0 + j1.tiles();
  if (blocks <= 0) return hipSuccess;
  const bool v0 = j0.vec(), v1 = j1.vec();
  if (v0 && v1)
    f32_pair<DUAL, true, true, ROUTE><<<blocks, 256, 0, s>>>(j0, j1, t0, sel);
  else if (v0)
    f32_pair<DUAL, true, false, ROUTE><<<blocks, 256, 0, s>>>(j0, j1, t0, sel);
  else if (v1)
    f32_pair<DUAL, false, true, ROUTE><<<blocks, 256, 0, s>>>(j0, j1, t0, sel);
  else
    f32_pair<DUAL, false, false, ROUTE><<<blocks, 256, 0, s>>>(j0, j1, t0, sel);
  return hipGetLastError();
}

// 32 x 32 tiles halve the operand bytes per product once they fill the CUs
bool f32_tiles_large(int M, int N) {
  return static_cast<long long>((M + 31) / 32) * ((N + 31) / 32) >= 2 * kCUs;
}

template <bool DUAL, int R, class Epi>
hipError_t run_f32_r(ARows<float> A, BRows<float> B, Epi epi, const int* m_count, int M_max, int N,
                     int K, bool vec, hipStream_t s) {
  const dim3 grid((M_max + 16 * R - 1) / (16 * R), (N + 16 * R - 1) / (16 * R));
  if (vec)
    f32_gemm<DUAL, R, true, Epi><<<grid, 256, 0, s>>>(A, B, epi, m_count, M_max, N, K);
  else
    f32_gemm<DUAL, R, false, Epi><<<grid, 256, 0, s>>>(A, B, epi, m_count, M_max, N, K);
  return hipGetLastError();
}

// Large fp32 products: 64 x 64 tiles through LDS on the VALU, 4 x 4 outputs per thread, full bounds
// checks.  The VALU's rate bounds it (64 TFLOP/s at 2990 rows of d = 2048, d_ff = 5632).
template <bool DUAL, class Epi>
__global__ __launch_bounds__(256) void f32_valu_gemm(ARows<float> A, BRows<float> B, Epi epi,
                                                    const int* __restrict__ m_count, int M_fixed,
                                                    int N, int K) {
  __shared__ float As[16][68];
  __shared__ float Bs[16][68];
  __shared__ float Us[DUAL ? 16 : 1][68];
  const int M = m_count ? *m_count : M_fixed;
  const int m0 = blockIdx.y * 64, n0 = blockIdx.x * 64;
  if (m0 >= M) return;
  const int tx = threadIdx.x & 15, ty = threadIdx.x >> 4;
  float acc[4][4], acu[4][4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = acu[i][j] = 0.f;
  for (int k0 = 0; k0 < K; k0 += 16) {
    for (int e = threadIdx.x; e < 64 * 16; e += 256) {
      const int r = e >> 4, kk = e & 15, k = k0 + kk;
      const int m = m0 + r, n = n0 + r;
      As[kk][r] = (m < M && k < K) ? A.row(m)[k] : 0.f;
      if (DUAL) {
        Bs[kk][r] = (n < N && k < K) ? B.gate_row(n)[k] : 0.f;
        Us[kk][r] = (n < N && k < K) ? B.up_row(n)[k] : 0.f;
      } else {
        Bs[kk][r] = (n < N && k < K) ? B.row(n)[k] : 0.f;
      }
    }
    __syncthreads();
#pragma unroll
    for (int kk = 0; kk < 16; ++kk) {
      float a[4], b[4], u[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        a[i] = As[kk][ty * 4 + i];
        b[i] = Bs[kk][tx * 4 + i];
        if (DUAL) u[i] = Us[kk][tx * 4 + i];
      }
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          acc[i][j] = fmaf(a[i], b[j], acc[i][j]);
          if (DUAL) acu[i][j] = fmaf(a[i], u[j], acu[i][j]);
        }
    }
    __syncthreads();
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int m = m0 + ty * 4 + i;
    if (m >= M) continue;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int n = n0 + tx * 4 + j;
      if (n >= N) continue;
      if constexpr (DUAL) {
        epi.store2(m, n, acc[i][j], acu[i][j]);
      } else {
        epi.store(m, n, acc[i][j]);
      }
    }
  }
}

// Where the VALU tiles are the faster ones, by the row bound M, columns N and depth K (matrix cores
// against VALU, us): eight or more of them per CU over 2048 rows for two products in one (2990 rows,
// d = 2048, d_ff = 5632: 2567 / 2147; d = 1024, d_ff = 2816: 642 / 596; but 1495 rows of the former
// 1307 / 1320), over 4096 rows for one (its down product of 5980 rows 2829 / 2710, of 11960
// 5840 / 4953; d = 1024, 5980 rows, six per CU: 736 / 777), two per CU for the adapters' few k-steps
// (K = 64, 2212 rows, 2048 columns: 50 / 35; 1106 rows, 1024 columns: 20 / 23).
bool f32_valu_fits(bool dual, int M, int N, int K) {
  const long long tiles = static_cast<long long>((M + 63) / 64) * ((N + 63) / 64);
  if ((M + 63) / 64 > 65535) return false;   // grid limit
  if (K <= 64) return tiles >= 2 * kCUs;
  return tiles >= 8 * kCUs && M >= (dual ? 2048 : 4096);
}

template <bool DUAL, class Epi>
hipError_t run_f32(ARows<float> A, BRows<float> B, Epi epi, const int* m_count, int M_max, int N,
                   int K, hipStream_t s) {
  if (M_max <= 0 || N <= 0) return hipSuccess;
  if (f32_valu_fits(DUAL, M_max, N, K)) {
    const dim3 grid((N + 63) / 64, (M_max + 63) / 64);
    f32_valu_gemm<DUAL, Epi><<<grid, 256, 0, s>>>(A, B, epi, m_count, M_max, N, K);
    return hipGetLastError();
  }
  const bool vec = F32Job<Epi>{A, B, epi, M_max, N, K}.vec();
  if (f32_tiles_large(M_max, N)) return run_f32_r<DUAL, 2>(A, B, epi, m_count, M_max, N, K, vec, s);
  return run_f32_r<DUAL, 1>(A, B, epi, m_count, M_max, N, K, vec, s);
}

// ---------------------------------------------------------------------------
// bf16 adapter: skinny GEMMs with MFMA fragments loaded straight from memory
// ---------------------------------------------------------------------------

// Adapter down-projection partial sums.  Workgroup (row tile of 32, k-group g) has
// 4 waves, each over a quarter of the group's k range; the 4 partial 32 x d_r
// tiles are summed in LDS and written to part[g][m][n] (fp32).
template <int TN, int SB>
__global__ __launch_bounds__(256) void adapter_down_bf16(const bf16_t* __restrict__ u0,
                                                         const int* __restrict__ idx,
                                                         const int* __restrict__ m_count,
                                                         const bf16_t* __restrict__ w0,
                                                         float* __restrict__ part0, int T, int K,
                                                         int k_group, const bf16_t* __restrict__ u_z1,
                                                         const bf16_t* __restrict__ w_z1,
                                                         float* __restrict__ part_z1) {
  // gridDim.z = 2 runs a second product over the same rows (the backward's z and e_a)
  const bf16_t* __restrict__ u = blockIdx.z ? u_z1 : u0;
  const bf16_t* __restrict__ w1 = blockIdx.z ? w_z1 : w0;
  float* __restrict__ part = blockIdx.z ? part_z1 : part0;
  constexpr int R = TN * 32;
  __shared__ float red[4][32][R + 1];
  const int M = *m_count;
  const int m0 = blockIdx.x * 32;
  if (m0 >= M) return;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int g = blockIdx.y;
  const int kw = k_group / 4;
  const int kbeg = g * k_group + wave * kw;
  const int m = min(m0 + (lane & 31), M - 1);
  const bf16_t* arow = u + static_cast<size_t>(idx[m]) * K + 8 * (lane >> 5);
  f32x16 acc[TN];
#pragma unroll
  for (int b = 0; b < TN; ++b)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[b][r] = 0.f;
  // SB 16-deep k-steps per batch, all of a batch's loads issued first (kw % (16 SB) == 0)
  for (int k = kbeg; k < kbeg + kw; k += 16 * SB) {
    bf16x8 fa[SB], fb[SB][TN];
#pragma unroll
    for (int st = 0; st < SB; ++st) {
      fa[st] = *reinterpret_cast<const bf16x8*>(arow + k + 16 * st);
#pragma unroll
      for (int b = 0; b < TN; ++b)
        fb[st][b] = *reinterpret_cast<const bf16x8*>(
            w1 + static_cast<size_t>(b * 32 + (lane & 31)) * K + 8 * (lane >> 5) + k + 16 * st);
    }
    __builtin_amdgcn_sched_barrier(0);   // keep the whole batch of loads ahead of the MFMAs
#pragma unroll
    for (int st = 0; st < SB; ++st)
#pragma unroll
      for (int b = 0; b < TN; ++b)
        acc[b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[st], fb[st][b], acc[b], 0, 0, 0);
  }
#pragma unroll
  for (int b = 0; b < TN; ++b)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int i = 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
      red[wave][i][b * 32 + (lane & 31)] = acc[b][r];
    }
  __syncthreads();
  for (int e = threadIdx.x; e < 32 * R; e += 256) {
    const int i = e / R, n = e % R;
    if (m0 + i >= M) continue;
    const float v = red[0][i][n] + red[1][i][n] + red[2][i][n] + red[3][i][n];
    part[(static_cast<size_t>(g) * T + m0 + i) * R + n] = v;
  }
}

// Adapter up-projection with scatter, one workgroup per (32 rows, 256 columns):
//   hid = SiLU(sum_g part[g]) for the 32 rows, rounded to bf16 (the MFMA A operand), in LDS;
//   each wave computes 64 columns; results are staged in LDS and every thread then writes
//   8-column pieces h_out[t] = hbar[t] + (1 - g_t) acc with hbar fetched at the start.
// BY_TOKEN: the G partials are held by token (row idx[m]) instead of by list position.
template <int KR, int G, bool BY_TOKEN>
__device__ __forceinline__ void adapter_up_tile(const float* __restrict__ part, const int* __restrict__ idx,
                                                const int* __restrict__ m_count, const bf16_t* __restrict__ w2,
                                                const bf16_t* __restrict__ hbar, const float* __restrict__ gate,
                                                bf16_t* __restrict__ out, int T, int d, int m0, int n0) {
  constexpr int NC = 256;
  constexpr int HP = KR + 8;     // hid row pitch (bf16)
  constexpr int SP = NC + 4;     // staged row pitch (fp32)
  constexpr int PPT = 32 * NC / 8 / 256;   // 8-column output pieces per thread
  __shared__ __attribute__((aligned(16))) bf16_t hid[32 * HP];
  __shared__ __attribute__((aligned(16))) float stg[32 * SP];
  const int M = *m_count;
  if (m0 >= M) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  EpiScatter<bf16_t, true> epi{idx, hbar, gate, out, d};
  typename EpiScatter<bf16_t, true>::Pre pre[PPT];
#pragma unroll
  for (int q = 0; q < PPT; ++q) {
    const int e = tid + 256 * q;
    pre[q] = epi.prep(min(m0 + (e >> 5), M - 1), n0 + (e & 31) * 8);
  }
  for (int e = tid; e < 32 * KR / 8; e += 256) {
    const int i = e / (KR / 8), k8 = (e % (KR / 8)) * 8;
    const int mi = min(m0 + i, M - 1), mr = BY_TOKEN ? idx[mi] : mi;
    f32x4 x[G][2];
#pragma unroll
    for (int g = 0; g < G; ++g) {
      const float* p = part + (static_cast<size_t>(g) * T + mr) * KR + k8;
      x[g][0] = *reinterpret_cast<const f32x4*>(p);
      x[g][1] = *reinterpret_cast<const f32x4*>(p + 4);
    }
    bf16x8 v;
#pragma unroll
    for (int c = 0; c < 8; ++c) {
      float h = 0.f;
#pragma unroll
      for (int g = 0; g < G; ++g) h += x[g][c >> 2][c & 3];
      v[c] = static_cast<__bf16>(siluf_(h));
    }
    *reinterpret_cast<bf16x8*>(hid + i * HP + k8) = v;
  }
  bf16x8 fb[KR / 16][2];
#pragma unroll
  for (int st = 0; st < KR / 16; ++st)
#pragma unroll
    for (int b = 0; b < 2; ++b)
      fb[st][b] = *reinterpret_cast<const bf16x8*>(
          w2 + static_cast<size_t>(n0 + wave * 64 + b * 32 + (lane & 31)) * KR + 16 * st + 8 * (lane >> 5));
  __syncthreads();
  f32x16 acc[2];
#pragma unroll
  for (int b = 0; b < 2; ++b)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[b][r] = 0.f;
#pragma unroll
  for (int st = 0; st < KR / 16; ++st) {
    const bf16x8 fa = *reinterpret_cast<const bf16x8*>(hid + (lane & 31) * HP + 16 * st + 8 * (lane >> 5));
#pragma unroll
    for (int b = 0; b < 2; ++b) acc[b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa, fb[st][b], acc[b], 0, 0, 0);
  }
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int i = 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
#pragma unroll
    for (int b = 0; b < 2; ++b) stg[i * SP + wave * 64 + b * 32 + (lane & 31)] = acc[b][r];
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < PPT; ++q) {
    const int e = tid + 256 * q;
    const int i = e >> 5, c8 = (e & 31) * 8;
    if (m0 + i < M) epi.emit8(pre[q], m0 + i, n0 + c8, stg + i * SP + c8);
  }
}

template <int KR, int G>
__global__ __launch_bounds__(256) void adapter_up_bf16(const float* __restrict__ part,
                                                       const int* __restrict__ idx,
                                                       const int* __restrict__ m_count,
                                                       const bf16_t* __restrict__ w2,
                                                       const bf16_t* __restrict__ hbar,
                                                       const float* __restrict__ gate,
                                                       bf16_t* __restrict__ out, int T, int d) {
  adapter_up_tile<KR, G, false>(part, idx, m_count, w2, hbar, gate, out, T, d, blockIdx.x * 32, blockIdx.y * 256);
}

template <int KR>
void adapter_up_launch(dim3 g2, hipStream_t s, int G, const float* part, const int* idx, const int* counts,
                       const bf16_t* w2, const bf16_t* hb, const float* gate, bf16_t* ho, int T, int d) {
  switch (G) {
    case 1: adapter_up_bf16<KR, 1><<<g2, 256, 0, s>>>(part, idx, counts, w2, hb, gate, ho, T, d); break;
    case 2: adapter_up_bf16<KR, 2><<<g2, 256, 0, s>>>(part, idx, counts, w2, hb, gate, ho, T, d); break;
    case 4: adapter_up_bf16<KR, 4><<<g2, 256, 0, s>>>(part, idx, counts, w2, hb, gate, ho, T, d); break;
    default: adapter_up_bf16<KR, 8><<<g2, 256, 0, s>>>(part, idx, counts, w2, hb, gate, ho, T, d); break;
  }
}

// K-slices of the adapter down-projection: up to 8, each deep enough for whole batches
// (four waves times SB 16-deep k-steps); eight-step batches where the depth allows.
int adapter_groups(int K) {
  int G = 8;
  while (G > 1 && K % (G * 512) != 0) G >>= 1;
  if (K % (G * 512) != 0) {
    G = 8;
    while (G > 1 && K % (G * 256) != 0) G >>= 1;
  }
  return G;
}
int adapter_batch(int K, int G) { return (K / G) % 512 == 0 ? 8 : 4; }
// The forward's K-slices for a call of up to n_max adapter rows: fewer as the rows alone give
// enough workgroups (the up-projection reads every slice once per 256-column block, so at the
// 8B stack's 12.7k adapter rows eight slices would be read 16 times over for nothing).
int adapter_groups_rows(int K, int n_max) {
  int G = adapter_groups(K);
  const long long row_tiles = (static_cast<long long>(n_max) + 31) / 32;
  while (G > 1 && row_tiles * G > 2048) G >>= 1;
  return G;
}

// router pre-activations: 128-row tiles over all 8 waves, K split four ways
using TileRouter = Tile<128, 256, 2, 4>;
using TileRouterNarrow = Tile<128, 128, 2, 4>;
// few tokens (a decode batch): 64-row tiles of 4 waves, four times the workgroups; each streams
// a quarter of K, with three k-tiles in flight
using TileRouterSmall = Tile<64, 128, 1, 4, 4>;

}  // namespace

// K split of the router pre-activation product: four slices while the tiles alone would leave
// most CUs idle (a 4096-token layer has 64 tiles of 128 x 256), fewer as the token count grows,
// none from one full round of tiles on (32768 tokens: 512 tiles), where the slices would only add
// fp32 partial traffic for the router's pre pass to read.
int router_gemm_splits(int dtype, int d, int T, int N) {
  if (dtype != 1 || d % (4 * 64) != 0) return 1;
  if (T <= 1024) return 4;
  const long long tiles = static_cast<long long>((T + TileRouter::BM - 1) / TileRouter::BM) *
                          ((N + TileRouter::BN - 1) / TileRouter::BN);
  return static_cast<int>(std::max(1LL, std::min(4LL, kCUs / std::max(1LL, tiles))));
}

hipError_t launch_decode_head_tiles(const void* hbar, const void* prev1, const void* prev2, const void* norm_w,
                                    const void* w_hd, const void* ps1, int T, int d, int d_e, int d_head, int j,
                                    float eps_norm, float* P, float* rowstat, void* u, hipStream_t s) {
  using C = TileRouterSmall;
  static_assert(C::OUT_N == 128, "d_e + d_head is a multiple of 128");
  const int N = d_e + d_head, splits = router_gemm_splits(1, d, T, N);
  const int mt = (T + C::BM - 1) / C::BM, nt = N / C::OUT_N, tiles = (mt * nt + 7) / 8 * 8;
  EpiStoreF32Rows epi{{P, N, static_cast<size_t>(T) * N}, tiles, T, d, j, static_cast<const bf16_t*>(hbar),
                      static_cast<const bf16_t*>(prev1), static_cast<const bf16_t*>(prev2),
                      static_cast<const bf16_t*>(norm_w), eps_norm, rowstat, static_cast<bf16_t*>(u)};
  ARows<bf16_t> A{static_cast<const bf16_t*>(hbar), nullptr, d};
  BRows<bf16_t> B{static_cast<const bf16_t*>(w_hd), static_cast<const bf16_t*>(ps1), d_e, d};
  const dim3 grid(tiles + (T + splits - 1) / splits, splits);
  mfma_gemm<C, EpiStoreF32Rows><<<grid, C::NT, 0, s>>>(A, B, epi, nullptr, T, d, mt, nt);
  return hipGetLastError();
}

bool f32_head_fits(int dtype, int T, int N) { return dtype != 1 && !f32_tiles_large(T, N); }

hipError_t launch_f32_head(const void* hbar, const void* prev1, const void* prev2, const void* norm_w,
                           const void* w_hd, const void* ps1, int T, int d, int d_e, int d_head, int j,
                           float eps_norm, float* P, float* rowstat, void* u, hipStream_t s) {
  const int N = d_e + d_head;
  const F32Job<EpiStoreF32> g{{static_cast<const float*>(hbar), nullptr, d},
                              {static_cast<const float*>(w_hd), static_cast<const float*>(ps1), d_e, d},
                              {P, N, static_cast<size_t>(T) * N}, T, N, d};
  const int tiles = g.tiles();
  const auto run = [&](auto kernel) {
    kernel<<<tiles + T, 256, 0, s>>>(g.A, g.B, g.epi, T, N, d, g.mt(), tiles, static_cast<const float*>(prev1),
                                     static_cast<const float*>(prev2), static_cast<const float*>(norm_w), j, eps_norm,
                                     rowstat, static_cast<float*>(u));
  };
  if (g.vec())
    run(f32_head<true>);
  else
    run(f32_head<false>);
  return hipGetLastError();
}

hipError_t launch_router_gemm(int dtype, const void* hbar, const void* w_hd, const void* ps1, int T,
                              int d, int d_e, int d_head, float* P, hipStream_t s) {
  const int N = d_e + d_head;
  EpiStoreF32 epi{P, N, static_cast<size_t>(T) * N};
  if (dtype == 1) {
    ARows<bf16_t> A{static_cast<const bf16_t*>(hbar), nullptr, d};
    BRows<bf16_t> B{static_cast<const bf16_t*>(w_hd), static_cast<const bf16_t*>(ps1), d_e, d};
    const int splits = router_gemm_splits(dtype, d, T, N);
    if (T <= 1024 && N % TileRouterSmall::OUT_N == 0)
      return run_tile<TileRouterSmall>(A, B, epi, nullptr, T, N, d, s, splits);
    // a full round or more of tiles: the FFN products' core (32768 tokens: 256 tiles of 256 x 256,
    // no K split)
    if (splits == 1 && T >= 16384 && N % 256 == 0) return run_phase<false>(A, B, epi, nullptr, T, N, d, s);
    if (N % TileRouter::OUT_N == 0) return run_tile<TileRouter>(A, B, epi, nullptr, T, N, d, s, splits);
    return run_tile<TileRouterNarrow>(A, B, epi, nullptr, T, N, d, s, splits);
  }
  ARows<float> A{static_cast<const float*>(hbar), nullptr, d};
  BRows<float> B{static_cast<const float*>(w_hd), static_cast<const float*>(ps1), d_e, d};
  return run_f32<false>(A, B, epi, nullptr, T, N, d, s);
}

namespace {

// ---------------------------------------------------------------------------
// FFN products with few rows (a decode batch): the plain launch has fewer output tiles than
// half the CUs, each streaming the whole of K.  K is then split S ways (the most that keeps
// the launch within one round of workgroups), the slices write fp32 partial sums, and a pass
// over them adds the S slices in a fixed order and finishes the epilogue.
// ---------------------------------------------------------------------------
using TileSplitGU = Tile<192, 256, 2, 4>;    // [W_g; W_u] as one 2 d_ff-row operand
constexpr int kMaxSplitGU = 8, kMaxSplitDown = 16;

// At most 256 rows (a decode batch): the skinny products.  Gate/up: one workgroup per CU, each
// with 2-4 blocks of 16 columns of W_g and W_u and the whole of K.  Down: blocks of 8 x 16 output
// columns by kSkinnyDownS K-slices, whose fp32 partial sums a pass adds in a fixed order.
constexpr int kSkinnyRows = kDecodeTokens, kSkinnyDownNB = 8, kSkinnyDownS = 8;
static_assert(kSkinnyRows <= 4 * 64, "the row blocks of skinny_gateup_nb");
bool skinny_gateup_fits(int n_max, int d, int d_ff) {
  const int nb = d_ff / 16;
  return n_max <= kSkinnyRows && d % BK == 0 && d_ff % 16 == 0 && nb <= 4 * kCUs;
}
int skinny_down_splits(int d, int d_ff) {
  const int G = d / (16 * kSkinnyDownNB), nkt = d_ff / BK;
  return std::max(1, std::min({kSkinnyDownS, kCUs / std::max(G, 1), nkt}));
}
bool skinny_down_fits(int n_max, int d, int d_ff) {
  return n_max <= kSkinnyRows && d % (16 * kSkinnyDownNB) == 0 && d_ff % BK == 0;
}

// route (may be null): the launch is a routed decode step's (decode_route)
struct GateUpCall {
  ARows<bf16_t> A;
  const bf16_t *wg, *wu, *tiled;
  bf16_t* act;
  const int* counts;
  int n_max, d, d_ff;
  const RouteArgs* route;
};

template <int NB, int RB>
hipError_t skinny_gateup_nb_rb(const GateUpCall& c, hipStream_t s) {
  using C = Skinny<NB, RB, 3, skinny_nsb(NB, RB, true, 3), true>;
  const int nb = c.d_ff / 16;
  const bf16_t *b0 = c.tiled ? c.tiled : c.wg, *b1 = c.tiled ? nullptr : c.wu;
  const int ldb = c.tiled ? 0 : c.d, tiled = c.tiled ? nb : 0;
  if (c.route) {
    // as few workgroups as keep the most blocks of one, in whole eights: each streams the activations
    // (256 tokens, with all the CUs that the adapter leaves: 8B layer 140 us, so 136)
    const int G = std::min(nb, ((nb + NB - 1) / NB + 7) / 8 * 8);
    skinny_gemm<C, true><<<c.route->na + G, 512, 0, s>>>(c.A, b0, b1, ldb, tiled, c.act, c.d_ff, 0, nullptr, c.n_max,
                                                         c.d, nb, G, 1, *c.route);
    return hipGetLastError();
  }
  return run_skinny<C>(c.A, b0, b1, ldb, tiled, c.act, c.d_ff, 0, c.counts, c.n_max, c.d, nb, std::min(kCUs, nb), 1, s);
}
template <int NB>
hipError_t skinny_gateup_nb(const GateUpCall& c, hipStream_t s) {
  switch ((c.n_max + 63) / 64) {
    case 1: return skinny_gateup_nb_rb<NB, 1>(c, s);
    case 2: return skinny_gateup_nb_rb<NB, 2>(c, s);
    case 3: return skinny_gateup_nb_rb<NB, 3>(c, s);
    default: return skinny_gateup_nb_rb<NB, 4>(c, s);
  }
}
int skinny_gateup_blocks(int d_ff) {   // most blocks a workgroup takes
  const int nb = d_ff / 16, G = std::min(kCUs, nb);
  return (nb + G - 1) / G;
}
hipError_t skinny_gateup(const GateUpCall& c, hipStream_t s) {
  switch (skinny_gateup_blocks(c.d_ff)) {
    case 1: return skinny_gateup_nb<1>(c, s);
    case 2: return skinny_gateup_nb<2>(c, s);
    case 3: return skinny_gateup_nb<3>(c, s);
    default: return skinny_gateup_nb<4>(c, s);
  }
}
template <int RB>
hipError_t skinny_down_rb(ARows<bf16_t> A, const bf16_t* wd, const bf16_t* tiled, float* part, size_t stride,
                          const int* counts, int n_max, int d, int d_ff, int S, hipStream_t s) {
  using C = Skinny<kSkinnyDownNB, RB, 3, skinny_nsb(kSkinnyDownNB, RB, false, 3), false>;
  const int nb = d / 16;
  if (tiled)
    return run_skinny<C>(A, tiled, nullptr, 0, nb, part, d, stride, counts, n_max, d_ff, nb, nb / kSkinnyDownNB, S, s);
  return run_skinny<C>(A, wd, nullptr, d_ff, 0, part, d, stride, counts, n_max, d_ff, nb, nb / kSkinnyDownNB, S, s);
}
hipError_t skinny_down(ARows<bf16_t> A, const bf16_t* wd, const bf16_t* tiled, float* part, size_t stride,
                       const int* counts, int n_max, int d, int d_ff, int S, hipStream_t s) {
  switch ((n_max + 63) / 64) {
    case 1: return skinny_down_rb<1>(A, wd, tiled, part, stride, counts, n_max, d, d_ff, S, s);
    case 2: return skinny_down_rb<2>(A, wd, tiled, part, stride, counts, n_max, d, d_ff, S, s);
    case 3: return skinny_down_rb<3>(A, wd, tiled, part, stride, counts, n_max, d, d_ff, S, s);
    default: return skinny_down_rb<4>(A, wd, tiled, part, stride, counts, n_max, d, d_ff, S, s);
  }
}

int split_ways(int tiles, int nkt, int cap) {
  if (tiles <= 0 || 2 * tiles > kCUs) return 1;
  return std::max(1, std::min({cap, kCUs / tiles, nkt}));
}
int gateup_split(int n, int d, int d_ff) {
  return split_ways((n + TileSplitGU::BM - 1) / TileSplitGU::BM * (2 * d_ff / TileSplitGU::OUT_N),
                    d / BK, kMaxSplitGU);
}
// K-slices that the workspace holds for the down product of n rows (192 x 128 tiles: the layout that
// the workspace size and the no-allocation limit are stated for)
int down_split_space(int n, int d, int d_ff) {
  return split_ways((n + 191) / 192 * (d / 128), d_ff / BK, kMaxSplitDown);
}
// ... and that its 128 x 256 tiles take: the most that fit one round of workgroups, of at least two
// k-tiles.  8B shape, 390 of at most 640 rows: 85 us in two slices of 192 x 128 tiles, 65 in three.
int down_split(int n, int d, int d_ff) {
  const int S = split_ways((n + 127) / 128 * (d / 256), d_ff / BK / 2, kMaxSplitDown);
  const size_t space = ffn_part_floats(1, d, d_ff, n) / (static_cast<size_t>(n) * d);
  return std::max(1, std::min(S, static_cast<int>(std::min<size_t>(space, kMaxSplitDown))));
}

// act[m][c] = bf16(SiLU(g) u) with g, u the sums over z < S of P[z][m][c] and P[z][m][d_ff + c];
// one thread per 8 columns of a row, rows m < *m_count
__global__ __launch_bounds__(256) void swiglu_reduce(const float* __restrict__ P, int S,
                                                    size_t stride, const int* __restrict__ m_count,
                                                    int n_max, int d_ff, bf16_t* __restrict__ act) {
  const int M = m_count ? min(*m_count, n_max) : n_max;
  const int q = d_ff / 8;
  const size_t e = static_cast<size_t>(blockIdx.x) * 256 + threadIdx.x;
  const int m = static_cast<int>(e / q), c = static_cast<int>(e % q) * 8;
  if (m >= M) return;
  const float* p = P + static_cast<size_t>(m) * 2 * d_ff + c;
  f32x4 g0 = *reinterpret_cast<const f32x4*>(p), g1 = *reinterpret_cast<const f32x4*>(p + 4);
  f32x4 u0 = *reinterpret_cast<const f32x4*>(p + d_ff), u1 = *reinterpret_cast<const f32x4*>(p + d_ff + 4);
  for (int z = 1; z < S; ++z) {
    const float* pz = p + z * stride;
    g0 += *reinterpret_cast<const f32x4*>(pz);
    g1 += *reinterpret_cast<const f32x4*>(pz + 4);
    u0 += *reinterpret_cast<const f32x4*>(pz + d_ff);
    u1 += *reinterpret_cast<const f32x4*>(pz + d_ff + 4);
  }
  u32x4 w;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const float ga = i < 2 ? g0[2 * i] : g1[2 * i - 4], gb = i < 2 ? g0[2 * i + 1] : g1[2 * i - 3];
    const float ua = i < 2 ? u0[2 * i] : u1[2 * i - 4], ub = i < 2 ? u0[2 * i + 1] : u1[2 * i - 3];
    const float lo = ga * __builtin_amdgcn_rcpf(1.0f + __expf(-ga)) * ua;
    const float hi = gb * __builtin_amdgcn_rcpf(1.0f + __expf(-gb)) * ub;
    w[i] = static_cast<uint32_t>(f32_to_bf16(lo)) | (static_cast<uint32_t>(f32_to_bf16(hi)) << 16);
  }
  *reinterpret_cast<u32x4*>(act + static_cast<size_t>(m) * d_ff + c) = w;
}

// h_out[t][n] = bf16(hbar[t][n] + g_t y) with y the sum over z < S of P[z][m][n], t = idx[m];
// one thread per 8 columns of a row, rows m < *m_count
__device__ __forceinline__ void scatter_reduce_block(int block, const float* __restrict__ P, int S, size_t stride,
                                                     const int* __restrict__ m_count, int n_max,
                                                     const int* __restrict__ idx,
                                                     const bf16_t* __restrict__ hbar,
                                                     const float* __restrict__ gate,
                                                     bf16_t* __restrict__ out, int d) {
  const int M = m_count ? min(*m_count, n_max) : n_max;
  const int q = d / 8;
  const size_t e = static_cast<size_t>(block) * 256 + threadIdx.x;
  const int m = static_cast<int>(e / q), n = static_cast<int>(e % q) * 8;
  if (m >= M) return;
  const float* p = P + static_cast<size_t>(m) * d + n;
  f32x4 y0 = *reinterpret_cast<const f32x4*>(p), y1 = *reinterpret_cast<const f32x4*>(p + 4);
  for (int z = 1; z < S; ++z) {
    y0 += *reinterpret_cast<const f32x4*>(p + z * stride);
    y1 += *reinterpret_cast<const f32x4*>(p + z * stride + 4);
  }
  const int t = idx ? idx[m] : m;
  const float sc = gate ? gate[t] : 1.0f;
  const size_t o = static_cast<size_t>(t) * d + n;
  const u32x4 h = *reinterpret_cast<const u32x4*>(hbar + o);
  u32x4 w;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const float ya = i < 2 ? y0[2 * i] : y1[2 * i - 4], yb = i < 2 ? y0[2 * i + 1] : y1[2 * i - 3];
    const float lo = __uint_as_float(h[i] << 16) + sc * ya;
    const float hi = __uint_as_float(h[i] & 0xffff0000u) + sc * yb;
    w[i] = static_cast<uint32_t>(f32_to_bf16(lo)) | (static_cast<uint32_t>(f32_to_bf16(hi)) << 16);
  }
  *reinterpret_cast<u32x4*>(out + o) = w;
}

__global__ __launch_bounds__(256) void scatter_reduce(const float* __restrict__ P, int S, size_t stride,
                                                     const int* __restrict__ m_count, int n_max,
                                                     const int* __restrict__ idx,
                                                     const bf16_t* __restrict__ hbar,
                                                     const float* __restrict__ gate,
                                                     bf16_t* __restrict__ out, int d) {
  scatter_reduce_block(static_cast<int>(blockIdx.x), P, S, stride, m_count, n_max, idx, hbar, gate, out, d);
}

// The last launch of a routed decode step: the first up_blocks workgroups are the adapter's
// up-projection (32 rows x 256 columns each, z by token), the others scatter_reduce.  The
// two write disjoint rows of h_out.
template <int KR>
__global__ __launch_bounds__(256) void decode_finish(RouteFinish f) {
  const int b = static_cast<int>(blockIdx.x);
  if (b < f.up_blocks) {
    const int nc = f.d / 256;
    adapter_up_tile<KR, 1, true>(f.z, f.idx_ad, f.counts + 1, f.w2, f.hbar, f.gate, f.out, f.T, f.d,
                                 b / nc * 32, b % nc * 256);
  } else {
    scatter_reduce_block(b - f.up_blocks, f.part, f.S, f.stride, f.counts, f.n_ffn_max, f.idx_ffn, f.hbar, f.gate,
                         f.out, f.d);
  }
}

// out[((kt NB + b) G + g) 16 + r][c] = W_g[16 b + r][64 kt + c] with NB = N / 16 blocks (w0: g = 0,
// w1: g = 1); one thread per 16-byte piece of the output, so the writes are contiguous and each
// group of eight threads reads one 128-byte run of a source row.
__global__ __launch_bounds__(256) void tile_ffn_weights_kernel(const bf16_t* __restrict__ w0,
                                                              const bf16_t* __restrict__ w1, int G, int K,
                                                              size_t pieces, bf16_t* __restrict__ out) {
  const size_t e = static_cast<size_t>(blockIdx.x) * 256 + threadIdx.x;
  if (e >= pieces) return;
  const int c8 = static_cast<int>(e & 7), r = static_cast<int>((e >> 3) & 15);
  const size_t t = e >> 7;                       // (kt NB + b) G + g
  const int g = static_cast<int>(t % G);
  const size_t bk = t / G;
  const size_t NB = pieces / (static_cast<size_t>(K / BK) * G * 128);
  const size_t b = bk % NB;
  const int kt = static_cast<int>(bk / NB);
  const bf16_t* src = (g ? w1 : w0) + (16 * b + r) * static_cast<size_t>(K) + kt * BK + 8 * c8;
  *reinterpret_cast<u32x4*>(out + 8 * e) = *reinterpret_cast<const u32x4*>(src);
}

}  // namespace

size_t ffn_part_floats(int dtype, int d, int d_ff, int T) {
  if (dtype != 1 || T <= 0) return 0;
  // S is fixed per row-tile count and the slices hold n rows: the largest n of each count
  size_t most = 0;
  const int ns = std::min(T, kSkinnyRows);
  if (skinny_down_fits(ns, d, d_ff)) most = static_cast<size_t>(skinny_down_splits(d, d_ff)) * ns * d;
  for (int mt = 1; (mt - 1) * TileSplitGU::BM < T; ++mt) {
    const int n = std::min(mt * TileSplitGU::BM, T);
    const int sg = gateup_split(n, d, d_ff), sd = down_split_space(n, d, d_ff);
    if (sg > 1) most = std::max(most, static_cast<size_t>(sg) * n * 2 * d_ff);
    if (sd > 1) most = std::max(most, static_cast<size_t>(sd) * n * d);
    if (sg == 1 && sd == 1) break;   // both counts only grow from here
  }
  return most;
}

hipError_t launch_tile_ffn_weights(const void* w0, const void* w1, int N, int K, void* out, hipStream_t s) {
  if (N <= 0 || K <= 0 || N % 16 != 0 || K % BK != 0) return hipErrorInvalidValue;
  const int G = w1 ? 2 : 1;
  const size_t pieces = static_cast<size_t>(N) * (K / 8) * G;
  tile_ffn_weights_kernel<<<static_cast<unsigned>((pieces + 255) / 256), 256, 0, s>>>(
      static_cast<const bf16_t*>(w0), static_cast<const bf16_t*>(w1), G, K, pieces, static_cast<bf16_t*>(out));
  return hipGetLastError();
}

hipError_t launch_ffn_gateup(int dtype, const void* u, const int* idx_ffn, const int* counts,
                             int n_max, const void* w_gate, const void* w_up, const void* w_gate_up_tiled,
                             void* act, float* part, int d, int d_ff, bool exact, hipStream_t s) {
  if (n_max <= 0) return hipSuccess;
  if (dtype == 1) {
    ARows<bf16_t> A{static_cast<const bf16_t*>(u), idx_ffn, d};
    if (skinny_gateup_fits(n_max, d, d_ff))
      return skinny_gateup({A, static_cast<const bf16_t*>(w_gate), static_cast<const bf16_t*>(w_up),
                            static_cast<const bf16_t*>(w_gate_up_tiled), static_cast<bf16_t*>(act), counts, n_max, d,
                            d_ff, nullptr}, s);
    const int S = gateup_split(n_max, d, d_ff);
    if (S > 1) {
      BRows<bf16_t> B{static_cast<const bf16_t*>(w_gate), static_cast<const bf16_t*>(w_up), d_ff, d};
      const size_t stride = static_cast<size_t>(n_max) * 2 * d_ff;
      hipError_t e = run_tile<TileSplitGU>(A, B, EpiStoreF32{part, 2 * d_ff, stride}, counts, n_max,
                                           2 * d_ff, d, s, S);
      if (e != hipSuccess) return e;
      const size_t n8 = static_cast<size_t>(n_max) * (d_ff / 8);
      swiglu_reduce<<<static_cast<unsigned>((n8 + 255) / 256), 256, 0, s>>>(
          part, S, stride, counts, n_max, d_ff, static_cast<bf16_t*>(act));
      return hipGetLastError();
    }
    BRows<bf16_t> B{static_cast<const bf16_t*>(w_gate), static_cast<const bf16_t*>(w_up), INT_MAX, d};
    return run_phase<true>(A, B, EpiSwiGLU<bf16_t>{static_cast<bf16_t*>(act), d_ff}, counts, n_max, d_ff, d, s, exact);
  }
  ARows<float> A{static_cast<const float*>(u), idx_ffn, d};
  BRows<float> B{static_cast<const float*>(w_gate), static_cast<const float*>(w_up), INT_MAX, d};
  return run_f32<true>(A, B, EpiSwiGLU<float>{static_cast<float*>(act), d_ff}, counts, n_max, d_ff,
                       d, s);
}

hipError_t launch_ffn_down(int dtype, const void* act, const int* idx_ffn, const int* counts,
                           int n_max, const void* w_down, const void* w_down_tiled, const void* hbar,
                           const float* gate, void* h_out, float* part, int d, int d_ff, bool exact, hipStream_t s) {
  if (n_max <= 0) return hipSuccess;
  if (dtype == 1) {
    ARows<bf16_t> A{static_cast<const bf16_t*>(act), nullptr, d_ff};
    BRows<bf16_t> B{static_cast<const bf16_t*>(w_down), nullptr, INT_MAX, d_ff};
    const bool skinny = skinny_down_fits(n_max, d, d_ff);
    const int S = skinny ? skinny_down_splits(d, d_ff) : down_split(n_max, d, d_ff);
    if (S > 1 || skinny) {
      const size_t stride = static_cast<size_t>(n_max) * d;
      hipError_t e = skinny ? skinny_down(A, static_cast<const bf16_t*>(w_down),
                                          static_cast<const bf16_t*>(w_down_tiled), part, stride, counts,
                                          n_max, d, d_ff, S, s)
                            : run_phase_split(A, B, EpiStoreF32{part, d, stride}, counts, n_max, d, d_ff, S, s);
      if (e != hipSuccess) return e;
      const size_t n8 = static_cast<size_t>(n_max) * (d / 8);
      scatter_reduce<<<static_cast<unsigned>((n8 + 255) / 256), 256, 0, s>>>(
          part, S, stride, counts, n_max, idx_ffn, static_cast<const bf16_t*>(hbar), gate,
          static_cast<bf16_t*>(h_out), d);
      return hipGetLastError();
    }
    EpiScatter<bf16_t, false> epi{idx_ffn, static_cast<const bf16_t*>(hbar), gate,
                                  static_cast<bf16_t*>(h_out), d};
    return run_phase<false>(A, B, epi, counts, n_max, d, d_ff, s, exact);
  }
  ARows<float> A{static_cast<const float*>(act), nullptr, d_ff};
  BRows<float> B{static_cast<const float*>(w_down), nullptr, INT_MAX, d_ff};
  EpiScatter<float, false> epi{idx_ffn, static_cast<const float*>(hbar), gate,
                               static_cast<float*>(h_out), d};
  return run_f32<false>(A, B, epi, counts, n_max, d, d_ff, s);
}

// ---------------------------------------------------------------------------
// Attention projections of a decoder block (Sec. 3.1, eq:dense_attention).
// [q; k; v] = x [W_q; W_k; W_v]^T runs on the GEMM core with an epilogue that applies the
// rotary embedding to q and k (pair (2i, 2i+1) of a head turned by pos * inv_freq[i]: a
// table of cos and sin for the call's positions, made once in fp32) and writes each head
// where the attention kernel reads it: q [B][n_h][S_pad][128], k [B][n_kv][S_pad][128] and
// v transposed, [B][n_kv][128][S_pad] with positions permuted within groups of 16 (the
// attention kernel's key order), written as 16-byte runs.  The output projection
// adds its product to the block input: hbar = h + o W_o^T.
// ---------------------------------------------------------------------------
namespace {

constexpr int kHeadDim = 128;

struct EpiQKV {
  bf16_t* q;
  bf16_t* k;
  bf16_t* vt;
  const float2* cs;   // [seq][64] (cos, sin) of pos * inv_freq[i]
  int seq, seq_pad, nh, nkv;
  struct Pre {};
  __device__ __forceinline__ Pre prep(int, int) const { return {}; }
  __device__ __forceinline__ void store(int, int, float) const {}
  __device__ __forceinline__ void emit8(const Pre&, int, int, const float*) const {}
  // a staged block of 16 token rows x `on` columns of one head (on | 128) starting at row mb,
  // column nb
  __device__ __forceinline__ void block(const float* stg, int opad, int on, int mb, int nb, int M,
                                        int lane) const {
    const int head = nb / kHeadDim, c0 = nb % kHeadDim;
    if (head < nh + nkv) {
      // q or k: 8-column row pieces, turned by the rotary table
      const int cpr = on / 8;
      for (int e = lane; e < 16 * cpr; e += kWave) {
        const int i = e / cpr, c8 = (e % cpr) * 8;
        const int m = mb + i;
        if (m >= M) continue;
        const int b = m / seq, pos = m - b * seq;
        const int c = c0 + c8;
        const float* v = stg + i * opad + c8;
        const float2* t = cs + static_cast<size_t>(pos) * (kHeadDim / 2) + c / 2;
        u32x4 w;
#pragma unroll
        for (int x = 0; x < 4; ++x) {
          const float2 r = t[x];
          const float a = v[2 * x], bb = v[2 * x + 1];
          w[x] = static_cast<uint32_t>(f32_to_bf16(a * r.x - bb * r.y)) |
                 (static_cast<uint32_t>(f32_to_bf16(a * r.y + bb * r.x)) << 16);
        }
        bf16_t* dst = head < nh
            ? q + ((static_cast<size_t>(b) * nh + head) * seq_pad + pos) * kHeadDim + c
            : k + ((static_cast<size_t>(b) * nkv + (head - nh)) * seq_pad + pos) * kHeadDim + c;
        *reinterpret_cast<u32x4*>(dst) = w;
      }
    } else {
      // v, transposed, positions permuted within each group of 16 (position p at slot
      // p with bits 2 and 3 swapped: 0-3, 8-11, 4-7, 12-15): a piece is one column over the
      // 8 positions 16G + 4X + {0..3} and 16G + 8 + 4X + {0..3} of the block, one 16-byte run
      const int vh = head - nh - nkv;
      for (int e = lane; e < 2 * on; e += kWave) {
        const int col = e % on, X = e / on;
        if (mb >= M) continue;
        const int b = mb / seq, p16 = mb - b * seq;
        bf16_t* row = vt + ((static_cast<size_t>(b) * nkv + vh) * kHeadDim + c0 + col) * seq_pad;
        if (mb + 15 < M && p16 + 15 < seq && (p16 & 15) == 0) {
          u32x4 w;
#pragma unroll
          for (int x = 0; x < 4; ++x) {
            const int r0 = x < 2 ? 4 * X + 2 * x : 8 + 4 * X + 2 * (x - 2);
            w[x] = static_cast<uint32_t>(f32_to_bf16(stg[r0 * opad + col])) |
                   (static_cast<uint32_t>(f32_to_bf16(stg[(r0 + 1) * opad + col])) << 16);
          }
          *reinterpret_cast<u32x4*>(row + p16 + 8 * X) = w;
        } else {
          for (int x = 0; x < 8; ++x) {
            const int r = x < 4 ? 4 * X + x : 8 + 4 * X + x - 4;
            const int mm = mb + r;
            if (mm >= M) continue;
            const int bx = mm / seq, px = mm - bx * seq;
            const int slot = (px & ~15) | (px & 3) | ((px & 4) << 1) | ((px & 8) >> 1);
            vt[((static_cast<size_t>(bx) * nkv + vh) * kHeadDim + c0 + col) * seq_pad + slot] =
                f32_to_bf16(stg[r * opad + col]);
          }
        }
      }
    }
  }
};

__global__ void rope_table_kernel(float2* __restrict__ cs, int seq, RopeTable rope) {
  const int e = blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= seq * (kHeadDim / 2)) return;
  const int pos = e / (kHeadDim / 2), i = e % (kHeadDim / 2);
  float sn, c;
  sincosf(static_cast<float>(pos) * rope.inv_freq[i], &sn, &c);
  cs[e] = make_float2(c, sn);
}

}  // namespace

hipError_t launch_rope_table(int seq, const RopeTable& rope, float* cs, hipStream_t s) {
  const int n = seq * (kHeadDim / 2);
  if (n <= 0) return hipSuccess;
  rope_table_kernel<<<(n + 255) / 256, 256, 0, s>>>(reinterpret_cast<float2*>(cs), seq, rope);
  return hipGetLastError();
}

hipError_t launch_attn_qkv(const void* x, const void* w_qkv, int T, int d, int seq, int seq_pad, int nh,
                           int nkv, const float* rope_cs, void* q, void* k, void* vt, hipStream_t s) {
  if (T <= 0) return hipSuccess;
  ARows<bf16_t> A{static_cast<const bf16_t*>(x), nullptr, d};
  BRows<bf16_t> B{static_cast<const bf16_t*>(w_qkv), nullptr, INT_MAX, d};
  EpiQKV epi{static_cast<bf16_t*>(q), static_cast<bf16_t*>(k), static_cast<bf16_t*>(vt),
             reinterpret_cast<const float2*>(rope_cs), seq, seq_pad, nh, nkv};
  return run_phase<false>(A, B, epi, nullptr, T, (nh + 2 * nkv) * kHeadDim, d, s);
}

hipError_t launch_attn_out(const void* o, const void* w_o, const void* h, void* hbar, int T, int d, int nh,
                           hipStream_t s) {
  if (T <= 0) return hipSuccess;
  const int K = nh * kHeadDim;
  ARows<bf16_t> A{static_cast<const bf16_t*>(o), nullptr, K};
  BRows<bf16_t> B{static_cast<const bf16_t*>(w_o), nullptr, INT_MAX, K};
  EpiScatter<bf16_t, false> epi{nullptr, static_cast<const bf16_t*>(h), nullptr, static_cast<bf16_t*>(hbar), d};
  return run_phase<false>(A, B, epi, nullptr, T, d, K, s);
}

// Wide adapters (ranks above 128, in steps of 128: the paper's d_r = 896).  The down-projection
// runs on the MFMA GEMM core with K split WIDE_SPLIT ways into fp32 partials, a reduction pass forms
// hid = bf16(SiLU(sum of the partials)), and the up-projection is a GEMM whose epilogue scatters
// hbar + (1 - g) (W_2 hid) into the adapter rows.
constexpr int WIDE_SPLIT = 4;
using TileWide = Tile<128, 128, 2, 4>;

bool adapter_wide(int d_r) { return d_r > 128; }

size_t adapter_part_floats(int dtype, int d, int d_r, int T) {
  if (dtype == 1 && adapter_wide(d_r))   // partials, then hid (bf16, half a float per element)
    return static_cast<size_t>(WIDE_SPLIT) * T * d_r + static_cast<size_t>(T) * d_r / 2;
  const int G = dtype == 1 ? adapter_groups(d) : 1;
  return static_cast<size_t>(G) * T * d_r;
}

namespace {

// hid[m][n] = bf16(SiLU(sum_z part[z][m][n])) for m < *m_count, eight columns per thread
__global__ __launch_bounds__(256) void adapter_hidden_wide(const float* __restrict__ part, size_t split_stride,
                                                           const int* __restrict__ m_count, int d_r,
                                                           bf16_t* __restrict__ hid) {
  const size_t n8 = static_cast<size_t>(*m_count) * d_r / 8;
  for (size_t e = blockIdx.x * static_cast<size_t>(256) + threadIdx.x; e < n8;
       e += static_cast<size_t>(gridDim.x) * 256) {
    f32x4 x[WIDE_SPLIT][2];
#pragma unroll
    for (int z = 0; z < WIDE_SPLIT; ++z) {
      const float* p = part + z * split_stride + 8 * e;
      x[z][0] = *reinterpret_cast<const f32x4*>(p);
      x[z][1] = *reinterpret_cast<const f32x4*>(p + 4);
    }
    float h[8];
#pragma unroll
    for (int c = 0; c < 8; ++c) {
      float v = 0.f;
#pragma unroll
      for (int z = 0; z < WIDE_SPLIT; ++z) v += x[z][c >> 2][c & 3];
      h[c] = siluf_(v);
    }
    st8(hid + 8 * e, h);
  }
}

}  // namespace

namespace {

// K-sliced partials of rows[idx[m]] W^T for the register-tiled ranks (32 .. 128); with u2 set, a
// second product over the same rows in the same launch (gridDim.z = 2)
hipError_t adapter_down_small(const bf16_t* uu, const int* idx_ad, const int* counts, int n_max, const bf16_t* ww,
                              float* part, int d, int d_r, hipStream_t s, const bf16_t* u2, const bf16_t* w2_,
                              float* p2, int G) {
  dim3 g1((n_max + 31) / 32, G, u2 ? 2 : 1);
  // the adapter rank is a compile-time count of 32-column MFMA tiles
  const bool b8 = adapter_batch(d, G) == 8;
#define HERO_ADAPTER_DOWN(TN_)                                                                       \
  (b8 ? adapter_down_bf16<TN_, 8><<<g1, 256, 0, s>>>(uu, idx_ad, counts, ww, part, n_max, d, d / G, u2, w2_, p2) \
      : adapter_down_bf16<TN_, 4><<<g1, 256, 0, s>>>(uu, idx_ad, counts, ww, part, n_max, d, d / G, u2, w2_, p2))
  switch (d_r) {
    case 32: HERO_ADAPTER_DOWN(1); break;
    case 64: HERO_ADAPTER_DOWN(2); break;
    case 96: HERO_ADAPTER_DOWN(3); break;
    case 128: HERO_ADAPTER_DOWN(4); break;
    default: return hipErrorInvalidValue;
  }
#undef HERO_ADAPTER_DOWN
  return hipGetLastError();
}

}  // namespace

hipError_t launch_adapter_down(int dtype, const void* u, const int* idx_ad, const int* counts,
                               int n_max, const void* w1, float* part, int d, int d_r,
                               hipStream_t s) {
  if (n_max <= 0) return hipSuccess;
  if (dtype == 1 && adapter_wide(d_r)) {
    ARows<bf16_t> A{static_cast<const bf16_t*>(u), idx_ad, d};
    BRows<bf16_t> B{static_cast<const bf16_t*>(w1), nullptr, INT_MAX, d};
    const size_t stride = static_cast<size_t>(n_max) * d_r;
    hipError_t e = run_tile<TileWide>(A, B, EpiStoreF32{part, d_r, stride}, counts, n_max, d_r, d, s, WIDE_SPLIT);
    if (e != hipSuccess) return e;
    bf16_t* hid = reinterpret_cast<bf16_t*>(part + WIDE_SPLIT * stride);
    const int blocks = static_cast<int>(std::min<size_t>((stride / 8 + 255) / 256, 2048));
    adapter_hidden_wide<<<blocks, 256, 0, s>>>(part, stride, counts, d_r, hid);
    return hipGetLastError();
  }
  if (dtype == 1)
    return adapter_down_small(static_cast<const bf16_t*>(u), idx_ad, counts, n_max, static_cast<const bf16_t*>(w1),
                              part, d, d_r, s, nullptr, nullptr, nullptr, adapter_groups_rows(d, n_max));
  // fp32: hid = SiLU(u W_1^T) into part[m][n]
  ARows<float> A{static_cast<const float*>(u), idx_ad, d};
  BRows<float> B{static_cast<const float*>(w1), nullptr, INT_MAX, d};
  return run_f32<false>(A, B, EpiSiLU<float>{part, d_r}, counts, n_max, d_r, d, s);
}

hipError_t launch_adapter_up(int dtype, const float* part, const int* idx_ad, const int* counts,
                             int n_max, const void* w2, const void* hbar, const float* gate,
                             void* h_out, int d, int d_r, hipStream_t s) {
  if (n_max <= 0) return hipSuccess;
  if (dtype == 1 && adapter_wide(d_r)) {
    const bf16_t* hid =
        reinterpret_cast<const bf16_t*>(part + static_cast<size_t>(WIDE_SPLIT) * n_max * d_r);
    ARows<bf16_t> A{hid, nullptr, d_r};
    BRows<bf16_t> B{static_cast<const bf16_t*>(w2), nullptr, INT_MAX, d_r};
    EpiScatter<bf16_t, true> epi{idx_ad, static_cast<const bf16_t*>(hbar), gate, static_cast<bf16_t*>(h_out), d};
    return run_tile<TileWide>(A, B, epi, counts, n_max, d, d_r, s);
  }
  if (dtype == 1) {
    const int G = adapter_groups_rows(d, n_max);
    dim3 g2((n_max + 31) / 32, d / 256);
    const bf16_t* ww = static_cast<const bf16_t*>(w2);
    const bf16_t* hb = static_cast<const bf16_t*>(hbar);
    bf16_t* ho = static_cast<bf16_t*>(h_out);
    switch (d_r) {
      case 32: adapter_up_launch<32>(g2, s, G, part, idx_ad, counts, ww, hb, gate, ho, n_max, d); break;
      case 64: adapter_up_launch<64>(g2, s, G, part, idx_ad, counts, ww, hb, gate, ho, n_max, d); break;
      case 96: adapter_up_launch<96>(g2, s, G, part, idx_ad, counts, ww, hb, gate, ho, n_max, d); break;
      case 128: adapter_up_launch<128>(g2, s, G, part, idx_ad, counts, ww, hb, gate, ho, n_max, d); break;
      default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
  }
  ARows<float> A{part, nullptr, d_r};
  BRows<float> B{static_cast<const float*>(w2), nullptr, INT_MAX, d_r};
  EpiScatter<float, true> epi{idx_ad, static_cast<const float*>(hbar), gate,
                              static_cast<float*>(h_out), d};
  return run_f32<false>(A, B, epi, counts, n_max, d, d_r, s);
}

bool decode_route_fits(int dtype, int T, int n_ffn_max, int d, int d_ff, int d_r) {
  return dtype == 1 && T <= kDecodeTokens && n_ffn_max > 0 && !adapter_wide(d_r) && d % 256 == 0 &&
         skinny_gateup_fits(n_ffn_max, d, d_ff) && skinny_down_fits(n_ffn_max, d, d_ff);
}

// fp32, few tiles in each product: the decision rides with the first pair as long as one wave holds
// the tokens
bool f32_route_fits(int dtype, int T, int n_ffn_max, int n_ad_max, int d, int d_ff, int d_r) {
  return dtype != 1 && T <= kDecodeTokens && !f32_tiles_large(n_ffn_max, d_ff) && !f32_tiles_large(n_ffn_max, d) &&
         !f32_tiles_large(n_ad_max, d_r) && !f32_tiles_large(n_ad_max, d);
}

hipError_t launch_f32_route_in(const DecodeRoute& r, hipStream_t s) {
  const float* u = static_cast<const float*>(r.u);
  const F32Job<EpiSwiGLU<float>> f{{u, nullptr, r.d},
                                   {static_cast<const float*>(r.w_gate), static_cast<const float*>(r.w_up), INT_MAX, r.d},
                                   {static_cast<float*>(r.act), r.d_ff}, r.n_ffn_max, r.d_ff, r.d};
  const F32Job<EpiSiLU<float>> a{{u, nullptr, r.d}, {static_cast<const float*>(r.w1), nullptr, INT_MAX, r.d},
                                 {r.part_ad, r.d_r}, r.n_ad_max, r.d_r, r.d};
  return run_f32_pair<true, true>(f, a, r.sel, s);
}

hipError_t launch_f32_route_out(const DecodeRoute& r, hipStream_t s) {
  const float* hb = static_cast<const float*>(r.hbar);
  float* out = static_cast<float*>(r.h_out);
  const F32Job<EpiScatter<float, false>> f{{static_cast<const float*>(r.act), nullptr, r.d_ff},
                                           {static_cast<const float*>(r.w_down), nullptr, INT_MAX, r.d_ff},
                                           {r.sel.idx_ffn, hb, r.gate, out, r.d}, r.n_ffn_max, r.d, r.d_ff};
  const F32Job<EpiScatter<float, true>> a{{r.part_ad, nullptr, r.d_r},
                                          {static_cast<const float*>(r.w2), nullptr, INT_MAX, r.d_r},
                                          {r.sel.idx_ad, hb, r.gate, out, r.d}, r.n_ad_max, r.d, r.d_r};
  return run_f32_pair<false, false>(f, a, r.sel, s);
}

namespace {
// Width, in 32-column blocks, of the adapter's workgroups beside the gate/up product: the narrowest
// that leaves the product's workgroups a CU each
int route_width(int T, int d_ff, int d_r) {
  const int NB = skinny_gateup_blocks(d_ff), spare = kCUs - (d_ff / 16 + NB - 1) / NB;
  const int tiles = (T + 31) / 32, all = d_r / 32;
  int tn = 1;
  while (tn < all && (all % tn != 0 || tiles * (all / tn) > spare)) ++tn;
  return tn;
}
}  // namespace

hipError_t launch_route_gateup(const DecodeRoute& r, hipStream_t s) {
  RouteArgs ra{};
  ra.sel = r.sel;
  if (r.n_ad_max > 0) {
    ra.tn = route_width(r.sel.T, r.d_ff, r.d_r);
    ra.groups = adapter_groups(r.d);
    ra.na = ((r.sel.T + 31) / 32 * (r.d_r / 32 / ra.tn) + 7) / 8 * 8;
    ra.d_r = r.d_r;
    ra.u = static_cast<const bf16_t*>(r.u);
    ra.w1 = static_cast<const bf16_t*>(r.w1);
    ra.z = r.part_ad;
  }
  return skinny_gateup({ARows<bf16_t>{static_cast<const bf16_t*>(r.u), nullptr, r.d}, static_cast<const bf16_t*>(r.w_gate),
                        static_cast<const bf16_t*>(r.w_up), static_cast<const bf16_t*>(r.w_gate_up_tiled),
                        static_cast<bf16_t*>(r.act), nullptr, r.n_ffn_max, r.d, r.d_ff, &ra}, s);
}

hipError_t launch_route_down(const DecodeRoute& r, hipStream_t s) {
  const int S = skinny_down_splits(r.d, r.d_ff);
  return skinny_down(ARows<bf16_t>{static_cast<const bf16_t*>(r.act), nullptr, r.d_ff},
                     static_cast<const bf16_t*>(r.w_down), static_cast<const bf16_t*>(r.w_down_tiled), r.part,
                     static_cast<size_t>(r.n_ffn_max) * r.d, r.sel.counts, r.n_ffn_max, r.d, r.d_ff, S, s);
}

hipError_t launch_route_finish(const DecodeRoute& r, hipStream_t s) {
  RouteFinish f{};
  f.z = r.part_ad;
  f.idx_ad = r.sel.idx_ad;
  f.idx_ffn = r.sel.idx_ffn;
  f.counts = r.sel.counts;
  f.w2 = static_cast<const bf16_t*>(r.w2);
  f.hbar = static_cast<const bf16_t*>(r.hbar);
  f.gate = r.gate;
  f.out = static_cast<bf16_t*>(r.h_out);
  f.T = r.sel.T;
  f.d = r.d;
  f.up_blocks = r.n_ad_max > 0 ? (r.n_ad_max + 31) / 32 * (r.d / 256) : 0;
  f.part = r.part;
  f.S = skinny_down_splits(r.d, r.d_ff);
  f.n_ffn_max = r.n_ffn_max;
  f.stride = static_cast<size_t>(r.n_ffn_max) * r.d;
  const size_t n8 = static_cast<size_t>(r.n_ffn_max) * (r.d / 8);
  const int blocks = f.up_blocks + static_cast<int>((n8 + 255) / 256);
  switch (r.d_r) {
    case 32: decode_finish<32><<<blocks, 256, 0, s>>>(f); break;
    case 64: decode_finish<64><<<blocks, 256, 0, s>>>(f); break;
    case 96: decode_finish<96><<<blocks, 256, 0, s>>>(f); break;
    case 128: decode_finish<128><<<blocks, 256, 0, s>>>(f); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Backward of the routed block (frozen FFN, trained adapter) on the same cores.  The frozen
// weights enter through transposed copies, so every product keeps K contiguous:
//   e    = dL/dh[idx] W_d         B = W_d^T [d_ff][d]          (FFN rows)
//   G, U recomputed from u[idx]   B = W_g, W_u                 epilogue: EpiSwiGLUBwd
//   du   = [dG dU] [W_g; W_u]     B = [W_g; W_u]^T [d][2 d_ff]
// and the adapter's: z = u[idx] W_1^T, e_a = dL/dh[idx] W_2 (B = W_2^T), du = dz W_1 (B = W_1^T).
// ---------------------------------------------------------------------------
int swiglu_bwd_parts(int dtype, int d_ff) { return dtype == 1 ? d_ff / Phase<256, true>::ON : d_ff; }

hipError_t launch_ffn_bwd_e(int dtype, const void* dh, const int* idx_ffn, const int* counts, int n_max,
                            const void* w_down_t, void* e, int d, int d_ff, bool exact, hipStream_t s) {
  if (n_max <= 0) return hipSuccess;
  if (dtype == 1) {
    ARows<bf16_t> A{static_cast<const bf16_t*>(dh), idx_ffn, d};
    BRows<bf16_t> B{static_cast<const bf16_t*>(w_down_t), nullptr, INT_MAX, d};
    EpiStore<bf16_t> epi{static_cast<bf16_t*>(e), d_ff};
    return d_ff % 256 == 0 ? run_phase<false>(A, B, epi, counts, n_max, d_ff, d, s, exact)
                           : run_tile<Tile<256, 128, 2, 4>>(A, B, epi, counts, n_max, d_ff, d, s);
  }
  ARows<float> A{static_cast<const float*>(dh), idx_ffn, d};
  BRows<float> B{static_cast<const float*>(w_down_t), nullptr, INT_MAX, d};
  return run_f32<false>(A, B, EpiStore<float>{static_cast<float*>(e), d_ff}, counts, n_max, d_ff, d, s);
}

hipError_t launch_ffn_bwd_gateup(int dtype, const void* u, const int* idx_ffn, const int* counts, int n_max,
                                 const void* w_gate, const void* w_up, const void* e, const float* gate,
                                 void* dgu, float* dgpart, int d, int d_ff, bool exact, hipStream_t s) {
  if (n_max <= 0) return hipSuccess;
  if (dtype == 1) {
    ARows<bf16_t> A{static_cast<const bf16_t*>(u), idx_ffn, d};
    BRows<bf16_t> B{static_cast<const bf16_t*>(w_gate), static_cast<const bf16_t*>(w_up), INT_MAX, d};
    EpiSwiGLUBwd<bf16_t> epi{static_cast<const bf16_t*>(e), d_ff, idx_ffn, gate, static_cast<bf16_t*>(dgu),
                             2 * d_ff, d_ff, dgpart, swiglu_bwd_parts(1, d_ff)};
    return run_phase<true>(A, B, epi, counts, n_max, d_ff, d, s, exact);
  }
  ARows<float> A{static_cast<const float*>(u), idx_ffn, d};
  BRows<float> B{static_cast<const float*>(w_gate), static_cast<const float*>(w_up), INT_MAX, d};
  EpiSwiGLUBwd<float> epi{static_cast<const float*>(e), d_ff, idx_ffn, gate, static_cast<float*>(dgu),
                          2 * d_ff, d_ff, dgpart, d_ff};
  return run_f32<true>(A, B, epi, counts, n_max, d_ff, d, s);
}

hipError_t launch_ffn_bwd_du(int dtype, const void* dgu, const int* counts, int n_max, const void* w_gate_up_t,
                             float* du, int d, int d_ff, bool exact, hipStream_t s) {
  if (n_max <= 0) return hipSuccess;
  const int K = 2 * d_ff;
  if (dtype == 1) {
    ARows<bf16_t> A{static_cast<const bf16_t*>(dgu), nullptr, K};
    BRows<bf16_t> B{static_cast<const bf16_t*>(w_gate_up_t), nullptr, INT_MAX, K};
    return run_phase<false>(A, B, EpiStoreF32{du, d, 0}, counts, n_max, d, K, s, exact);
  }
  ARows<float> A{static_cast<const float*>(dgu), nullptr, K};
  BRows<float> B{static_cast<const float*>(w_gate_up_t), nullptr, INT_MAX, K};
  return run_f32<false>(A, B, EpiStoreF32{du, d, 0}, counts, n_max, d, K, s);
}

int adapter_proj_splits(int dtype, int d, int d_r) {
  if (dtype != 1) return 1;
  return adapter_wide(d_r) ? WIDE_SPLIT : adapter_groups(d);
}

hipError_t launch_adapter_proj2(int dtype, const void* rows0, const void* w0, float* part0, const void* rows1,
                                const void* w1, float* part1, const int* idx_ad, const int* counts, int n_max, int d,
                                int d_r, hipStream_t s) {
  if (n_max <= 0) return hipSuccess;
  if (dtype == 1 && !adapter_wide(d_r))
    return adapter_down_small(static_cast<const bf16_t*>(rows0), idx_ad, counts, n_max, static_cast<const bf16_t*>(w0),
                              part0, d, d_r, s, static_cast<const bf16_t*>(rows1), static_cast<const bf16_t*>(w1),
                              part1, adapter_groups(d));
  hipError_t e = launch_adapter_proj(dtype, rows0, idx_ad, counts, n_max, w0, part0, d, d_r, s);
  if (e != hipSuccess) return e;
  return launch_adapter_proj(dtype, rows1, idx_ad, counts, n_max, w1, part1, d, d_r, s);
}

hipError_t launch_adapter_proj(int dtype, const void* rows, const int* idx_ad, const int* counts, int n_max,
                               const void* w, float* part, int d, int d_r, hipStream_t s) {
  if (n_max <= 0) return hipSuccess;
  if (dtype == 1 && adapter_wide(d_r)) {
    // the K-sliced partials only (the forward's SiLU hidden rows are not needed here)
    ARows<bf16_t> A{static_cast<const bf16_t*>(rows), idx_ad, d};
    BRows<bf16_t> B{static_cast<const bf16_t*>(w), nullptr, INT_MAX, d};
    const size_t stride = static_cast<size_t>(n_max) * d_r;
    return run_tile<TileWide>(A, B, EpiStoreF32{part, d_r, stride}, counts, n_max, d_r, d, s, WIDE_SPLIT);
  }
  // the backward's consumers sum adapter_proj_splits() = adapter_groups(d) slices
  if (dtype == 1)
    return adapter_down_small(static_cast<const bf16_t*>(rows), idx_ad, counts, n_max, static_cast<const bf16_t*>(w),
                              part, d, d_r, s, nullptr, nullptr, nullptr, adapter_groups(d));
  ARows<float> A{static_cast<const float*>(rows), idx_ad, d};
  BRows<float> B{static_cast<const float*>(w), nullptr, INT_MAX, d};
  return run_f32<false>(A, B, EpiStoreF32{part, d_r, 0}, counts, n_max, d_r, d, s);
}

hipError_t launch_adapter_du(int dtype, const void* dz, const int* counts, int n_max, const void* w1t, float* du,
                             int d, int k, hipStream_t s) {
  if (n_max <= 0) return hipSuccess;
  if (dtype == 1) {
    ARows<bf16_t> A{static_cast<const bf16_t*>(dz), nullptr, k};
    BRows<bf16_t> B{static_cast<const bf16_t*>(w1t), nullptr, INT_MAX, k};
    return run_tile<TileWide>(A, B, EpiStoreF32{du, d, 0}, counts, n_max, d, k, s);
  }
  ARows<float> A{static_cast<const float*>(dz), nullptr, k};
  BRows<float> B{static_cast<const float*>(w1t), nullptr, INT_MAX, k};
  return run_f32<false>(A, B, EpiStoreF32{du, d, 0}, counts, n_max, d, k, s);
}

namespace {
struct EpiAccF32 {  // C[m][n] += acc
  float* out;
  int ld;
  __device__ __forceinline__ void store(int m, int n, float v) const { out[static_cast<size_t>(m) * ld + n] += v; }
};
}  // namespace

// The router's backward, its two large products.  dP enters as two bf16 terms, hi + lo, in one
// product each, so that the fp32 result is touched once.
namespace {
struct EpiStoreF32Two : EpiStoreF32 {
  static constexpr bool kTwoTerm = true;
};

// dhbar[t][n] += acc + the row's RMSNorm and transition terms, c_norm hbar + ddelta with
// ddelta = c1 delta_j + c2 delta_{j-1} (rowcoef), so that this is the only pass over dhbar
struct EpiRouterDh {
  static constexpr bool kTwoTerm = true;
  float* out;
  int ld;
  const float* coef;                   // [T][8]
  const bf16_t *h0, *h1, *h2;          // hbar_j, hbar_{j-1} (or null), hbar_{j-2} (or null)
  struct Pre {
    f32x4 o[2];
    u32x4 x, y, z;
    f32x4 c;
  };
  __device__ __forceinline__ Pre prep(int m, int n) const {
    Pre p;
    const size_t e = static_cast<size_t>(m) * ld + n;
    p.o[0] = *reinterpret_cast<const f32x4*>(out + e);
    p.o[1] = *reinterpret_cast<const f32x4*>(out + e + 4);
    p.c = *reinterpret_cast<const f32x4*>(coef + 8 * static_cast<size_t>(m));
    p.x = *reinterpret_cast<const u32x4*>(h0 + e);
    p.y = h1 ? *reinterpret_cast<const u32x4*>(h1 + e) : p.x;
    p.z = h2 ? *reinterpret_cast<const u32x4*>(h2 + e) : p.y;
    return p;
  }
  __device__ __forceinline__ void emit8(const Pre& p, int m, int n, const float* v) const {
    float r[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const auto at = [k](const u32x4& w) {
        return __uint_as_float(k & 1 ? w[k >> 1] & 0xffff0000u : w[k >> 1] << 16);
      };
      const float x = at(p.x), y = at(p.y), z = at(p.z);
      r[k] = p.o[k >> 2][k & 3] + v[k] + (p.c[0] * x + (p.c[1] * (x - y) + p.c[2] * (y - z)));
    }
    float* o = out + static_cast<size_t>(m) * ld + n;
    *reinterpret_cast<f32x4*>(o) = *reinterpret_cast<const f32x4*>(r);
    *reinterpret_cast<f32x4*>(o + 4) = *reinterpret_cast<const f32x4*>(r + 4);
  }
};

// C0 rows [0, m0), then C1: C[m][n] += sum over z < S of part[z][m][n], four columns a thread
__global__ __launch_bounds__(256) void acc_slices_kernel(const float* __restrict__ part, int S, int M, int N, int m0,
                                                        float* __restrict__ C0, float* __restrict__ C1) {
  const size_t e = (static_cast<size_t>(blockIdx.x) * 256 + threadIdx.x) * 4, n = static_cast<size_t>(M) * N;
  if (e >= n) return;
  f32x4 v = *reinterpret_cast<const f32x4*>(part + e);
  for (int z = 1; z < S; ++z) v += *reinterpret_cast<const f32x4*>(part + z * n + e);
  const size_t split = static_cast<size_t>(m0) * N;
  f32x4* c = reinterpret_cast<f32x4*>(e < split ? C0 + e : C1 + (e - split));
  *c += v;
}
}  // namespace

int router_bwd_dw_slices(int NP, int d, int kp) {
  const int tiles = (NP + 127) / 128 * (d / 256);
  return std::max(1, std::min({8, kCUs / std::max(tiles, 1), kp / BK}));
}

hipError_t launch_router_bwd_dw(const void* hi, const void* lo, int kp, int d_e, int NP, const void* hT, int d,
                                float* part, float* w_hd, float* ps1, hipStream_t s) {
  ARows<bf16_t> A{static_cast<const bf16_t*>(hi), nullptr, kp, static_cast<const bf16_t*>(lo), kp / BK};
  BRows<bf16_t> B{static_cast<const bf16_t*>(hT), nullptr, INT_MAX, kp};
  const int S = router_bwd_dw_slices(NP, d, kp);
  EpiStoreF32Two epi{{part, d, static_cast<size_t>(NP) * d}};
  const hipError_t e = run_phase_split(A, B, epi, nullptr, NP, d, 2 * kp, S, s);
  if (e != hipSuccess) return e;
  const size_t n4 = static_cast<size_t>(NP) * d / 4;
  acc_slices_kernel<<<static_cast<unsigned>((n4 + 255) / 256), 256, 0, s>>>(part, S, NP, d, d_e, w_hd, ps1);
  return hipGetLastError();
}

hipError_t launch_router_bwd_dh(const void* hi, const void* lo, int T, int NP, const void* wT, int d,
                                const float* coef, const void* hbar, const void* prev1, const void* prev2,
                                float* dhbar, hipStream_t s) {
  ARows<bf16_t> A{static_cast<const bf16_t*>(hi), nullptr, NP, static_cast<const bf16_t*>(lo), NP / BK};
  BRows<bf16_t> B{static_cast<const bf16_t*>(wT), nullptr, INT_MAX, NP};
  EpiRouterDh epi{dhbar, d, coef, static_cast<const bf16_t*>(hbar), static_cast<const bf16_t*>(prev1),
                  static_cast<const bf16_t*>(prev2)};
  return run_phase<false>(A, B, epi, nullptr, T, d, 2 * NP, s);
}

hipError_t launch_gemm_acc_f32(const float* A, int lda, int M, const float* B, int ldb, int N, int K, float* C,
                               int ldc, hipStream_t s) {
  ARows<float> a{A, nullptr, lda};
  BRows<float> b{B, nullptr, INT_MAX, ldb};
  return run_f32<false>(a, b, EpiAccF32{C, ldc}, nullptr, M, N, K, s);
}

hipError_t launch_gemm_nt_f32(const void* A, int M, const void* B, int N, int K, float* C, int ldc, hipStream_t s) {
  if (M <= 0 || N <= 0 || K <= 0) return hipSuccess;
  ARows<bf16_t> a{static_cast<const bf16_t*>(A), nullptr, K};
  BRows<bf16_t> b{static_cast<const bf16_t*>(B), nullptr, INT_MAX, K};
  return run_tile<TileWide>(a, b, EpiStoreF32{C, ldc, 0}, nullptr, M, N, K, s);
}

}  // namespace hero
