// Grouped expert GEMMs over the [E][C][*] dispatch layout.
//
// One launch covers every expert.  Two raggedness modes:
//   ragged-M (forward and dX products): expert e owns buffer rows
//     [rb_e, re_e); C(m, n) = sum_k A(rb_e + m, k) B(k, n) with A row-major
//     (K contiguous).  Tiles past the expert's row count exit at once, so no
//     host read-back of the counts is needed.
//   ragged-K (dW products): C_e = A_e^T B_e reduced over the expert's rows
//     [rb_e, re_e); both operands are row-major in the token dimension, i.e.
//     MN contiguous.  An expert with no rows stores exact zeros.
//
// bf16 path: a persistent kernel with v_mfma_f32_16x16x32_bf16 and float
// accumulation; operand tiles stream global -> LDS asynchronously through a
// multi-stage ring (details below).  Epilogues: plain store, (H, act(H))
// store, dA * act'(H) for the backward, a residual add, and float partials of
// a K-split dense weight gradient.
// The same kernel serves dense products (one group, no row ranges): the
// block's projections and, with row-major operands split into token ranges,
// their weight gradients.
// f32 path: a plain LDS-tiled FMA GEMM with the same addressing.
#include "internal.h"
#include "gemm_wide.h"

#include <cmath>
#include <utility>
#include <vector>

namespace lmoe {

template <typename OutT> __device__ __forceinline__ void store_out(OutT* p, float v);
template <> __device__ __forceinline__ void store_out<uint16_t>(uint16_t* p, float v) { *p = (uint16_t)f32_to_bf16_bits(v); }
template <> __device__ __forceinline__ void store_out<float>(float* p, float v) { *p = v; }
template <typename OutT> __device__ __forceinline__ float load_out(const OutT* p);
template <> __device__ __forceinline__ float load_out<uint16_t>(const uint16_t* p) { return bf16_bits_to_f32(*p); }
template <> __device__ __forceinline__ float load_out<float>(const float* p) { return *p; }

template <int EPI, typename OutT>
__device__ __forceinline__ void epilogue_store(const GemmParams& p, int64_t off, float v) {
  OutT* C = (OutT*)p.C;
  if constexpr (EPI == EPI_FWD1) {
    store_out<OutT>(C + off, v);
    store_out<OutT>((OutT*)p.C2 + off, act_fwd(v, p.act));
  } else if constexpr (EPI == EPI_DACT) {
    const float h = load_out<OutT>((const OutT*)p.Aux + off);
    store_out<OutT>(C + off, v * act_bwd(h, p.act));
  } else {
    store_out<OutT>(C + off, v);
  }
}

// ------------------------------------------------------------------ f32 path
template <bool B_K, bool RAGGED_K, int EPI>
__global__ __launch_bounds__(256) void gemm_f32_kernel(GemmParams p) {
  constexpr int BM = 64, BN = 64, BK = 16;
  __shared__ float As[BK][BM + 4];
  __shared__ float Bs[BK][BN + 4];
  const int tid = threadIdx.x;
  const int tx = tid % 16, ty = tid / 16;
  const int g = blockIdx.z;
  const int m0 = blockIdx.y * BM, n0 = blockIdx.x * BN;
  int lo, span;
  group_rows(p, g, lo, span);
  int Mlim, Klim;
  if constexpr (RAGGED_K) {
    Mlim = p.M;
    Klim = span;
  } else {
    Mlim = span;
    Klim = p.K;
    if (m0 >= Mlim) return;
  }
  const float* Ab = (const float*)p.A + g * p.sA + (int64_t)lo * p.lda;
  const float* Bb = (const float*)p.B + g * p.sB + (RAGGED_K ? (int64_t)lo * p.ldb : 0);
  float acc[4][4] = {};
  for (int k0 = 0; k0 < Klim; k0 += BK) {
    for (int i = tid; i < BM * BK; i += 256) {
      int m, k;
      float a = 0.f;
      if constexpr (RAGGED_K) {
        k = i / BM; m = i % BM;
        if (m0 + m < Mlim && k0 + k < Klim) a = Ab[(int64_t)(k0 + k) * p.lda + m0 + m];
      } else {
        m = i / BK; k = i % BK;
        if (m0 + m < Mlim && k0 + k < Klim) a = Ab[(int64_t)(m0 + m) * p.lda + k0 + k];
      }
      As[k][m] = a;
    }
    for (int i = tid; i < BN * BK; i += 256) {
      int n, k;
      float b = 0.f;
      if constexpr (B_K && !RAGGED_K) {
        n = i / BK; k = i % BK;
        if (n0 + n < p.N && k0 + k < Klim) b = Bb[(int64_t)(n0 + n) * p.ldb + k0 + k];
      } else {
        k = i / BN; n = i % BN;
        if (n0 + n < p.N && k0 + k < Klim) b = Bb[(int64_t)(k0 + k) * p.ldb + n0 + n];
      }
      Bs[k][n] = b;
    }
    __syncthreads();
#pragma unroll
    for (int kk = 0; kk < BK; ++kk) {
      float a[4], b[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) a[i] = As[kk][ty * 4 + i];
#pragma unroll
      for (int j = 0; j < 4; ++j) b[j] = Bs[kk][tx * 4 + j];
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = fmaf(a[i], b[j], acc[i][j]);
    }
    __syncthreads();
  }
  const int64_t cbase = (int64_t)g * p.sC + (RAGGED_K ? 0 : (int64_t)lo * p.ldc);
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int row = m0 + ty * 4 + i;
    if (row >= Mlim) continue;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int col = n0 + tx * 4 + j;
      if (col < p.N) epilogue_store<EPI, float>(p, cbase + (int64_t)row * p.ldc + col, acc[i][j]);
    }
  }
}

// --------------------------------------------------------------- launchers

// Workspace of the ragged-M bf16 expert products: a partial float tile per
// block, for a K-split last round.
size_t expert_sk_ws_bytes(const moe_cfg& c) { return c.dtype == MOE_BF16 ? (size_t)kSkPartElems * sizeof(float) : 0; }

// Tile choice of the wide kernel's ragged-M products.  A product's blocks
// advance in rounds of `slots` tiles.  A tile takes K / 32 steps of `full` ns
// when the round fills the chip, `part` ns when at most one block is on a CU,
// and `store` ns for its epilogue (two outputs, or an output and H).  The
// larger tile moves fewer bytes per flop (its step is the cheapest per output
// element); the smaller one wastes less on ragged rows and on rounds that leave
// CUs idle.  The constants are measured (whole products on one MI355X divided
// by their steps); the shape with the least modelled time runs.  Where the line
// lies, 256-tiles against the choice: expert_out of 1531 tokens (d 768, f 3072,
// 8 experts) 68 -> 26 us, of 48 tokens (d 1024, f 4096, 16 experts) 75 -> 44,
// of 2048 tokens (d 768) 73 -> 40, of 3108 tokens 78 -> 65; at 4096 tokens
// (d 1024, 16 experts) 110 stays against 128 with 128-tiles, and the fused
// products keep 256-tiles from 2048 tokens on (37 against 41).
struct TileCost {
  int bm, bn, slots;
  double full, part, store;
  void (*run)(const WideCall&, hipStream_t);
};
static const TileCost kTilesM[] = {{256, 256, 256, 650., 650., 8000., run_wide_256x256},
                                   {128, 128, 512, 520., 330., 4500., run_wide_128x128},
                                   {64, 128, 512, 390., 230., 3000., run_wide_64x128},
                                   {64, 64, 512, 300., 190., 2000., run_wide_64x64}};
static double tile_cost(const TileCost& t, const WideCall& w) {
  // M-tiles of a group: the mean over one standard deviation of routed rows.
  const double tm = 0.5 * (std::ceil(std::max(1., w.expect - w.spread) / t.bm) + std::ceil((w.expect + w.spread) / t.bm));
  const double tiles = std::ceil(w.groups * tm * std::ceil((double)w.cols / t.bn));
  const double rounds = std::floor(tiles / t.slots), rem = tiles - rounds * t.slots;
  const double steps = w.p.K / 32., store = w.kind == WK_FWD1 || w.kind == WK_DACT ? t.store : t.store / 2;
  return rounds * (steps * t.full + store) + (rem <= 0 ? 0. : steps * (rem <= 256 ? t.part : t.full) + store);
}
static void run_wide_any(const WideCall& w, hipStream_t s) {
  if (w.rows <= 0 || w.cols <= 0 || w.groups <= 0) return;
  if (w.kind >= WK_DW) {
    // Ragged-K: 128-tiles where 256-tiles would not make two rounds (dW of 2048
    // tokens, d 768, 8 experts, 288 large tiles: 43 -> 32 us; of 20000 tokens,
    // d 512, 128 large tiles: 82 -> 57); with more the larger tile wins (8192
    // tokens, d 1024, 16 experts, 1024 large tiles: 142 against 166).
    const int64_t large = (w.rows + 255) / 256 * ((w.cols + 255) / 256) * w.groups;
    return large <= 512 ? run_wide_128x128(w, s) : run_wide_256x256(w, s);
  }
  const TileCost* best = &kTilesM[0];
  for (const TileCost& t : kTilesM)
    if (tile_cost(t, w) < tile_cost(*best, w)) best = &t;
  best->run(w, s);
}

// Expert products.  bf16: blocked operands, wide tiles; outputs that a later
// product reads (H, A, dH) blocked, the others (expert_out, dXe, which only
// the gathers read, and the dW products) row-major.  float: the FMA kernel,
// row-major.
// rows: rows of the output per group (ragged-M: the capacity C, with up to 15
// alignment rows; ragged-K: M); cols: N.
template <bool B_K, bool RAGGED_K, int EPI>
static void run_expert(const moe_cfg& c, WideKind kind, const GemmParams& p, int64_t rows, int cols, hipStream_t s) {
  if (rows <= 0 || cols <= 0 || c.E <= 0) return;
  if (c.dtype != MOE_BF16) {
    dim3 grid((unsigned)((cols + 63) / 64), (unsigned)((rows + 63) / 64), (unsigned)c.E);
    hipLaunchKernelGGL((gemm_f32_kernel<B_K, RAGGED_K, EPI>), grid, dim3(256), 0, s, p);
    return;
  }
  // Rows a group is expected to hold: the call's assignments spread evenly (T is
  // only a hint here: rows may come from elsewhere).
  const double expect = c.T > 0 ? std::min<double>(c.C, (double)c.T * c.k / c.E) : c.C;
  run_wide_any(WideCall{kind, c.act, c.E, rows, cols, expect, std::sqrt(expect * (1. - (double)c.k / c.E)), p}, s);
}

// Rows per expert block of an [E][C][*] buffer (C rounded up to 16 for bf16).
static int64_t rows_alloc(const moe_cfg& c) { return c.dtype == MOE_BF16 ? pad16(c.C) : c.C; }

// Per-product timing (moe_product_timing): while on, each expert product
// launch of this thread is bracketed by a pair of events on its stream (the
// K-split fix-up launch inside the pair); product_times sums them per product.
namespace {
struct ProductTimer {
  bool on = false;
  int dev = -1;
  bool failed = false;
  std::vector<hipEvent_t> pool;      // events of this device, reused after each readout
  size_t next = 0;
  std::vector<std::pair<int, size_t>> rec;   // (product, index of its first event)
};
thread_local ProductTimer g_ptimer;

hipEvent_t ptimer_event() {
  ProductTimer& t = g_ptimer;
  if (t.next == t.pool.size()) {
    hipEvent_t e = nullptr;
    if (hipEventCreate(&e) != hipSuccess) {
      t.failed = true;
      return nullptr;
    }
    t.pool.push_back(e);
  }
  return t.pool[t.next++];
}
// Records the opening event of product `prod` on s; returns false when timing is off.
bool ptimer_begin(int prod, hipStream_t s) {
  ProductTimer& t = g_ptimer;
  if (!t.on) return false;
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev != t.dev) {   // events belong to the device timing was started on
    t.failed = true;
    return false;
  }
  const size_t i = t.next;
  hipEvent_t a = ptimer_event(), b = ptimer_event();
  if (!a || !b || hipEventRecord(a, s) != hipSuccess) {
    t.failed = true;
    return false;
  }
  t.rec.push_back({prod, i});
  return true;
}
void ptimer_end(bool begun, hipStream_t s) {
  if (!begun) return;
  ProductTimer& t = g_ptimer;
  if (hipEventRecord(t.pool[t.rec.back().second + 1], s) != hipSuccess) t.failed = true;
}
}  // namespace

hipError_t product_timing(bool on) {
  ProductTimer& t = g_ptimer;
  int dev = 0;
  const hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev != t.dev) {   // a different device: the pool's events belong to the old one (left, not destroyed)
    t.pool.clear();
    t.dev = dev;
  }
  t.on = on;
  t.failed = false;
  t.next = 0;
  t.rec.clear();
  return hipSuccess;
}

hipError_t product_times(double* ms, int32_t* counts) {
  ProductTimer& t = g_ptimer;
  for (int q = 0; q < kProducts; ++q) {
    ms[q] = 0.0;
    counts[q] = 0;
  }
  if (t.failed) return hipErrorUnknown;
  for (const auto& r : t.rec) {
    hipError_t e = hipEventSynchronize(t.pool[r.second + 1]);
    float v = 0.f;
    if (e == hipSuccess) e = hipEventElapsedTime(&v, t.pool[r.second], t.pool[r.second + 1]);
    if (e != hipSuccess) return e;
    ms[r.first] += v;
    counts[r.first] += 1;
  }
  t.next = 0;
  t.rec.clear();
  return hipSuccess;
}

void launch_expert_fwd(const moe_cfg& c, const void* X, const int32_t* rb, const int32_t* re, const void* W1,
                       const void* W2, void* H, void* A, void* O, void* ws, hipStream_t s) {
  const int64_t d = c.d_model, f = c.d_ff, C = c.C, Cp = rows_alloc(c);
  GemmParams p1{X, d, Cp * d, W1, d, f * d, H, f, Cp * f, A, nullptr, rb, re, 0, (int)f, (int)d, c.act, (int)C};
  p1.part = (float*)ws;
  p1.ksplit = c.ksplit;
  bool tb = ptimer_begin(kProdFwd1, s);
  run_expert<true, false, EPI_FWD1>(c, WK_FWD1, p1, C, (int)f, s);
  ptimer_end(tb, s);
  GemmParams p2{A, f, Cp * f, W2, f, d * f, O, d, Cp * d, nullptr, nullptr, rb, re, 0, (int)d, (int)f, c.act, (int)C};
  p2.part = (float*)ws;
  p2.ksplit = c.ksplit;
  tb = ptimer_begin(kProdFwd2, s);
  run_expert<true, false, EPI_STORE>(c, WK_NK, p2, C, (int)d, s);   // expert_out row-major
  ptimer_end(tb, s);
}

void launch_expert_bwd_dx(const moe_cfg& c, const void* dO, const int32_t* rb, const int32_t* re, const void* H,
                          const void* W1, const void* W2, void* dH, void* dXe, void* ws, hipStream_t s) {
  const int64_t d = c.d_model, f = c.d_ff, C = c.C, Cp = rows_alloc(c);
  // dA = dO W2_e  (B(k=i, n=j) = W2[e][i][j], N contiguous), epilogue dH = dA * act'(H)
  GemmParams p1{dO, d, Cp * d, W2, f, d * f, dH, f, Cp * f, nullptr, H, rb, re, 0, (int)f, (int)d, c.act, (int)C};
  p1.part = (float*)ws;
  p1.ksplit = c.ksplit;
  bool tb = ptimer_begin(kProdDA, s);
  run_expert<false, false, EPI_DACT>(c, WK_DACT, p1, C, (int)f, s);
  ptimer_end(tb, s);
  // dXe = dH W1_e  (B(k=i, n=j) = W1[e][i][j])
  GemmParams p2{dH, f, Cp * f, W1, d, f * d, dXe, d, Cp * d, nullptr, nullptr, rb, re, 0, (int)d, (int)f, c.act, (int)C};
  p2.part = (float*)ws;
  p2.ksplit = c.ksplit;
  tb = ptimer_begin(kProdDXe, s);
  run_expert<false, false, EPI_STORE>(c, WK_KN, p2, C, (int)d, s);   // dXe row-major
  ptimer_end(tb, s);
}

void launch_expert_bwd_dw(const moe_cfg& c, const void* X, const void* A, const void* dO, const void* dH,
                          const int32_t* rb, const int32_t* re, void* dW1, void* dW2, hipStream_t s) {
  const int64_t d = c.d_model, f = c.d_ff, C = c.C, Cp = rows_alloc(c);
  // dW2_e [d][f] = dO_e^T A_e : A-operand(m, k) = dO[e][k][m], B(k, n) = A[e][k][n]
  // (wpacked: written in the blocked layout of the packed weights)
  GemmParams p2{dO, d, Cp * d, A, f, Cp * f, dW2, f, d * f, nullptr, nullptr, rb, re, (int)d, (int)f, 0, c.act, (int)C};
  // dW1_e [f][d] = dH_e^T X_e
  GemmParams p1{dH, f, Cp * f, X, d, Cp * d, dW1, d, f * d, nullptr, nullptr, rb, re, (int)f, (int)d, 0, c.act, (int)C};
  const bool blk = c.wpacked && c.dtype == MOE_BF16;
  bool tb = ptimer_begin(kProdDW2, s);
  run_expert<false, true, EPI_STORE>(c, blk ? WK_DW_BLK : WK_DW, p2, d, (int)f, s);
  ptimer_end(tb, s);
  tb = ptimer_begin(kProdDW1, s);
  run_expert<false, true, EPI_STORE>(c, blk ? WK_DW_BLK : WK_DW, p1, f, (int)d, s);
  ptimer_end(tb, s);
}

// Sum of the S float partials of a K-split weight gradient, in group order,
// rounded once to bf16: 8 consecutive elements per thread.
__global__ __launch_bounds__(256) void gemm_wgrad_reduce_kernel(const float* __restrict__ part, int S, int64_t MN,
                                                                 uint16_t* __restrict__ C) {
  const int64_t i = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) * 8;
  if (i >= MN) return;
  f32x4 a0 = *reinterpret_cast<const f32x4*>(part + i), a1 = *reinterpret_cast<const f32x4*>(part + i + 4);
  for (int g = 1; g < S; ++g) {
    a0 += *reinterpret_cast<const f32x4*>(part + (int64_t)g * MN + i);
    a1 += *reinterpret_cast<const f32x4*>(part + (int64_t)g * MN + i + 4);
  }
  const float v0[4] = {a0[0], a0[1], a0[2], a0[3]}, v1[4] = {a1[0], a1[1], a1[2], a1[3]};
  const u32x2 lo = pack4_bf16(v0), hi = pack4_bf16(v1);
  *reinterpret_cast<u32x4*>(C + i) = u32x4{lo[0], lo[1], hi[0], hi[1]};
}

// Token ranges of the dense weight gradients: the block's 2048 x 2048 and
// 6144 x 2048 products have 64 and 192 tiles of 256 x 256, so four ranges give
// every CU work (256 and 768 tile-ranges).
constexpr int kWgradSplit = 4;
size_t wgrad_ws_bytes(int M, int N) { return (size_t)kWgradSplit * M * N * sizeof(float); }

// Weight gradient C[M][N] = A^T B of the block's dense projections, A [K][M]
// and B [K][N] row-major bf16 (K = tokens), C bf16: the wide kernel's ragged-K
// product with K split into wgrad_ksplit(M, N) token ranges of equal length
// (multiples of 32), one float partial per range in `part`
// (wgrad_ws_bytes(M, N) bytes), then their sum in range order.
void launch_dense_wgrad(int M, int N, int64_t K, const void* A, const void* B, void* C, void* part, hipStream_t s) {
  if (M <= 0 || N <= 0) return;
  const int S = kWgradSplit;
  const int64_t MN = (int64_t)M * N;
  GemmParams p{A, M, 0, B, N, 0, part, N, MN, nullptr, nullptr, nullptr, nullptr, M, N, 0, 0, (int)K};
  p.kchunk = (int)(((K + S - 1) / S + 31) / 32 * 32);
  run_wide_any(WideCall{WK_WGF32, MOE_ACT_IDENTITY, S, M, N, 0., 0., p}, s);
  hipLaunchKernelGGL(gemm_wgrad_reduce_kernel, dim3((unsigned)((MN / 8 + 255) / 256)), dim3(256), 0, s,
                     (const float*)part, S, MN, (uint16_t*)C);
}

// Row-major [M][K] bf16 -> the blocked layout with pad16(M) rows (rows past M
// zero).  One wave per 16 x 32 block: each lane reads 16 bytes of one row and
// the wave writes the block's 1 KiB as one contiguous run.
__global__ __launch_bounds__(256) void pack_rows_kernel(const uint16_t* __restrict__ src, uint16_t* __restrict__ dst,
                                                        int64_t M, int K) {
  const int64_t b = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
  const int lane = threadIdx.x & 63;
  const int kb = K >> 5;
  const int64_t rb = b / kb;
  if (rb * 16 >= pad16(M)) return;
  const int cb = (int)(b - rb * kb);
  const int64_t row = rb * 16 + (lane >> 2);
  const int col = cb * 32 + (lane & 3) * 8;
  u32x4 v = u32x4{0u, 0u, 0u, 0u};
  if (row < M) v = *reinterpret_cast<const u32x4*>(src + row * K + col);
  *reinterpret_cast<u32x4*>(dst + b * 512 + lane * 8) = v;
}

void launch_pack_rows(const void* src, void* dst, int64_t M, int K, hipStream_t s) {
  if (M <= 0 || K <= 0) return;
  const int64_t blocks = pad16(M) / 16 * (K / 32);
  hipLaunchKernelGGL(pack_rows_kernel, dim3((unsigned)((blocks * 64 + 255) / 256)), dim3(256), 0, s,
                     (const uint16_t*)src, (uint16_t*)dst, M, K);
}

// Dense products on the wide MFMA kernel: one group of M rows, both operands
// blocked (A [pad16(M)][K]; B [N][K] if b_nk else [K][N]), output row-major,
// + resid (row-major like C) if given.  Every output element is one in-order
// K sum (no K-split), so a product over a batch partition's rows gives the
// same bits as over the whole batch.
void launch_dense_wide(int64_t M, int N, int K, const void* A, const void* B, bool b_nk, void* C, int64_t ldc,
                       const void* resid, hipStream_t s) {
  if (M <= 0 || N <= 0 || K <= 0) return;
  GemmParams p{A, K, pad16(M) * K, B, b_nk ? K : N, (int64_t)N * K, C, ldc, M * ldc, nullptr, resid, nullptr, nullptr,
               0, N, K, 0, (int)M};
  p.ksplit = 0;
  run_wide_any(WideCall{b_nk ? (resid ? WK_NK_RES : WK_NK) : WK_KN, MOE_ACT_IDENTITY, 1, M, N, (double)M, 0., p}, s);
}

}  // namespace lmoe
