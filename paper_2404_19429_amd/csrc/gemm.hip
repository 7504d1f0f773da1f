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
// f32 path: LDS-tiled float MFMAs with the same addressing.
#include "internal.h"
#include "gemm_wide.h"

#include <cmath>
#include <utility>
#include <vector>

namespace lmoe {

// ------------------------------------------------------------------ f32 path
// v_mfma_f32_16x16x4_f32 over LDS tiles, float in, float accumulation.  Bound:
// the matrix cores' float rate (157 TFLOP/s nominal); an MFMA takes 32 cycles
// for two 4-byte operands per lane, so plain loads (global -> registers -> LDS,
// one stage ahead) and LDS reads hide under it.  Training step of 2000 tokens
// (d 512, f 2048, 8 experts, one MI355X), against a 64 x 64 tile of vector
// multiply-adds: H 191 -> 113 us, expert_out 358 -> 125, each dW 146 -> 104 (81
// TFLOP/s); a 128-tile was slower on all but dW (its ragged rows and rounds).
//
// A block is 2 x 2 waves of WT x WT fragments of 16 x 16: a tile of 32 WT on a
// side, 64 / WT of K per stage (the same 16 KB of LDS and four 16-byte loads
// per thread and stage for either WT).  The MFMA adds its four products to the
// accumulator one fused multiply-add at a time in K order (measured: the same
// bits as a loop of fmaf), and every element takes its K in ascending order, so
// results do not depend on WT and are those of the plain sum.
// The product is computed transposed: a lane ends with four consecutive output
// columns of one row.
template <int WT, bool KC>
struct F32Tile {
  static constexpr int ROWS = 32 * WT, BK = 64 / WT;   // rows or columns of the operand; K per stage
  static constexpr int LD = KC ? BK + 4 : ROWS + 16;   // padded LDS row: a wave's reads spread over the banks
  static constexpr int ELEMS = (KC ? ROWS : BK) * LD;
  static constexpr int NLD = ROWS * BK / 4 / 256;      // 16-byte loads per thread and stage
  static constexpr int W = KC ? BK / 4 : ROWS / 4;     // chunks per LDS row
  const float* rp[NLD];                                // the thread's row (KC) or column of chunk i, at K = 0
  // KC: [ROWS][K] from row r0 < rlim; else [K][ROWS] from column r0.  Rows or
  // columns past the limit repeat the last (their outputs are not stored).
  __device__ void plan(const float* base, int64_t ld, int r0, int rlim) {
#pragma unroll
    for (int i = 0; i < NLD; ++i) {
      const int c = threadIdx.x + 256 * i;
      if constexpr (KC) rp[i] = base + min(r0 + c / W, rlim - 1) * ld;
      else rp[i] = base + min(r0 + 4 * (c % W), rlim - 4);
    }
  }
  __device__ static int kofs(int i) { return KC ? 4 * ((threadIdx.x + 256 * i) % W) : (threadIdx.x + 256 * i) / W; }
  // The stage at k0, from addresses clamped into K (klim > 0): without a branch
  // every load of the stage is in flight together.
  __device__ void load(f32x4 (&v)[NLD], int64_t ld, int k0, int klim) const {
#pragma unroll
    for (int i = 0; i < NLD; ++i) {
      const int k = min(k0 + kofs(i), klim - (KC ? 4 : 1));
      v[i] = *reinterpret_cast<const f32x4*>(rp[i] + (KC ? k : k * ld));
    }
  }
  // To LDS, K at and past klim as zeros.  KC: within 16 of K, k = 4 s + q goes
  // to place 4 q + s, so that a lane's elements of four MFMAs are one 16-byte read.
  __device__ static void store(const f32x4 (&v)[NLD], float* st, int k0, int klim) {
#pragma unroll
    for (int i = 0; i < NLD; ++i) {
      const int c = threadIdx.x + 256 * i;
      const f32x4 x = k0 + kofs(i) < klim ? v[i] : f32x4{0.f, 0.f, 0.f, 0.f};
      if constexpr (KC) {
        float* o = st + c / W * LD + (c % W >> 2) * 16 + (c & 3);
#pragma unroll
        for (int q = 0; q < 4; ++q) o[4 * q] = x[q];
      } else {
        *reinterpret_cast<f32x4*>(st + c / W * LD + 4 * (c % W)) = x;
      }
    }
  }
  // The lane's elements of the four MFMAs of the stage's 16-K block kb (K 4 s + lane / 16
  // for MFMA s) for row or column r16 + lane % 16.
  __device__ static f32x4 frag(const float* st, int r16, int kb, int lane) {
    const int r = r16 + (lane & 15), q = lane >> 4;
    if constexpr (KC) {
      return *reinterpret_cast<const f32x4*>(st + r * LD + 16 * kb + 4 * q);
    } else {
      const float* o = st + (16 * kb + q) * LD + r;
      return f32x4{o[0], o[4 * LD], o[8 * LD], o[12 * LD]};
    }
  }
};

template <int EPI>
__device__ __forceinline__ void f32_store(const GemmParams& p, int64_t off, const f32x4& v) {
  f32x4 o = v;
  if constexpr (EPI == EPI_DACT) {
    const f32x4 h = *reinterpret_cast<const f32x4*>((const float*)p.Aux + off);
#pragma unroll
    for (int u = 0; u < 4; ++u) o[u] = v[u] * act_bwd(h[u], p.act);
  }
  *reinterpret_cast<f32x4*>((float*)p.C + off) = o;
  if constexpr (EPI == EPI_FWD1) {
#pragma unroll
    for (int u = 0; u < 4; ++u) o[u] = act_fwd(v[u], p.act);
    *reinterpret_cast<f32x4*>((float*)p.C2 + off) = o;
  }
}

// Ragged-M: the tiles of the rows that are there, n fastest, fall into eight
// contiguous ranges, one per XCD (block index modulo 8), so an XCD's L2 holds
// the operands its blocks share and every XCD has the same number of tiles.
// Ragged-K (tiles as long as their group): rows of tn tiles are dealt to the
// XCDs in turn, so a few large experts still spread over the chip.
template <int WT, bool B_K, bool RAGGED_K, int EPI>
__global__ __launch_bounds__(256) void gemm_f32_kernel(GemmParams p, int tm, int tn, int groups) {
  using TA = F32Tile<WT, !RAGGED_K>;
  using TB = F32Tile<WT, B_K && !RAGGED_K>;
  constexpr int BM = TA::ROWS, BK = TA::BK;
  __shared__ __attribute__((aligned(16))) float As[2][TA::ELEMS];
  __shared__ __attribute__((aligned(16))) float Bs[2][TB::ELEMS];
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  const int xcd = blockIdx.x % 8, local = blockIdx.x / 8;
  int g, m0, n0, lo, span;
  if constexpr (RAGGED_K) {
    const int tr = (local / tn) * 8 + xcd;
    if (tr >= groups * tm) return;
    g = tr / tm;
    m0 = (tr - g * tm) * BM;
    n0 = (local % tn) * BM;
    group_rows(p, g, lo, span);
  } else {
    const WPrefix P = wide_tile_prefix<BM, false, false>(p, lane, groups, tm, tn);
    const int per = (P.NF + 7) / 8, t = xcd * per + local;
    if (local >= per || t >= P.NF) return;
    g = __builtin_amdgcn_readfirstlane(__popcll(__ballot(lane < groups && P.incl <= t)));
    const int q = t - __builtin_amdgcn_readlane(P.excl, g);
    m0 = q / tn * BM;
    n0 = q % tn * BM;
    lo = __builtin_amdgcn_readlane(P.lo, g);
    span = __builtin_amdgcn_readlane(P.span, g);
  }
  const int Mlim = RAGGED_K ? p.M : span, Klim = RAGGED_K ? span : p.K;
  if (m0 >= Mlim) return;
  const float* Ab = (const float*)p.A + g * p.sA + (int64_t)lo * p.lda;
  const float* Bb = (const float*)p.B + g * p.sB + (RAGGED_K ? (int64_t)lo * p.ldb : 0);
  const int wm = (wid >> 1) * 16 * WT, wn = (wid & 1) * 16 * WT;
  f32x4 acc[WT][WT];
#pragma unroll
  for (int i = 0; i < WT; ++i)
#pragma unroll
    for (int j = 0; j < WT; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  f32x4 va[TA::NLD], vb[TB::NLD];
  TA ta;
  TB tb;
  ta.plan(Ab, p.lda, m0, Mlim);
  tb.plan(Bb, p.ldb, n0, p.N);
  if (Klim > 0) {
    ta.load(va, p.lda, 0, Klim);
    tb.load(vb, p.ldb, 0, Klim);
  }
  int buf = 0;
  for (int k0 = 0; k0 < Klim; k0 += BK, buf ^= 1) {
    TA::store(va, As[buf], k0, Klim);
    TB::store(vb, Bs[buf], k0, Klim);
    __syncthreads();   // this stage is in LDS; every wave is past the stage before (the other buffer)
    // The next stage's loads, in flight under this stage's MFMAs (past the last
    // stage: one that is not stored).  The opaque start keeps the compiler from
    // moving them to their use at the top of the loop.
    int kn = k0 + BK;
    asm volatile("" : "+s"(kn));
    ta.load(va, p.lda, kn, Klim);
    tb.load(vb, p.ldb, kn, Klim);
    __builtin_amdgcn_sched_barrier(0);
    constexpr int KB = BK / 16;
    f32x4 fa[KB][WT], fb[KB][WT];
#pragma unroll
    for (int kb = 0; kb < KB; ++kb) {
#pragma unroll
      for (int i = 0; i < WT; ++i) fa[kb][i] = TA::frag(As[buf], wm + 16 * i, kb, lane);
#pragma unroll
      for (int j = 0; j < WT; ++j) fb[kb][j] = TB::frag(Bs[buf], wn + 16 * j, kb, lane);
    }
    __builtin_amdgcn_sched_barrier(0);   // the stage's reads together, ahead of its MFMAs
#pragma unroll
    for (int kb = 0; kb < KB; ++kb)
#pragma unroll
      for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int i = 0; i < WT; ++i)
#pragma unroll
          for (int j = 0; j < WT; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(fb[kb][j][s], fa[kb][i][s], acc[i][j], 0, 0, 0);
  }
  const int64_t cbase = (int64_t)g * p.sC + (RAGGED_K ? 0 : (int64_t)lo * p.ldc);
#pragma unroll
  for (int i = 0; i < WT; ++i) {
    const int row = m0 + wm + 16 * i + (lane & 15);
    if (row >= Mlim) continue;
#pragma unroll
    for (int j = 0; j < WT; ++j) {
      const int col = n0 + wn + 16 * j + 4 * (lane >> 4);
      if (col < p.N)   // (N is a multiple of 8)
        f32_store<EPI>(p, cbase + (int64_t)row * p.ldc + col, acc[i][j]);
    }
  }
}

template <int WT, bool B_K, bool RAGGED_K, int EPI>
static void launch_f32(const GemmParams& p, int groups, int64_t rows, int cols, hipStream_t s) {
  // (ragged-M: with up to 15 alignment rows, as wide_tile_prefix counts them)
  const int tm = (int)((rows + (RAGGED_K ? 0 : 15) + 32 * WT - 1) / (32 * WT)), tn = (cols + 32 * WT - 1) / (32 * WT);
  const int64_t blocks = RAGGED_K ? ((int64_t)groups * tm + 7) / 8 * 8 * tn : ((int64_t)groups * tm * tn + 7) / 8 * 8;
  hipLaunchKernelGGL((gemm_f32_kernel<WT, B_K, RAGGED_K, EPI>), dim3((unsigned)blocks), dim3(256), 0, s, p, tm, tn,
                     groups);
}

// --------------------------------------------------------------- launchers

// Workspace of the ragged-M bf16 expert products: a partial float tile per
// block, for a K-split last round.
size_t expert_sk_ws_bytes(const moe_cfg& c) { return c.dtype == MOE_BF16 ? (size_t)kSkPartElems * sizeof(float) : 0; }

// Tile choice of the wide kernel's ragged-M products.  A product's blocks
// advance in rounds of per_cu tiles per CU.  A tile takes K / 32 steps of `full`
// ns when the round fills the chip, `part` ns when at most one block is on a CU,
// and `store` ns for its epilogue (two outputs, or an output and H).  The
// larger tile moves fewer bytes per flop (its step is the cheapest per output
// element); the smaller one wastes less on ragged rows and on rounds that leave
// CUs idle.  The constants are measured (whole products on one MI355X divided
// by their steps); the shape with the least modelled time runs.  The rows are
// taken as spread evenly over the groups: how a routing is skewed shows on the
// device only.
// Where the line lies, 256-tiles against the choice: expert_out of 1531 tokens (d
// 768, f 3072, 8 experts) 68 -> 26 us, of 48 tokens (d 1024, f 4096, 16 experts) 75 -> 44,
// of 2048 tokens (d 768) 73 -> 40, of 3108 tokens 78 -> 65; at 4096 tokens
// (d 1024, 16 experts) 128-tiles lose (128 against 110), and the fused products
// keep 256-tiles from 2048 tokens on (37 against 41).  192-row tiles, for rows
// that end just past a multiple of 256: expert_out of 4096 tokens (d 2048, 16
// experts, no K-split) 372 -> 328, of 6000 tokens (d 1536, 32 experts) 178 -> 145;
// of 16384 tokens (8 experts) 256-tiles stay, 948 against 971.
struct TileCost {
  int bm, bn, per_cu;   // per_cu: blocks of this shape on a CU, so a round is per_cu tiles per CU
  double full, part, store;
  void (*run)(const WideCall&, hipStream_t);
};
static const TileCost kTilesM[] = {{256, 256, 1, 650., 650., 8000., run_wide_256x256},
                                   {192, 256, 1, 560., 560., 7000., run_wide_192x256},
                                   {128, 128, 2, 520., 330., 4500., run_wide_128x128},
                                   {64, 128, 2, 390., 230., 3000., run_wide_64x128},
                                   {64, 64, 2, 300., 190., 2000., run_wide_64x64}};
static double tile_cost(const TileCost& t, const WideCall& w, int cus) {
  // M-tiles of a group: a mean over the routed rows' spread.
  const double tm = 0.25 * std::ceil(std::max(1., w.expect - w.spread) / t.bm) + 0.5 * std::ceil(w.expect / t.bm) +
                    0.25 * std::ceil((w.expect + w.spread) / t.bm);
  const double tiles = std::ceil(w.groups * tm * std::ceil((double)w.cols / t.bn));
  const double slots = (double)t.per_cu * cus;
  const double rounds = std::floor(tiles / slots), rem = tiles - rounds * slots;
  const double steps = w.p.K / 32., store = w.kind == WK_FWD1 || w.kind == WK_DACT ? t.store : t.store / 2;
  double last = rem <= 0 ? 0. : steps * (rem <= cus ? t.part : t.full) + store;
  // A K-split last round: its share of a round, and the partial tiles' write and sum.
  if (t.bm == 256 && w.p.ksplit && (w.kind == WK_NK || w.kind == WK_KN) && rounds > 0 && rem > 0 && 4 * rem <= slots)
    last = steps * t.full * rem / slots + 15000.;
  return rounds * (steps * t.full + store) + last;
}
// The tile of a ragged-M product (index into kTilesM).
static int tile_m(const WideCall& w, int cus) {
  int best = 0;
  for (int i = 1; i < (int)(sizeof kTilesM / sizeof kTilesM[0]); ++i)
    if (tile_cost(kTilesM[i], w, cus) < tile_cost(kTilesM[best], w, cus)) best = i;
  return best;
}
// The tile of a ragged-K product: 128 or 256 wide.  A tile is as long as its group
// and its blocks stay on the CUs, so whole rounds decide: 256-tiles one per CU,
// 128-tiles three.  Modelled, in ns per 32 rows of a group: a round of 256-tiles 720
// to half full, 900 full; of 128-tiles 440 where no CU has more than one, 620 two, 850
// three in several rounds and 1000 in a single one (780 with at most 128 operand
// slices of 128, which the L2s then share); 4000 and 2000 for a round's stores, 8000
// and 7000 once, 3000 for an idle launch.  Below 512 rows per group the choice is
// worth 2 us at most, and 128-tiles run.
//
// Measured on one MI355X, one product, 128- against 256-tiles: 128 large tiles of
// 2048 rows (d 512, f 2048, 8 experts) 46 and 57 us; 160 of 11506 rows (d 192, f 2560,
// 16 experts) 350 and 297; 192 (d 768) of 512 rows 25 and 27, of 4096 132 and 119, (d
// 2048, 3 experts) of 2048 55 and 60; 240 (d 640, f 1280, 16 experts) of 2048 122 and 81; 256 (d
// 1024) of 200 20 and 19, of 1024 50 and 41, of 8192 343 and 239; 288 (d 768, f 3072)
// of 512 34 and 38, of 8192 387 and 405; 384 of 512 39 and 40, of 8192 449 and 409;
// 512 of 1024 88 and 73.  Past two rounds of 256-tiles they win or tie at any length.
//
// Routed groups may be skewed, which shows on the device only; there the longest
// group's tiles are the time, and smaller ones share them between CUs (Zipf 1.2,
// capacity twice the mean of 4096 rows: 256 large tiles of 8 experts 152 and 191 us,
// of 64 experts 174 and 194; 512 large tiles 239 and 245, of 1024 rows 72 and 74; 64
// experts of d 832, f 512, 512 large tiles in part-filled columns, 182 and 218).  So up
// to one and a half rounds, and up to two where an idle launch (3 us) is little
// against the product, both shapes are launched and the row counts pick the one that
// runs.
// The dense weight gradients' groups are token ranges of one length (w.expect): where
// they are not short, 128-tiles take 3/4 of the time of a 256-tile round for the work
// of 192 large tiles.  dW of 256 large tiles and 8192 rows each, 128- against
// 256-tiles (two launches) 645 and 505 us, of 416 tiles and 1260 rows 191 and 170; of
// 512 tiles and 75 rows 45 and 50.
//
// Where other work runs beside the product (the block's weight stream), it fills the
// CUs that a part-filled round leaves idle, and the tile with the least CU time wins:
// 256-tiles from three quarters of a round on.  Block backward on three streams, the choice above
// against 256-tiles: 6 x 2501 tokens (d 1536, f 3072, 4 experts; 288 large tiles, dWo
// 144, dWqkv 432) 2561 and 2296 us, 8 x 2048 (d 1024, f 4096, 8 experts; 512, 64, 192)
// 1877 and 1762; with all products below a full round 128-tiles stay ahead (4 x 500
// tokens, d 512, f 2048, 8 experts; 128, 16, 48) 208 and 244.  (Nor is an idle launch
// little there: its blocks wait for CUs that the other work holds.)
enum TileK { kTileK128, kTileK256, kTileKByRows };
static TileK tile_k(const WideCall& w, int cus) {
  const auto tiles = [&](int t) { return (w.rows + t - 1) / t * ((w.cols + t - 1) / t) * w.groups; };
  const int64_t large = tiles(256);
  if (large > 2 * cus) return kTileK256;
  if (w.beside && 4 * large >= 3 * cus) return kTileK256;
  if (w.kind == WK_WGF32) {
    const int64_t three = cus * 3 / 4;
    return w.expect >= 512. && 3 * ((large + three - 1) / three) >= 4 * ((large + cus - 1) / cus) ? kTileK256
                                                                                                  : kTileK128;
  }
  if (w.expect < 512.) return kTileK128;
  const double steps = w.expect / 32.;
  auto cost = [&](int64_t n, int64_t per, double full, double store, double last) {
    return n / per * (steps * full + store) + (n % per ? steps * last + store : 0.);
  };
  const double fill = (double)(large % cus) / cus;
  const double c256 = 8000. + cost(large, cus, 900., 4000., fill <= 0.5 ? 720. : 540. + 360. * fill);
  const int64_t small = tiles(128), per = 3 * cus, rem = small % per;
  const int64_t slices = ((w.rows + 127) / 128 + (w.cols + 127) / 128) * w.groups;
  const double three = small > per ? 850. : slices <= 128 ? 780. : 1000.;
  const double c128 = 7000. + cost(small, per, three, 2000., rem <= cus ? 440. : rem <= 2 * cus ? 620. : three);
  if (c128 <= c256 + 3000.) return kTileK128;
  return 2 * large <= 3 * cus || c256 >= 1e5 ? kTileKByRows : kTileK256;
}
static void run_wide_any(const WideCall& w, hipStream_t s) {
  if (w.rows <= 0 || w.cols <= 0 || w.groups <= 0) return;
  if (w.kind < WK_DW) return kTilesM[tile_m(w, num_cus())].run(w, s);
  const TileK t = tile_k(w, num_cus());
  WideCall q = w;
  q.p.only = t == kTileKByRows ? 1 : 0;
  if (t != kTileK128) run_wide_256x256(q, s);
  q.p.only = t == kTileKByRows ? 2 : 0;
  if (t != kTileK256) run_wide_128x128(q, s);
}

// Rows a group is expected to hold, and their standard deviation: the call's
// assignments spread evenly (T is only a hint here: rows may come from elsewhere).
static WideCall expert_call(const moe_cfg& c, WideKind kind, const GemmParams& p, int64_t rows, int cols, bool later) {
  const double expect = c.T > 0 ? std::min<double>(c.C, (double)c.T * c.k / c.E) : c.C;
  const double spread = std::sqrt(expect * (1. - (double)c.k / c.E));
  // A later partition's rows start anywhere in a 16-row block.
  return WideCall{kind, c.act, c.E, rows, cols, expect + (later ? 7.5 : 0.), spread, p};
}
// The tile of a float product: the one whose busiest CU has the least work, tiles
// per CU times area, the 32-tile's extra loads per flop counted as 30 %.
// Measured, 64-tile against 32-tile: expert_out of 2000 tokens (d 512, f 2048, 8
// experts) 136 and 125 us, its H 113 and 123; dW of 63 tokens (d 640, f 1280, 8
// experts) 15 and 23, its H 24 and 15.
static int f32_tile(const WideCall& w, int cus) {
  auto cost = [&](int t, double f) {
    const double n = w.kind >= WK_DW ? std::ceil((double)w.rows / t)
                                     : 0.5 * (std::ceil(std::max(1., w.expect - w.spread) / t) +
                                              std::ceil((w.expect + w.spread) / t));
    return std::ceil(w.groups * n * std::ceil((double)w.cols / t) / cus) * t * t * f;
  };
  const bool fits = (double)w.groups * ((w.rows + 46) / 32) * ((w.cols + 31) / 32) <= 1 << 22;   // bounds the grid
  return fits && cost(32, 1.3) < cost(64, 1.) ? 32 : 64;
}

// Expert products.  bf16: blocked operands, wide tiles; outputs that a later
// product reads (H, A, dH) blocked, the others (expert_out, dXe, which only
// the gathers read, and the dW products) row-major.  float: the float MFMA
// kernel, row-major.
// rows: rows of the output per group (ragged-M: the capacity C, with up to 15
// alignment rows; ragged-K: M); cols: N.
template <bool B_K, bool RAGGED_K, int EPI>
static void run_expert(const moe_cfg& c, WideKind kind, const GemmParams& p, int64_t rows, int cols, hipStream_t s,
                       bool later = false, bool beside = false) {
  if (rows <= 0 || cols <= 0 || c.E <= 0) return;
  WideCall w = expert_call(c, kind, p, rows, cols, later);
  w.beside = beside;
  if (c.dtype != MOE_BF16) {
    if (f32_tile(w, num_cus()) == 32) launch_f32<1, B_K, RAGGED_K, EPI>(p, c.E, rows, cols, s);
    else launch_f32<2, B_K, RAGGED_K, EPI>(p, c.E, rows, cols, s);
    return;
  }
  run_wide_any(w, s);
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
                       const void* W2, void* H, void* A, void* O, void* ws, hipStream_t s, bool later) {
  const int64_t d = c.d_model, f = c.d_ff, C = c.C, Cp = rows_alloc(c);
  GemmParams p1{X, d, Cp * d, W1, d, f * d, H, f, Cp * f, A, nullptr, rb, re, 0, (int)f, (int)d, c.act, (int)C};
  p1.part = (float*)ws;
  p1.ksplit = c.ksplit;
  bool tb = ptimer_begin(kProdFwd1, s);
  run_expert<true, false, EPI_FWD1>(c, WK_FWD1, p1, C, (int)f, s, later);
  ptimer_end(tb, s);
  GemmParams p2{A, f, Cp * f, W2, f, d * f, O, d, Cp * d, nullptr, nullptr, rb, re, 0, (int)d, (int)f, c.act, (int)C};
  p2.part = (float*)ws;
  p2.ksplit = c.ksplit;
  tb = ptimer_begin(kProdFwd2, s);
  run_expert<true, false, EPI_STORE>(c, WK_NK, p2, C, (int)d, s, later);   // expert_out row-major
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
                          const int32_t* rb, const int32_t* re, void* dW1, void* dW2, hipStream_t s, bool beside) {
  const int64_t d = c.d_model, f = c.d_ff, C = c.C, Cp = rows_alloc(c);
  // dW2_e [d][f] = dO_e^T A_e : A-operand(m, k) = dO[e][k][m], B(k, n) = A[e][k][n]
  // (wpacked: written in the blocked layout of the packed weights)
  GemmParams p2{dO, d, Cp * d, A, f, Cp * f, dW2, f, d * f, nullptr, nullptr, rb, re, (int)d, (int)f, 0, c.act, (int)C};
  // dW1_e [f][d] = dH_e^T X_e
  GemmParams p1{dH, f, Cp * f, X, d, Cp * d, dW1, d, f * d, nullptr, nullptr, rb, re, (int)f, (int)d, 0, c.act, (int)C};
  const bool blk = c.wpacked && c.dtype == MOE_BF16;
  bool tb = ptimer_begin(kProdDW2, s);
  run_expert<false, true, EPI_STORE>(c, blk ? WK_DW_BLK : WK_DW, p2, d, (int)f, s, false, beside);
  ptimer_end(tb, s);
  tb = ptimer_begin(kProdDW1, s);
  run_expert<false, true, EPI_STORE>(c, blk ? WK_DW_BLK : WK_DW, p1, f, (int)d, s, false, beside);
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
void launch_dense_wgrad(int M, int N, int64_t K, const void* A, const void* B, void* C, void* part, hipStream_t s,
                        bool beside) {
  if (M <= 0 || N <= 0) return;
  const int S = kWgradSplit;
  const int64_t MN = (int64_t)M * N;
  GemmParams p{A, M, 0, B, N, 0, part, N, MN, nullptr, nullptr, nullptr, nullptr, M, N, 0, 0, (int)K};
  p.kchunk = (int)(((K + S - 1) / S + 31) / 32 * 32);
  run_wide_any(WideCall{WK_WGF32, MOE_ACT_IDENTITY, S, M, N, (double)std::min<int64_t>(K, p.kchunk), 0., p, beside},
               s);
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

// The tile, (rows << 16) + columns, that the choices above give an expert product
// (kProd*) of a call, or a dense product, on `cus` compute units (0: by the
// row counts).
int expert_tile(const moe_cfg& c, int product, bool later, int cus) {
  static const WideKind kinds[kProducts] = {WK_FWD1, WK_NK, WK_DACT, WK_KN, WK_DW, WK_DW};
  const bool to_f = product == kProdFwd1 || product == kProdDA || product == kProdDW2;   // N = f (else d)
  GemmParams p{};
  p.K = to_f ? c.d_model : c.d_ff;
  p.ksplit = c.ksplit;
  const bool dw = product == kProdDW2 || product == kProdDW1;
  const WideCall w = expert_call(c, kinds[product], p, dw ? (to_f ? c.d_model : c.d_ff) : c.C,
                                 to_f ? c.d_ff : c.d_model, later);
  if (c.dtype != MOE_BF16) return f32_tile(w, cus) * ((1 << 16) + 1);
  if (dw) {
    const TileK t = tile_k(w, cus);
    return t == kTileKByRows ? 0 : t == kTileK256 ? (256 << 16) + 256 : (128 << 16) + 128;
  }
  const TileCost& t = kTilesM[tile_m(w, cus)];
  return (t.bm << 16) + t.bn;
}
int dense_tile(int64_t M, int N, int K, int cus) {
  GemmParams p{};
  p.K = K;
  const TileCost& t = kTilesM[tile_m(WideCall{WK_NK, MOE_ACT_IDENTITY, 1, M, N, (double)M, 0., p}, cus)];
  return (t.bm << 16) + t.bn;
}

}  // namespace lmoe
