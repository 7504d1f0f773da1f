// The bf16 grouped GEMM: tiles of a persistent MFMA kernel, templated on the
// tile shape (see gemm.hip for the products and the choice of a tile).
#pragma once

#include "internal.h"
#include "lds_ops.h"

#include <type_traits>
#include <utility>

namespace lmoe {

// EPI_WGF32: the dense weight-gradient product C = A^T B of the block, both
// operands row-major [K][*] (not blocked), K split into groups of kchunk rows
// (group g: rows [g kchunk, (g + 1) kchunk)), each group's float partial C at
// C + g sC; gemm_wgrad_reduce_kernel adds the partials in group order.
enum { EPI_STORE = 0, EPI_FWD1 = 1, EPI_DACT = 2, EPI_RES = 3, EPI_WGF32 = 4 };

struct GemmParams {
  const void* A;
  int64_t lda, sA;
  const void* B;
  int64_t ldb, sB;
  void* C;
  int64_t ldc, sC;
  void* C2;         // EPI_FWD1: act(acc), same layout as C
  const void* Aux;  // EPI_DACT: pre-activation H; EPI_RES: residual added to the product; same layout as C
  const int32_t* rb;
  const int32_t* re;
  int M, N, K;      // ragged-M: N, K used;  ragged-K: M, N used
  int act;
  int cap;          // rows per expert block (C): row ranges are clamped to [0, cap]; re == NULL means [0, cap)
  float* part;      // wide ragged-M products: partial tiles of the K-split (stream-K) schedule
  int ksplit;       // wide plain-store ragged-M products: 1 = a short last round may be K-split
  int kchunk;       // rb == re == NULL and kchunk > 0: group g's rows are [g kchunk, (g + 1) kchunk)
  int only;         // ragged-K: 1 = run only if the groups are even, 2 = only if they are skewed, 0 = always
};

// Row range of group g, clamped to the buffer so bad ranges cannot reach outside it.
__device__ __forceinline__ void group_rows(const GemmParams& p, int g, int& lo, int& span) {
  int a = p.rb ? p.rb[g] : (p.kchunk > 0 ? g * p.kchunk : 0);
  int b = p.re ? p.re[g] : (p.kchunk > 0 ? (g + 1) * p.kchunk : p.cap);
  a = a < 0 ? 0 : (a > p.cap ? p.cap : a);
  b = b < a ? a : (b > p.cap ? p.cap : b);
  lo = a;
  span = b - a;
}

// ----------------------------------------------------------------- bf16 MFMA
// Operand tiles (BK = 32, one MFMA K step) move global -> LDS with buffer
// loads into LDS (each lane's 16 bytes land at LDS base + 16 * lane) into a
// multi-stage ring; a lane whose element lies outside the operand reads zeros.
//
// LDS layouts of a stage:
//  * K-contiguous operand, ROWS x 32: fragment-linear.  The 16 x 32 MFMA
//    fragment of rows 16f..16f+15 is 1 KB at offset 1 KB * f, lane L's 16
//    bytes (row 16f + L%16, k = 8*(L/16) .. +7) at 16 * L: one DMA instruction
//    fills one fragment and one ds_read_b128 reads it, both linear.
//  * MN-contiguous operand, 32 x COLS (row = k): [2][COLS/32] blocks of 16
//    rows x 4 chunks of 16 bytes, chunk c of block row r at c ^ bsw(r): the 16
//    lanes of a transposed read cover rows r..r+3 and the next lane group rows
//    r+8..r+11, and this swizzle puts those 8 x 32 bytes on distinct banks.
//    Fragments are read with ds_read_b64_tr_b16: within each 16-lane group,
//    lane j addresses row k0 + j/4, columns n0 + 4*(j%4) .. +3, and receives
//    column n0 + j of rows k0 .. k0+3 -- two such reads give the 8-element K
//    run of the MFMA operand.
constexpr int kBKb = 32;

// MN-contiguous operand: 32 x COLS tile (row = k), 64 chunks per wave instruction.
__device__ __forceinline__ int bsw(int r) { return 2 * (((r >> 1) ^ (r >> 3)) & 1); }
// LDS element offset of (k, col) in a stage of COLS columns.
template <int COLS>
__device__ __forceinline__ int mn_lds_off(int k, int col) {
  const int r = k & 15;
  return ((k >> 4) * (COLS / 32) + (col >> 5)) * 512 + r * 32 + ((((col & 31) >> 3) ^ bsw(r)) << 3) + (col & 7);
}

// Tiles of a group are numbered panel by panel (kPanelN tile columns wide),
// m-tile by m-tile inside a panel, n fastest, so the tiles an XCD has in
// flight form a square-ish patch whose operand slices are shared through that
// XCD's L2.
constexpr int kPanelN = 8;

// ------------------------------------------------------ wide bf16 MFMA tiles
// The largest shape (tile shapes: below), which the expert products take at full
// size.  256 x 256 block tiles, one block per CU,
// eight waves in a 2 x 4 grid, each owning a 128 x 64 tile (32 accumulator
// fragments) -- two waves per SIMD, so one wave's MFMAs issue while the other
// waits on memory.  Against 128 x 128 block tiles this halves the operand
// bytes a CU moves global -> LDS per flop; the per-CU load path is what limits
// the smaller tile.
//
// Operands reach LDS through raw buffer loads with the LDS flag: a scalar
// buffer descriptor covers the operand's group from the current K-step on, so
// a K-step only moves the descriptor, and an out-of-range lane sets bit 31 of
// its offset, which the buffer range check turns into zeros.  Each K-step's
// fragment reads for the next step and the loads refilling the stage just
// consumed are interleaved one instruction at a time between the step's
// MFMAs, so the wave keeps issuing MFMAs while memory operations queue.
//
// The K loop runs continuously over every tile a block owns: the load cursor
// runs STAGES K-steps ahead of the compute cursor and crosses into the block's
// next tile while the current one finishes, so that tile's first stages land
// while the epilogue stores.  After an epilogue the first wait is a full
// vmcnt(0): stores and loads share the counter, and the order in which they
// complete is not relied on.
//
// The accumulators live in AGPRs through inline-asm MFMAs ("+a"), which keeps
// every fragment in one register quad for the whole tile.  The compiler does
// not see those MFMAs, so the hazards it would otherwise cover are fenced by
// hand: s_nop after VALU writes of fragment registers an MFMA reads next, and
// after the last MFMA of a tile before the accumulators are read.
//
// The product is computed transposed (MFMA A operand = a B fragment, B operand
// = an A fragment), so each lane's four accumulator values are four
// consecutive output columns of one row: the epilogue converts them with
// v_cvt_pk_bf16_f32, swaps halves of two fragments between lane groups and
// stores 16-byte vectors straight from registers.
//
// LDS stages: four with one block barrier per K-step; five (the whole LDS)
// with one barrier per two K-steps (PAIR: the barrier before an even step
// covers the stages of both steps of the pair).  The products whose B operand
// is MN-contiguous (read transposed) run PAIR -- measured faster there (the
// ragged-K weight-gradient products -7 % at d_model 2048) -- and the
// K-contiguous ones four stages (PAIR measured +4 % there).
//
// Tile shapes.  Wide<BM, BN, NW, WGN, SUB, STB, STT, WPE, KSPLIT>: a BM x BN
// block tile, NW waves as (NW / WGN) x WGN, SUB MFMA K-steps of 32 per pipeline
// step, STB / STT stages for a K-contiguous / MN-contiguous B operand, WPE
// waves per SIMD, and whether a short last round may be K-split.  A product
// sums the same 32-wide MFMAs in K order whatever its tile, so tiles of any
// shape give the same bits.
template <int BM_, int BN_, int NW_, int WGN_, int SUB_, int STB, int STT, int WPE_, bool KSPLIT_, int BMT_ = BM_>
struct Wide {
  static constexpr int BM = BM_, BN = BN_, NW = NW_, WGN = WGN_, SUB = SUB_;
  static constexpr int BK = 32 * SUB;                     // K per step: SUB MFMA K-steps of 32
  static constexpr int WGM = NW / WGN;                    // wave grid WGM x WGN
  static constexpr int BMT = BMT_;                        // rows of a tile (the LDS stage has room for BM)
  static constexpr int WTM = BMT / WGM, WTN = BN / WGN;   // wave tile
  static constexpr int FM = WTM / 16, FN = WTN / 16;      // fragments per wave tile side
  static constexpr int NIA = BM / 16 / NW, NIB = BN / 16 / NW;   // loads per wave and 32 K (1 KB each)
  static constexpr int HALF = (BM + BN) * kBKb;           // elements per 32 K: A tile, then B tile
  static constexpr int STAGE = SUB * HALF;                // elements per pipeline stage
  static_assert(BM % (16 * NW) == 0 && BN % (16 * NW) == 0 && WTM % 32 == 0 && WTN % 32 == 0 && BMT <= BM, "tile / waves mismatch");
  static constexpr int WPE = WPE_;                        // waves per SIMD
  static constexpr int stages(bool b_k) { return b_k ? STB : STT; }
  static constexpr bool pair(bool b_k) { return stages(b_k) >= 5; }
  static constexpr bool KSPLIT = KSPLIT_;
  static constexpr size_t lds_bytes(bool b_k) { return (size_t)stages(b_k) * STAGE * sizeof(uint16_t); }
  static constexpr int per_cu(bool b_k) {                 // blocks resident on a CU
    return (int)std::min<size_t>(4 * WPE / NW, (size_t)160 * 1024 / lds_bytes(b_k));
  }
};

// Immediate byte offset of fragment read r from its base (see read_base in the
// kernel): K-contiguous fragment r sits r KB on; an MN-contiguous half r % 2
// of fragment r / 2 sits (r / 4) blocks and (r % 2) * 4 rows on.
template <bool KC, int R>
constexpr int wide_read_imm() {
  return KC ? R * 1024 : ((R >> 2) * 512 + (R & 1) * 128) * 2;
}

// Compile-time loop: f(std::integral_constant<int, I>) for I in [B, E).
template <int B, int E, typename Fn>
__device__ __forceinline__ void static_for(Fn&& f) {
  if constexpr (B < E) {
    f(std::integral_constant<int, B>{});
    static_for<B + 1, E>(f);
  }
}

struct WGeo {
  int g;        // group (expert)
  int m0, n0;   // tile origin (rows relative to lo_al for ragged-M products)
  int lo, hi;   // the group's row range in its [C][*] block
  int lo_al;    // lo rounded down to the 16-row block: origin of the tile rows (ragged-M) or of K (ragged-K)
  int Mlim, Klim, nk;
};

__device__ __forceinline__ uint32_t cvt_pk_bf16(float lo, float hi) {
  typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
  typedef float f32x2_t __attribute__((ext_vector_type(2)));
  return __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2_t{lo, hi}), bf16x2_t));
}
__device__ __forceinline__ u32x2 pack4_bf16(const float (&v)[4]) {
  return u32x2{cvt_pk_bf16(v[0], v[1]), cvt_pk_bf16(v[2], v[3])};
}

__device__ __forceinline__ void mfma_acc(f32x4& acc, const u32x4& a, const u32x4& b) {
  asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(acc) : "v"(a), "v"(b));
}
// Wait states between VALU writes of fragment registers and the MFMAs that
// read them: no MFMA on these fragments moves above the fence.
template <int N>
__device__ __forceinline__ void valu_to_mfma_fence(u32x4 (&f)[N]) {
  static_assert(N % 2 == 0, "fragment count");
#pragma unroll
  for (int i = 2; i < N; i += 2) asm volatile("" : "+v"(f[i]), "+v"(f[i + 1]));
  asm volatile("s_nop 4" : "+v"(f[0]), "+v"(f[1]));
}
// Pins a row of accumulators in AGPRs at this point of the instruction stream.
template <int N>
__device__ __forceinline__ void acc_pin(f32x4 (&a)[N]) {
#pragma unroll
  for (int i = 0; i < N; i += 2) asm volatile("" : "+a"(a[i]), "+a"(a[i + 1]));
}
// The same, ordered after every earlier memory operation.
template <int N>
__device__ __forceinline__ void acc_pin_mem(f32x4 (&a)[N]) {
#pragma unroll
  for (int i = 0; i < N; i += 2) asm volatile("" : "+a"(a[i]), "+a"(a[i + 1])::"memory");
}

// One operand's loads for the K-steps of a tile (ROWS rows or columns x 32 K
// per stage, blocked source), as raw buffer loads into LDS.  The buffer
// descriptor spans the operand's group (expert) from the current K-step on, so
// a K-step only moves the descriptor (scalar adds), and a lane whose chunk is
// out of range carries bit 31 in its offset, which the buffer range check
// turns into zeros.  K-contiguous (KC): the chunk of fragment q is a whole
// 16 x 32 block, rows past `lim` read zeros.  MN-contiguous: 32 K rows x ROWS
// columns as 2 x ROWS / 32 blocks, each lane's chunk placed at its swizzled position;
// columns past `lim` and, with KCHK, K rows outside [klo, khi) read zeros.
constexpr int kBufCfg = 0x00020000;   // buffer descriptor word 3: raw 32-bit data, gfx9 family
constexpr uint32_t kOob = 0x80000000u;
// RM (MN-contiguous only): the operand is row-major [K][ld] instead of blocked;
// a lane loads the same 16-byte chunk (K row, 8 columns) that it would take
// from the blocked layout, so the stage's LDS layout is the same.
template <bool KC, bool KCHK, int NW, int ROWS, bool RM = false>
struct WOp {
  static constexpr int kWNI = ROWS / 16 / NW;   // loads per wave per stage (1 KB blocks)
  const char* base;      // the group's operand (uniform)
  uint32_t bytes;        // its extent in bytes (uniform)
  uint32_t stride;       // bytes per K-step (uniform)
  uint32_t voff[kWNI];   // byte offset of the lane's chunk at K-step 0, | kOob if out of range
  int kr[kWNI];          // KCHK: K row of the lane's chunk at K-step 0
  int klo, khi;

  // KC: row0 = first row of the tile (multiple of 16), lim = row limit.
  // MN: row0 = first column of the tile, lim = column limit, korg = K origin (multiple of 16).
  __device__ __forceinline__ void plan(const uint16_t* b, int64_t extent, int64_t ld, int row0, int lim, int korg,
                                       int lo, int hi, int wid, int lane) {
    base = (const char*)b;
    bytes = (uint32_t)(extent * 2);
    klo = lo;
    khi = hi;
    if constexpr (KC) {
      stride = 1024;
#pragma unroll
      for (int i = 0; i < kWNI; ++i) {
        const int rb = (row0 >> 4) + i * NW + wid;
        const uint32_t off = (uint32_t)(rb * (int)(ld >> 5) * 512 + (lane & 15) * 32 + (lane >> 4) * 8) * 2u;
        voff[i] = (16 * rb + (lane & 15) < lim) ? off : (off | kOob);
        kr[i] = 0;
      }
    } else {
      const int nb = (int)(ld >> 5);
      stride = RM ? (uint32_t)(32 * ld * 2) : (uint32_t)nb * 2048u;
      const int r = lane >> 2;
      const int c = (lane & 3) ^ bsw(r);
#pragma unroll
      for (int i = 0; i < kWNI; ++i) {
        const int b2 = i * NW + wid;
        const int kb = b2 / (ROWS / 32), cb = b2 % (ROWS / 32);
        const int col = row0 + 32 * cb;
        const uint32_t off =
            RM ? (uint32_t)(((int64_t)(korg + 16 * kb + r) * ld + col + c * 8) * 2)
               : (uint32_t)((((korg >> 4) + kb) * nb + (col >> 5)) * 512 + r * 32 + c * 8) * 2u;
        voff[i] = col < lim ? off : (off | kOob);
        kr[i] = korg + 16 * kb + r;
      }
    }
  }
  // Load i (0 .. kWNI-1) of K-step kk into its place in the stage.
  __device__ __forceinline__ void issue(int i, int kk, uint16_t* stage, int wid) const {
    const uint32_t adv = (uint32_t)kk * stride;
    const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc((void*)(base + adv), (short)0, (int)(bytes - adv), kBufCfg);
    uint32_t vo = voff[i];
    if constexpr (KCHK) {
      const int k = kr[i] + 32 * kk;
      if (k < klo || k >= khi) vo |= kOob;
    }
    __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (lds_void*)(stage + (i * NW + wid) * 512), 16, vo, 0, 0, 0);
  }
  // The same, branch-free, with the K-step's descriptor made once per step:
  // with live false the descriptor is empty, so the load writes zeros into
  // the stage (a stage no later step reads).
  __device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc(int kk, bool live) const {
    const uint32_t adv = (uint32_t)kk * stride;
    return __builtin_amdgcn_make_buffer_rsrc((void*)(base + adv), (short)0, live ? (int)(bytes - adv) : 0, kBufCfg);
  }
  __device__ __forceinline__ void issue_r(int i, __amdgpu_buffer_rsrc_t r, int kk, uint16_t* stage, int wid) const {
    uint32_t vo = voff[i];
    if constexpr (KCHK) {
      const int k = kr[i] + 32 * kk;
      if (k < klo || k >= khi) vo |= kOob;
    }
    __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (lds_void*)(stage + (i * NW + wid) * 512), 16, vo, 0, 0, 0);
  }
};

// Schedule of one XCD's n tiles xtile(0 .. n-1) over its nslot blocks.  Rounds
// of whole tiles run in lock step (block s takes tiles xtile(q nslot + s)), so the
// tiles in flight share their K position and their operand slices in L2.  A
// last round that would leave most blocks idle (r <= nslot / 4 tiles) is
// split instead: the r tiles' K-steps go to all nslot blocks, each tile to a
// contiguous group of blocks, each block a contiguous K range of one tile;
// the partial sums are added by gemm_wide_fixup_kernel.
struct WSched {
  int R, r;      // full rounds; tiles left for the last round
  bool split;    // the last round is K-split
  // K-split: the remainder tile of block `slot`, the first block of that tile,
  // its number of blocks, and the block's K range [k0, k1).
  __device__ __forceinline__ void split_part(int slot, int nslot, int nk, int& q, int& first, int& cnt, int& k0,
                                             int& k1) const {
    q = slot * r / nslot;
    first = (q * nslot + r - 1) / r;
    cnt = ((q + 1) * nslot + r - 1) / r - first;
    const int rank = slot - first;
    k0 = rank * nk / cnt;
    k1 = (rank + 1) * nk / cnt;
  }
};
__device__ __forceinline__ WSched wide_sched(int n, int nslot, bool allow_split) {
  WSched w;
  w.R = n / nslot;
  w.r = n - w.R * nslot;
  w.split = allow_split && w.r > 0 && 4 * w.r <= nslot;
  return w;
}

// Lane-per-group tile counts of a wide product and their prefixes (groups <= 64).
// Ragged-K, or ragged-M without SEP: every tile of a group (with rows); ragged-K
// prefixes run over the groups by rows, most first.
// Ragged-M with SEP: the full M-tiles (BM rows) and, separately, the short
// last M-tile of a group whose rows are not a multiple of BM; tile numbers
// [0, NF) are the full tiles, [NF, NF + NP) the short ones, so a schedule can
// place the short (cheaper) tiles last.
struct WPrefix {
  int incl, excl;     // full tiles (ragged-K: all tiles), lane = group
  int inclP, exclP;   // ragged-M short tiles, lane = group
  int NF, NP;         // totals (uniform)
  int lo, span;       // the group's clamped row range (group_rows), lane = group: read once, so a
                      // tile change never waits on a memory load (which would drain the wave's
                      // in-flight operand loads and epilogue stores)
};
template <int BM, bool RAGGED_K, bool SEP>
__device__ __forceinline__ WPrefix wide_tile_prefix(const GemmParams& p, int lane, int groups, int tilesM,
                                                    int tilesN) {
  int cnt = 0, cntP = 0;
  int lo = 0, span = 0;
  if (lane < groups) {
    group_rows(p, lane, lo, span);
    if constexpr (RAGGED_K) {
      cnt = span > 0 ? tilesM * tilesN : 0;   // an empty group's output is zeroed in the prologue
    } else {
      const int rows = span > 0 ? span + (lo & 15) : 0;   // from the 16-row block holding the first row
      const int tm = (rows + BM - 1) / BM;
      const int sh = (SEP && (rows % BM) != 0) ? 1 : 0;
      cnt = (tm - sh) * tilesN;
      cntP = sh * tilesN;
    }
  }
  WPrefix P;
  P.lo = lo;
  P.span = span;
  if constexpr (RAGGED_K) {
    // Groups by rows, most first (ties by index): a tile is as long as its group,
    // and a round of the schedule then holds tiles of nearly one length.  One key per
    // group (rows past 2^25 count as that many), so a group costs a broadcast, a
    // comparison and an addition.
    const int key = min(span, (1 << 25) - 1) * 64 + 63 - lane;
    int ahead = 0;
    for (int h = 0; h < groups; ++h) ahead += __builtin_amdgcn_readlane(key, h) > key ? 1 : 0;
    const int per = tilesM * tilesN;   // (of a group with rows; the groups without are the last)
    const int before = per * ahead;
    const int all = per * __popcll(__ballot(span > 0));
    P.excl = before;
    P.incl = before + cnt;
    P.inclP = P.exclP = 0;
    P.NF = all;
    P.NP = 0;
    return P;
  }
  P.incl = cnt;
  P.inclP = cntP;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int u = __shfl_up(P.incl, o, 64);
    const int v = __shfl_up(P.inclP, o, 64);
    if (lane >= o) {
      P.incl += u;
      P.inclP += v;
    }
  }
  P.excl = P.incl - cnt;
  P.exclP = P.inclP - cntP;
  P.NF = __builtin_amdgcn_readfirstlane(__shfl(P.incl, groups - 1, 64));
  P.NP = __builtin_amdgcn_readfirstlane(__shfl(P.inclP, groups - 1, 64));
  return P;
}

// Geometry of tile t of a wide product.  Within a group, tiles (with SEP: the
// full tiles) are numbered panel by panel (kPanelN tile columns), m-tiles
// within a panel, n fastest, so the tiles one XCD has in flight form a
// square-ish patch; with SEP a group's short last M-tile has its own numbers
// (t >= NF), n order.
template <int BM, int BN, int BK, bool RAGGED_K, bool SEP>
__device__ __forceinline__ WGeo wide_geo(const GemmParams& p, int t, int lane, int groups, const WPrefix& P,
                                         int tilesM, int tilesN) {
  WGeo G;
  const bool shrt = SEP && !RAGGED_K && t >= P.NF;
  const int tt = shrt ? t - P.NF : t;
  const int inc = shrt ? P.inclP : P.incl;
  const int exc = shrt ? P.exclP : P.excl;
  // The group holding tile tt: by its own range (ragged-K: groups in row order), or counting the groups before it.
  G.g = RAGGED_K ? __builtin_ctzll(__ballot(lane < groups && exc <= tt && tt < inc) | (1ull << 63))
                 : __builtin_amdgcn_readfirstlane(__popcll(__ballot(lane < groups && inc <= tt)));
  const int local = tt - __builtin_amdgcn_readlane(exc, G.g);
  const int lo = __builtin_amdgcn_readlane(P.lo, G.g);
  int span = __builtin_amdgcn_readlane(P.span, G.g);
  G.lo = lo;
  G.hi = lo + span;
  G.lo_al = lo & ~15;
  if (span > 0) span += lo - G.lo_al;
  if (shrt) {
    G.m0 = ((span + BM - 1) / BM - 1) * BM;
    G.n0 = local * BN;
  } else {
    const int tmg = RAGGED_K ? tilesM : (SEP ? span / BM : (span + BM - 1) / BM);   // (full) M-tiles
    const int pnl = local / (tmg * kPanelN);
    const int rem = local - pnl * tmg * kPanelN;
    const int pw = min(kPanelN, tilesN - pnl * kPanelN);
    G.m0 = (rem / pw) * BM;
    G.n0 = (pnl * kPanelN + rem % pw) * BN;
  }
  G.Mlim = RAGGED_K ? p.M : span;
  G.Klim = RAGGED_K ? span : p.K;
  G.nk = max(1, (G.Klim + BK - 1) / BK);
  return G;
}

// One XCD's tiles of a ragged-M product: an even share of the full tiles, as
// one contiguous range (neighbouring operand panels in the XCD's L2), then an
// even share of the short tiles.  tile(j) = the XCD's j-th tile.
struct WRange {
  int f0, nf, p0, np, NF;
  __device__ __forceinline__ int tile(int j) const { return j < nf ? f0 + j : NF + p0 + (j - nf); }
};
__device__ __forceinline__ WRange wide_range(const WPrefix& P, int xcd) {
  WRange r;
  const int perF = (P.NF + 7) / 8, perP = (P.NP + 7) / 8;
  r.f0 = xcd * perF;
  r.nf = max(min(P.NF, r.f0 + perF) - r.f0, 0);
  r.p0 = xcd * perP;
  r.np = max(min(P.NP, r.p0 + perP) - r.p0, 0);
  r.NF = P.NF;
  return r;
}

// Epilogue of one wave's tile from its accumulators: bf16 conversion and the
// EPI-specific store (plain, (H, act(H)), or dA * act'(H) with H read back).
// acc[i][j] holds output row 16 i + l % 16, columns 16 j + 4 (l / 16) .. +3 of
// the wave tile at (G.m0 + wm WTM, G.n0 + wn WTN).
template <int FM, int FN, int WTM, int WTN, bool RAGGED_K, int EPI, int ACT, bool CBLK>
__device__ __forceinline__ void wide_epilogue(const GemmParams& p, const WGeo& G, f32x4 (&acc)[FM][FN], int wm,
                                              int wn, int lane, int i_lo = 0, int i_hi = FM) {
  // Buffer stores and loads over the group's output: a lane outside the
  // product carries an out-of-range offset (store dropped, load zero), so
  // the epilogue is branch-free and dA * act'(H) issues all of a half's H
  // loads together.  Group offsets fit 31 bits (validated on the host).
  const int64_t cofs = (int64_t)G.g * p.sC + (RAGGED_K || CBLK ? 0 : (int64_t)G.lo_al * p.ldc);
  constexpr int ESZ = EPI == EPI_WGF32 ? 4 : 2;   // bytes per output element
  void* const cbase = EPI == EPI_WGF32 ? (void*)((float*)p.C + cofs) : (void*)((uint16_t*)p.C + cofs);
  const __amdgpu_buffer_rsrc_t rC = __builtin_amdgcn_make_buffer_rsrc(cbase, (short)0, 0x7fffffff, kBufCfg);
  __amdgpu_buffer_rsrc_t rC2 = rC, rAux = rC;
  if constexpr (EPI == EPI_FWD1)
    rC2 = __builtin_amdgcn_make_buffer_rsrc((uint16_t*)p.C2 + cofs, (short)0, 0x7fffffff, kBufCfg);
  if constexpr (EPI == EPI_DACT || EPI == EPI_RES)
    rAux = __builtin_amdgcn_make_buffer_rsrc((uint16_t*)p.Aux + cofs, (short)0, 0x7fffffff, kBufCfg);
  const int rl = lane & 15, q = lane >> 4;
  auto voff = [&](bool ok, int row, int col) __attribute__((always_inline)) -> uint32_t {
    const int64_t e = CBLK ? blk_off((RAGGED_K ? 0 : G.lo_al) + row, col, p.ldc) : (int64_t)row * p.ldc + col;
    return ok ? (uint32_t)(e * ESZ) : kOob;
  };
  auto row_of = [&](int i) __attribute__((always_inline)) { return G.m0 + wm * WTM + 16 * i + rl; };
  auto row_ok = [&](int i) __attribute__((always_inline)) {
    const int row = row_of(i);
    return row < G.Mlim && (RAGGED_K || G.lo_al + row >= G.lo) && i >= i_lo && i < i_hi;
  };
  if constexpr (EPI == EPI_WGF32) {
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
      for (int j = 0; j < FN; ++j) {
        const int col = G.n0 + wn * WTN + 16 * j + 4 * q;
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, acc[i][j]), rC,
                                               (int)voff(row_ok(i) && col < p.N, row_of(i), col), 0, 0);
      }
    return;
  }
  // bf16 outputs move as 16 bytes per lane: of a pair of fragments (32 columns)
  // a lane holds columns 4 q .. +3 of each 16; swapping the odd 16-lane groups of
  // the first with the even ones of the second leaves it columns cq .. cq + 7 of
  // the 32, cq = 16 (q % 2) + 8 (q / 2), so a wave's store covers whole 64-byte
  // row pieces (a blocked output: one contiguous KiB) with half the instructions.
  const int cq = 16 * (q & 1) + 8 * (q >> 1);
  constexpr int FP = FN / 2;
  auto swap = [](u32x2& a, u32x2& b) __attribute__((always_inline)) {   // (its own inverse)
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const auto r = __builtin_amdgcn_permlane16_swap(a[u], b[u], false, false);
      a[u] = r[0];
      b[u] = r[1];
    }
  };
  auto store = [&](u32x2 a, u32x2 b, __amdgpu_buffer_rsrc_t rs, int vo) __attribute__((always_inline)) {
    swap(a, b);
    __builtin_amdgcn_raw_buffer_store_b128(u32x4{a[0], a[1], b[0], b[1]}, rs, vo, 0, 0);
  };
  constexpr int HR = FM % 4 == 0 ? 4 : FM % 3 == 0 ? 3 : 2;
#pragma unroll
  for (int h = 0; h < FM / HR; ++h) {    // groups of up to four fragment rows
    u32x4 aux[HR][FP];
    if constexpr (EPI == EPI_DACT || EPI == EPI_RES) {   // all loads of the group first, then the math
#pragma unroll
      for (int ii = 0; ii < HR; ++ii)
#pragma unroll
        for (int jp = 0; jp < FP; ++jp) {
          const int col = G.n0 + wn * WTN + 32 * jp + cq;
          aux[ii][jp] = __builtin_amdgcn_raw_buffer_load_b128(
              rAux, (int)voff(row_ok(HR * h + ii) && col < p.N, row_of(HR * h + ii), col), 0, 0);
        }
    }
#pragma unroll
    for (int ii = 0; ii < HR; ++ii) {
      const int i = HR * h + ii;
      if (i < i_lo || i >= i_hi) continue;
#pragma unroll
      for (int jp = 0; jp < FP; ++jp) {
        const int col = G.n0 + wn * WTN + 32 * jp + cq;
        const int vo = (int)voff(row_ok(i) && col < p.N, row_of(i), col);
        float v[2][4];
#pragma unroll
        for (int e = 0; e < 2; ++e)
#pragma unroll
          for (int u = 0; u < 4; ++u) v[e][u] = acc[i][2 * jp + e][u];
        if constexpr (EPI == EPI_FWD1) {
          store(pack4_bf16(v[0]), pack4_bf16(v[1]), rC, vo);
#pragma unroll
          for (int e = 0; e < 2; ++e)
#pragma unroll
            for (int u = 0; u < 4; ++u) v[e][u] = act_fwd_t<ACT>(v[e][u]);
          store(pack4_bf16(v[0]), pack4_bf16(v[1]), rC2, vo);
          continue;
        }
        if constexpr (EPI == EPI_DACT || EPI == EPI_RES) {
          u32x2 x[2] = {u32x2{aux[ii][jp][0], aux[ii][jp][1]}, u32x2{aux[ii][jp][2], aux[ii][jp][3]}};
          swap(x[0], x[1]);
#pragma unroll
          for (int e = 0; e < 2; ++e) {
            const float f[4] = {__uint_as_float(x[e][0] << 16), __uint_as_float(x[e][0] & 0xffff0000u),
                                __uint_as_float(x[e][1] << 16), __uint_as_float(x[e][1] & 0xffff0000u)};
#pragma unroll
            for (int u = 0; u < 4; ++u) v[e][u] = EPI == EPI_DACT ? v[e][u] * act_bwd_t<ACT>(f[u]) : v[e][u] + f[u];
          }
        }
        store(pack4_bf16(v[0]), pack4_bf16(v[1]), rC, vo);
      }
    }
  }
}

template <class TC, bool B_K, bool RAGGED_K, int EPI, int ACT, bool CBLK>
__global__ __attribute__((amdgpu_flat_work_group_size(TC::NW * 64, TC::NW * 64), amdgpu_waves_per_eu(TC::WPE, TC::WPE))) void
gemm_wide_kernel(GemmParams p, int tilesM, int tilesN, int groups) {
  constexpr int BK = TC::BK, SUB = TC::SUB, HALF = TC::HALF;
  constexpr int BM = TC::BM, BN = TC::BN, BMT = TC::BMT, NW = TC::NW, WGN = TC::WGN;
  constexpr int WTM = TC::WTM, WTN = TC::WTN;   // wave tile
  constexpr int FM = TC::FM, FN = TC::FN;       // fragments per wave tile side
  constexpr int NIA = TC::NIA, NIB = TC::NIB;
  constexpr int STAGE = TC::STAGE;              // elements per pipeline stage
  constexpr bool AK = !RAGGED_K;                // A, B K-contiguous (else MN-contiguous)
  constexpr bool BKK = B_K && !RAGGED_K;
  constexpr int STAGES = TC::stages(B_K);
  constexpr int LPS = SUB * (NIA + NIB);         // loads per wave per stage
  // Every 32-K half of a step must start inside the operand (a descriptor's
  // size past its end would wrap): ragged-M products have K a multiple of 64,
  // a ragged-K group may end in any 32 rows.
  static_assert(SUB == 1 || (SUB == 2 && !RAGGED_K), "two halves per step: ragged-M products only");
  static_assert(BMT == BM || !RAGGED_K, "short tiles: ragged-M products only");
  static_assert(STAGES >= 2 && LPS * (STAGES - 1) < 64, "vmcnt range");
  constexpr bool PAIR = TC::pair(B_K);
  extern __shared__ __attribute__((aligned(16))) uint16_t lds[];

  const int lane = threadIdx.x & 63;
  const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wid / WGN, wn = wid % WGN;

  // Tile counts per group and their prefix (every wave computes the same values).
  // Only the plain-store ragged-M products may K-split their last round (the
  // narrow-N products where a ragged last round idles most of the GPU); the
  // others keep the simpler whole-tile schedule and its register budget.
  // The K-split products place their short tiles last (SEP), so the split
  // round holds the short tiles, whose partial sums stop at the group's rows.
  constexpr bool SPLIT = TC::KSPLIT && !RAGGED_K && EPI == EPI_STORE;
  if constexpr (RAGGED_K && EPI != EPI_WGF32) {
    // A product launched on two tile shapes: the row counts say which one runs
    // (skewed: the longest group has at least 1.5 times the mean of all).
    if (p.only != 0) {
      int lo = 0, span = 0;
      if (lane < groups) group_rows(p, lane, lo, span);
      int most = span, all = span;   // (64 groups of less than 2^24 rows)
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) {
        most = max(most, __shfl_xor(most, o, kWave));
        all += __shfl_xor(all, o, kWave);
      }
      const bool skewed = 2 * (int64_t)most * groups >= 3 * (int64_t)all;
      if (__builtin_amdgcn_readfirstlane((int)skewed) != (p.only == 2 ? 1 : 0)) return;
    }
  }
  const WPrefix P = wide_tile_prefix<BMT, RAGGED_K, SPLIT>(p, lane, groups, tilesM, tilesN);
  const int total = P.NF + P.NP;
  if constexpr (RAGGED_K) {
    // Groups without rows have no tiles: their [M][N] outputs are zeroed here,
    // spread over the whole grid (16-byte stores; no tile writes them).
    uint64_t empty = __ballot(lane < groups && P.incl == P.excl);
    const int64_t chunks = (int64_t)p.M * p.N / (EPI == EPI_WGF32 ? 4 : 8);
    const int64_t gtid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x, gstride = (int64_t)gridDim.x * blockDim.x;
    while (empty) {
      const int g = __builtin_ctzll(empty);
      empty &= empty - 1;
      u32x4* o = EPI == EPI_WGF32 ? reinterpret_cast<u32x4*>((float*)p.C + (int64_t)g * p.sC)
                                  : reinterpret_cast<u32x4*>((uint16_t*)p.C + (int64_t)g * p.sC);
      for (int64_t i = gtid; i < chunks; i += gstride) o[i] = u32x4{0u, 0u, 0u, 0u};
    }
  }
  const int nslot = gridDim.x / 8;
  const int xcd = blockIdx.x % 8, slot = blockIdx.x / 8;
  // The XCD's tiles: ragged-M products (one K length) take a contiguous range
  // of the (full) tiles, so the XCD's L2 holds neighbouring operand panels,
  // then with SEP their share of the short last M-tiles;
  // ragged-K products, whose tiles cost as many K-steps as their group has
  // rows, take every eighth tile, so each XCD gets an even share of every
  // group (with skewed routing, a contiguous range could hold the few large
  // groups), longest groups first.  xtile(j) = the XCD's j-th tile.  (In index
  // order the large groups' tiles met on the same slots: dW of 32768 tokens over
  // 64 experts, Zipf 1.2, 220 to 265 us by where they stood; by rows 190 to 201.)
  // The block's segments (see WSched): nd whole tiles xtile(e nslot + slot),
  // then, if the last round is K-split (ragged-M products, one K length), the
  // K range [sk0, sk1) of remainder tile xtile(R nslot + sq).
  const WRange XR = wide_range(P, xcd);
  const int nx = RAGGED_K ? (total > xcd ? (total - xcd + 7) / 8 : 0) : XR.nf + XR.np;
  auto xtile = [&](int j) __attribute__((always_inline)) { return RAGGED_K ? xcd + 8 * j : XR.tile(j); };
  const int nkU = (p.K + BK - 1) / BK;
  const WSched W = wide_sched(nx, nslot, SPLIT && p.ksplit != 0);
  int sq = 0, sfirst = 0, scnt = 0, sk0 = 0, sk1 = 0;
  if (SPLIT && W.split) W.split_part(slot, nslot, nkU, sq, sfirst, scnt, sk0, sk1);
  // (uniform values: keep them in scalar registers)
  const int WR = __builtin_amdgcn_readfirstlane(W.R);
  sq = __builtin_amdgcn_readfirstlane(sq);
  sk0 = __builtin_amdgcn_readfirstlane(sk0);
  sk1 = __builtin_amdgcn_readfirstlane(sk1);
  // Ragged-K rounds run through the slots forth and back (as the groups come
  // longest first, a slot that got the longer tile of one round gets the shorter
  // of the next).
  auto slot_of = [&](int e) __attribute__((always_inline)) { return RAGGED_K && (e & 1) ? nslot - 1 - slot : slot; };
  const int nd = __builtin_amdgcn_readfirstlane(W.R + (!W.split && slot_of(W.R) < W.r ? 1 : 0));
  const int nseg = __builtin_amdgcn_readfirstlane(nd + (SPLIT && W.split && sk0 < sk1 ? 1 : 0));
  if (nseg == 0) return;

  auto geo = [&](int t) __attribute__((always_inline)) {
    return wide_geo<BMT, BN, BK, RAGGED_K, SPLIT>(p, t, lane, groups, P, tilesM, tilesN);
  };

  // Segment e: tile, first K-step, end K-step (0 = the tile's own count).
  auto seg = [&](int e, int& t, int& k0, int& k1) __attribute__((always_inline)) {
    if (e < nd) {
      t = xtile(e * nslot + slot_of(e));
      k0 = 0;
      k1 = 0;
    } else {
      t = xtile(WR * nslot + sq);
      k0 = sk0;
      k1 = sk1;
    }
  };
  // Load cursor: segment le, its tile lt, K-step lk, end lkend; ls = stages
  // issued so far.
  // EPI_WGF32: both operands row-major and shared by every group (each group
  // a K range of them), so the extent is the whole operand.
  constexpr bool RMO = EPI == EPI_WGF32;
  static_assert(!RMO || RAGGED_K, "row-major operands: ragged-K products only");
  WOp<AK, RAGGED_K, NW, BM, RMO> opA;
  WOp<BKK, RAGGED_K, NW, BN, RMO> opB;
  int le = 0, lt = 0, lk = 0, lkend = 0, ls = 0;
  auto plan = [&](int t) __attribute__((always_inline)) {
    const WGeo G = geo(t);
    const uint16_t* Ab = (const uint16_t*)p.A + (RMO ? 0 : G.g * p.sA);
    const uint16_t* Bb = (const uint16_t*)p.B + (RMO ? 0 : G.g * p.sB);
    const int64_t extA = RMO ? (int64_t)p.cap * p.lda : p.sA, extB = RMO ? (int64_t)p.cap * p.ldb : p.sB;
    // (rows of the stage past the tile's BMT are not loaded: their places get zeros, which no wave reads)
    const int rlim = min((int)pad16(p.cap), G.lo_al + G.m0 + BMT);
    if constexpr (AK) opA.plan(Ab, p.sA, p.lda, G.lo_al + G.m0, rlim, 0, 0, 0, wid, lane);
    else opA.plan(Ab, extA, p.lda, G.m0, p.M, G.lo_al, G.lo, G.hi, wid, lane);
    if constexpr (BKK) opB.plan(Bb, p.sB, p.ldb, G.n0, p.N, 0, 0, 0, wid, lane);
    else if constexpr (RAGGED_K) opB.plan(Bb, extB, p.ldb, G.n0, p.N, G.lo_al, G.lo, G.hi, wid, lane);
    else opB.plan(Bb, p.sB, p.ldb, G.n0, p.N, 0, 0, p.K, wid, lane);
    if (lkend == 0) lkend = G.nk;
  };
  auto enter = [&]() __attribute__((always_inline)) {   // load cursor onto segment le
    seg(le, lt, lk, lkend);
    plan(lt);
  };
  enter();
  auto loads_left = [&]() __attribute__((always_inline)) { return le < nseg; };
  // Loads of the next stage.
  auto issue_stage = [&]() __attribute__((always_inline)) {
    if (!loads_left()) return;
#pragma unroll
    for (int h = 0; h < SUB; ++h) {
      uint16_t* st = lds + ((unsigned)ls % STAGES) * STAGE + h * HALF;
#pragma unroll
      for (int q = 0; q < NIA; ++q) opA.issue(q, lk * SUB + h, st, wid);
#pragma unroll
      for (int q = 0; q < NIB; ++q) opB.issue(q, lk * SUB + h, st + BM * kBKb, wid);
    }
  };
  // Moves the load cursor past the stage just issued.
  auto advance = [&]() __attribute__((always_inline)) {
    if (!loads_left()) return;
    ++ls;
    if (++lk == lkend) {
      ++le;
      if (loads_left()) enter();
    }
  };

  f32x4 acc[FM][FN];
  auto zero_acc = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
      for (int j = 0; j < FN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    asm volatile("s_nop 4" ::: "memory");
#pragma unroll
    for (int i = 0; i < FM; ++i) acc_pin(acc[i]);
  };
  auto epilogue = [&](const WGeo& G) __attribute__((always_inline)) {
    // Wait states between the last MFMA and the first read of its accumulator.
    asm volatile("s_nop 15\n s_nop 15" ::: "memory");
#pragma unroll
    for (int i = 0; i < FM; ++i) acc_pin(acc[i]);
    wide_epilogue<FM, FN, WTM, WTN, RAGGED_K, EPI, ACT, CBLK>(p, G, acc, wm, wn, lane);
  };

  int cs = 0;                // compute steps done (over all of the block's tiles)
  // The first step after an epilogue drains every store before its barrier
  // (measured faster than letting the stores overlap the next tile's loads).
  bool stores_pending = false;
  // One K-step: multiply the fragments in (ca, cb) while the next stage's
  // loads are issued and its fragments read into (na, nb).
  // Fragment read plan of the next stage: NRA reads for A, NRB for B (one
  // ds_read_b128 per K-contiguous fragment, two ds_read_b64_tr_b16 per
  // MN-contiguous one), each landing in its fragment or in a half-fragment
  // pending register.
  constexpr int NRA = AK ? FM : 2 * FM, NRB = BKK ? FN : 2 * FN, NRH = NRA + NRB, NRD = SUB * NRH;
  constexpr int NMH = FM * FN, NMF = SUB * NMH, NDMA = LPS;
  // PRE: MFMAs of a step issued before its wait and barrier (they use the
  // fragments read in the previous step), at the low wave priority; the rest
  // of the step, with the reads and refills, follows the barrier at the raised
  // priority.  Of the two waves on a SIMD the older one wins every tie for the
  // matrix core, so it finishes its MFMAs first and then waits at the barrier
  // while the other still issues; the early wave's PRE MFMAs of the next step
  // fill the matrix core while the late wave finishes its step, waits and
  // passes the barrier.  Measured (16384-token layer, one MI355X, per-wave
  // cycle counters): FWD2 1750 -> 1564 cycles per K-step, dXe 1773 -> 1505;
  // the layer's ragged-M calls -4 to -7 %, 12 and 16 equal, 20 and 24 slower.
  // The ragged-K (dW) products were measured slower with it (+2 %) and keep 0.
  constexpr int PRE = RAGGED_K ? 0 : NMF / 2;
  constexpr int RSPAN = (NMF - PRE) * 3 / 4;  // reads issued within the first 3/4 of the MFMAs after PRE
  u32x2 qa[SUB * 2 * FM], qb[SUB * 2 * FN];               // pending halves of MN-contiguous fragments
  // LDS byte address of read r of an operand = base(par) + imm(r), with a
  // compile-time immediate, so a step needs one or two base registers per
  // operand.  K-contiguous: fragment r, base at fragment 0, imm = r KB.
  // MN-contiguous: half h = r % 2 of fragment u = r / 2; within the swizzled
  // 16 x 32 blocks the lane's chunk depends on u % 2 (par) and on the lane,
  // while the block (u / 2) and the +4 rows of the second half are constant
  // offsets (rows k and k + 4 share their swizzle).
  auto read_base = [&](auto kc, auto cols, const uint16_t* st, int c0, int par) __attribute__((always_inline)) -> uint32_t {
    if constexpr (decltype(kc)::value) {
      return lds_addr(st + (c0 >> 4) * 512 + lane * 8);
    } else {
      const int j = lane & 15;
      const int k = 8 * (lane >> 4) + (j >> 2);
      return lds_addr(st + mn_lds_off<decltype(cols)::value>(k, c0 + 16 * par + 4 * (j & 3)));
    }
  };
  auto base_a = [&](const uint16_t* st, int par) __attribute__((always_inline)) {
    return read_base(std::integral_constant<bool, AK>{}, std::integral_constant<int, BM>{}, st, wm * WTM, par);
  };
  auto base_b = [&](const uint16_t* st, int par) __attribute__((always_inline)) {
    return read_base(std::integral_constant<bool, BKK>{}, std::integral_constant<int, BN>{}, st + BM * kBKb, wn * WTN, par);
  };
  // Read r of a stage's NRD fragment reads (per 32 K: A's, then B's) into (na, nb) or their pending halves.
  auto read_one = [&](auto rc, u32x4 (&na)[SUB * FM], u32x4 (&nb)[SUB * FN], uint32_t ra0, uint32_t ra1, uint32_t rb0,
                      uint32_t rb1) __attribute__((always_inline)) {
    constexpr int rd = decltype(rc)::value;
    constexpr int h = rd / NRH, r = rd % NRH, ho = h * HALF * 2;
    if constexpr (r < NRA) {
      constexpr int imm = wide_read_imm<AK, r>() + ho;
      if constexpr (AK) rd128_issue_at<imm>(na[h * FM + r], ra0);
      else rdtr_issue_at<imm>(qa[h * NRA + r], ((r >> 1) & 1) ? ra1 : ra0);
    } else {
      constexpr int rr = r - NRA;
      constexpr int imm = wide_read_imm<BKK, rr>() + ho;
      if constexpr (BKK) rd128_issue_at<imm>(nb[h * FN + rr], rb0);
      else rdtr_issue_at<imm>(qb[h * NRB + rr], ((rr >> 1) & 1) ? rb1 : rb0);
    }
    if constexpr (rd % 8 == 7 && rd + 1 < NRD) lds_wait_le<7>();
  };
  // Completes the reads: waits for them and joins the halves of MN-contiguous fragments.
  auto read_done = [&](u32x4 (&na)[SUB * FM], u32x4 (&nb)[SUB * FN]) __attribute__((always_inline)) {
    lds_wait_all();
    if constexpr (AK) {
      lds_mark(na);
    } else {
      lds_mark(qa);
#pragma unroll
      for (int u = 0; u < SUB * FM; ++u) na[u] = u32x4{qa[2 * u][0], qa[2 * u][1], qa[2 * u + 1][0], qa[2 * u + 1][1]};
      valu_to_mfma_fence(na);
    }
    if constexpr (BKK) {
      lds_mark(nb);
    } else {
      lds_mark(qb);
#pragma unroll
      for (int u = 0; u < SUB * FN; ++u) nb[u] = u32x4{qb[2 * u][0], qb[2 * u][1], qb[2 * u + 1][0], qb[2 * u + 1][1]};
      valu_to_mfma_fence(nb);
    }
  };

  // Prologue: fill the ring (PAIR: all but one stage, the slot the first
  // step refills), wait for the first stage, read its fragments.
#pragma unroll
  for (int s = 0; s < (PAIR ? STAGES - 1 : STAGES); ++s) {
    issue_stage();
    advance();
  }
  wait_vm_tiles<LPS, STAGES - 1>(ls - 1);
  lds_barrier();
  u32x4 fa0[SUB * FM], fb0[SUB * FN], fa1[SUB * FM], fb1[SUB * FN];
  {
    const uint32_t ra0 = base_a(lds, 0), ra1 = AK ? ra0 : base_a(lds, 1);
    const uint32_t rb0 = base_b(lds, 0), rb1 = BKK ? rb0 : base_b(lds, 1);
    __builtin_amdgcn_sched_barrier(0);
    static_for<0, NRD>([&](auto rc) __attribute__((always_inline)) { read_one(rc, fa0, fb0, ra0, ra1, rb0, rb1); });
    read_done(fa0, fb0);
  }
  zero_acc();

  // One K-step: the MFMAs of (ca, cb), with the next stage's fragment reads
  // into (na, nb) and the refill of this step's stage interleaved between
  // them one instruction at a time, so the wave keeps issuing MFMAs while the
  // memory operations queue.
  // MMA false: a wave whose rows of the tile are all past the group's last
  // row keeps its share of the loads and reads but issues no MFMAs, leaving
  // the matrix core to the other wave on its SIMD.
  auto step = [&](auto mmac, u32x4 (&ca)[SUB * FM], u32x4 (&cb)[SUB * FN], u32x4 (&na)[SUB * FM],
                  u32x4 (&nb)[SUB * FN]) __attribute__((always_inline)) {
    constexpr bool MMA = decltype(mmac)::value;
    const uint16_t* st = lds + ((unsigned)(cs + 1) % STAGES) * STAGE;
    // This step's refill: stage ls, K-step lk of the load cursor (issued
    // unconditionally; past the block's last load it writes zeros into the
    // ring slot of a K-step already consumed, which no later step reads).
    uint16_t* const dst = lds + ((unsigned)ls % STAGES) * STAGE;
    const bool live = loads_left();
    const int kdma = lk * SUB;
    __amdgpu_buffer_rsrc_t rsa[SUB], rsb[SUB];
#pragma unroll
    for (int h = 0; h < SUB; ++h) {
      rsa[h] = opA.rsrc(kdma + h, live);
      rsb[h] = opB.rsrc(kdma + h, live);
    }
    const bool more = cs + 1 < ls;
    auto sync = [&]() __attribute__((always_inline)) {
    if constexpr (PAIR) {
      // Even step: stages cs+1 and cs+2 have landed (at most stage cs+3 is
      // pending) and, after the barrier, are in LDS for every wave; every wave
      // is past step cs-1, so no wave reads the stages of K-steps cs-1 and cs
      // any more -- the refills of steps cs and cs+1 (ls <= cs+4 and ls+1:
      // ring slots of K-steps ls-5 <= cs-1 and cs).  Odd step: nothing to wait
      // for but this wave's epilogue stores.
      if ((cs & 1) == 0) {
        if (more) {
          if (stores_pending) {
            wait_vm<0>();
            stores_pending = false;
          } else {
            wait_vm_tiles<LPS, STAGES - 4>(ls - cs - 3);
          }
          lds_barrier();
        }
      } else if (stores_pending) {
        wait_vm<0>();
        stores_pending = false;
      }
    } else if (more) {
      if (stores_pending) {
        wait_vm<0>();
        stores_pending = false;
      } else {
        wait_vm_tiles<LPS, STAGES - 2>(ls - cs - 2);   // stage cs+1 has landed
      }
      lds_barrier();   // stage cs+1 is in LDS for every wave; no wave reads stage cs any more
    }
    };
    if constexpr (PRE == 0) sync();
    // The reads are unconditional (branch-free, so pending registers are never
    // copied); what they read after the last step is not used.
    const uint32_t ra0 = base_a(st, 0), ra1 = AK ? ra0 : base_a(st, 1);
    const uint32_t rb0 = base_b(st, 0), rb1 = BKK ? rb0 : base_b(st, 1);
    __builtin_amdgcn_sched_barrier(0);
    // Raised wave priority while this step's MFMAs after the barrier and the
    // reads issue: of the two waves on a SIMD, the one past the barrier keeps
    // the matrix core fed while the other waits (measured: FWD2 -3 %, the
    // layer step -1 %).  PRE MFMAs before the barrier issue at the low priority.
    if constexpr (PRE == 0) __builtin_amdgcn_s_setprio(1);
    static_for<0, NMF>([&](auto mc) __attribute__((always_inline)) {
      constexpr int m = decltype(mc)::value;
      if constexpr (PRE > 0 && m == PRE) {
        __builtin_amdgcn_sched_barrier(0);
        sync();
        __builtin_amdgcn_s_setprio(1);
        __builtin_amdgcn_sched_barrier(0);
      }
      if constexpr (MMA) {
        constexpr int h = m / NMH, i = m % NMH / FN, j = m % FN;
        mfma_acc(acc[i][j], cb[h * FN + j], ca[h * FM + i]);
      }
      static_for<0, NRD>([&](auto rc) __attribute__((always_inline)) {
        constexpr int r = decltype(rc)::value;
        if constexpr (m >= PRE && (r * RSPAN) / NRD == m - PRE) read_one(rc, na, nb, ra0, ra1, rb0, rb1);
      });
      // The step's refills: the ragged-K (dW) products spread them over the
      // MFMAs after the barrier; the others issue them at the last MFMA
      // slots, after the fragment reads (measured: the dX call -18 us, the
      // forward -7 us on the 16384-token layer; the dW products +5 % that way).
      static_for<0, NDMA>([&](auto dc) __attribute__((always_inline)) {
        constexpr int d = decltype(dc)::value;
        constexpr int slot = RAGGED_K ? std::min((d * (NMF - PRE)) / NDMA + 1 + PRE, NMF - 1)
                                      : std::max(NMF - NDMA - 1, PRE) + d;
        static_assert(slot >= PRE && slot < NMF, "refills follow the step's barrier");
        // A and B loads alternate; the larger operand's extra loads come last.
        constexpr int h = d / (NIA + NIB), dd = d % (NIA + NIB);
        constexpr int NP = 2 * (NIA < NIB ? NIA : NIB);
        constexpr bool isB = dd < NP ? (dd & 1) : NIB > NIA;
        constexpr int q = dd < NP ? dd >> 1 : dd - NP / 2;
        if constexpr (slot == m) {
          __builtin_amdgcn_sched_barrier(0);
          if constexpr (isB) opB.issue_r(q, rsb[h], kdma + h, dst + h * HALF + BM * kBKb, wid);
          else opA.issue_r(q, rsa[h], kdma + h, dst + h * HALF, wid);
          __builtin_amdgcn_sched_barrier(0);
        }
      });
    });
    __builtin_amdgcn_s_setprio(0);
    read_done(na, nb);
    __builtin_amdgcn_sched_barrier(0);
    if (more) advance();
    ++cs;
  };
  // Partial tile of a K-split remainder tile: stored to this block's slot in
  // accumulator order -- wave w, fragment (i, j), lane l at
  // ((w FM + i) FN + j) 64 + l -- for the fix-up kernel to add.
  // Fragment rows past the group's rows are not stored (the fix-up never
  // reads them).
  auto partial = [&](const WGeo& Cg) __attribute__((always_inline)) {
    asm volatile("s_nop 15\n s_nop 15" ::: "memory");   // last MFMA -> accumulator reads
    float* mine = p.part + (int64_t)blockIdx.x * (BMT * BN) + ((int64_t)wid * FM * FN * 64 + lane) * 4;
    const int rows = Cg.Mlim - (Cg.m0 + wm * WTM);   // the wave's rows in the group (uniform)
    // One fragment row at a time (the pin orders each row's register moves
    // after the previous row's stores, so only a row is ever out of AGPRs).
#pragma unroll
    for (int i = 0; i < FM; ++i) {
      acc_pin_mem(acc[i]);
      if (16 * i < rows) {
#pragma unroll
        for (int j = 0; j < FN; ++j) *reinterpret_cast<f32x4*>(mine + (i * FN + j) * 256) = acc[i][j];
      }
    }
  };

  auto run_steps_t = [&](int n, auto mmac) __attribute__((always_inline)) {
    int kk = 0;
    for (; kk + 2 <= n; kk += 2) {
      step(mmac, fa0, fb0, fa1, fb1);
      step(mmac, fa1, fb1, fa0, fb0);
    }
    if (kk < n) {   // odd step count: the next fragments are in set 1
      step(mmac, fa0, fb0, fa1, fb1);
#pragma unroll
      for (int u = 0; u < SUB * FM; ++u) fa0[u] = fa1[u];
#pragma unroll
      for (int u = 0; u < SUB * FN; ++u) fb0[u] = fb1[u];
      valu_to_mfma_fence(fa0);
      valu_to_mfma_fence(fb0);
    }
  };
  auto run_steps = [&](int n, bool mma) __attribute__((always_inline)) {
    if (mma) run_steps_t(n, std::true_type{});
    else run_steps_t(n, std::false_type{});
  };
  for (int e = 0; e < nseg; ++e) {
    int ct, k0, k1;
    seg(e, ct, k0, k1);
    const WGeo Cg = geo(ct);
    // Ragged-M: does the wave hold any of the group's rows in this tile?
    const bool mma = RAGGED_K || __builtin_amdgcn_readfirstlane((int)(Cg.m0 + wm * WTM < Cg.Mlim));
    if constexpr (SPLIT) {
      run_steps(e < nd ? Cg.nk : k1 - k0, mma);
      if (e < nd) epilogue(Cg);
      else partial(Cg);
    } else {
      run_steps(Cg.nk, mma);
      epilogue(Cg);
    }
    zero_acc();
    stores_pending = true;
  }
  wait_vm<0>();
}

// Adds the partial sums of the K-split remainder tiles -- in block order, so
// the result does not depend on timing -- and applies the epilogue.  Block b
// takes fragment row i = (b / 8) % FM of remainder tile (b / 8) / FM of XCD
// b % 8 (both waves rows of the tile's 2 x WGN wave grid), so a tile's sum is
// spread over FM blocks.  The schedule is recomputed exactly as the product
// made it (nslot blocks per XCD).
template <class TC, int EPI, int ACT, bool CBLK>
__global__ __launch_bounds__(TC::NW * 64) void gemm_wide_fixup_kernel(GemmParams p, int tilesM, int tilesN, int groups,
                                                                   int nslot) {
  constexpr int BM = TC::BMT, BN = TC::BN, WGN = TC::WGN, WTM = TC::WTM, WTN = TC::WTN, FM = TC::FM, FN = TC::FN;
  const int lane = threadIdx.x & 63;
  const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wid / WGN, wn = wid % WGN;
  const WPrefix P = wide_tile_prefix<BM, false, true>(p, lane, groups, tilesM, tilesN);
  const int xcd = blockIdx.x % 8, q = (blockIdx.x / 8) / FM, i = (blockIdx.x / 8) % FM;
  const WRange XR = wide_range(P, xcd);
  const int nkU = (p.K + TC::BK - 1) / TC::BK;
  const WSched W = wide_sched(XR.nf + XR.np, nslot, p.ksplit != 0);
  if (!W.split || q >= W.r) return;
  const WGeo G = wide_geo<BM, BN, TC::BK, false, true>(p, XR.tile(W.R * nslot + q), lane, groups, P, tilesM, tilesN);
  // fragment row i of the wave's rows: nothing to add past the group's rows
  const bool live = 16 * i < G.Mlim - (G.m0 + wm * WTM);
  // the blocks of remainder tile q: [first, first + cnt); an empty K range wrote nothing
  int q0, first, cnt, k0, k1;
  W.split_part((q * nslot + W.r - 1) / W.r, nslot, nkU, q0, first, cnt, k0, k1);
  const int64_t lane_off = ((int64_t)wid * FM * FN * 64 + lane) * 4 + (int64_t)i * FN * 256;
  f32x4 sum[FN];
  bool any = false;
  for (int sl = first; sl < first + cnt; ++sl) {
    int qq, ff, cc, a0, a1;
    W.split_part(sl, nslot, nkU, qq, ff, cc, a0, a1);
    if (a0 >= a1 || !live) continue;
    const float* src = p.part + (int64_t)(sl * 8 + xcd) * (BM * BN) + lane_off;
    f32x4 v[FN];
#pragma unroll
    for (int j = 0; j < FN; ++j) v[j] = *reinterpret_cast<const f32x4*>(src + j * 256);
#pragma unroll
    for (int j = 0; j < FN; ++j) sum[j] = any ? sum[j] + v[j] : v[j];
    any = true;
  }
  if (!any) {   // rows past the group, or an empty K range everywhere: nothing stored
#pragma unroll
    for (int j = 0; j < FN; ++j) sum[j] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  f32x4 acc[FM][FN];
  static_for<0, FM>([&](auto ic) {   // row i of acc (compile-time index), the others unused
    constexpr int I = decltype(ic)::value;
    if (I == i) {
#pragma unroll
      for (int j = 0; j < FN; ++j) acc[I][j] = sum[j];
      wide_epilogue<FM, FN, WTM, WTN, false, EPI, ACT, CBLK>(p, G, acc, wm, wn, lane, I, I + 1);
    }
  });
}


// --------------------------------------------------------------- launchers
// A product of the wide kernel: its operand orders and epilogue.
enum WideKind {
  WK_FWD1,      // B [N][K], (H, act(H)) epilogue, blocked outputs
  WK_NK,        // B [N][K], plain store, row-major output
  WK_NK_RES,    // the same with a residual added
  WK_DACT,      // B [K][N], dA * act'(H) epilogue, blocked output
  WK_KN,        // B [K][N], plain store, row-major output
  WK_DW,        // (this kind and the later ones) ragged-K, row-major output
  WK_DW_BLK,    // ragged-K, blocked output
  WK_WGF32      // ragged-K over row-major operands, float partials
};
struct WideCall {
  WideKind kind;
  int act;
  int groups;
  int64_t rows;   // rows of the output per group (ragged-M: the capacity; ragged-K: M)
  int cols;       // N
  double expect;  // rows a group is expected to hold (WK_WGF32: its K), and their
  double spread;  // standard deviation (hints for the tile choice)
  GemmParams p;
  bool beside = false;   // ragged-K: other work runs beside it on another stream
};

constexpr int64_t kSkPartElems = (int64_t)256 * 256 * 256;   // floats of the K-split's partial tiles (one per block)

template <class TC, bool B_K, bool RAGGED_K, int EPI, int ACT, bool CBLK>
static void launch_wide(const WideCall& w, hipStream_t s) {
  constexpr size_t shmem = TC::lds_bytes(B_K);
  constexpr bool SPLIT = TC::KSPLIT && !RAGGED_K && EPI == EPI_STORE;
  const GemmParams& p = w.p;
  auto kern = gemm_wide_kernel<TC, B_K, RAGGED_K, EPI, ACT, CBLK>;
  static std::atomic<uint64_t> lds_ok{0};
  allow_dyn_lds((const void*)kern, (int)shmem, lds_ok);
  const int tm = (int)((w.rows + (RAGGED_K ? 0 : 15) + TC::BMT - 1) / TC::BMT), tn = (w.cols + TC::BN - 1) / TC::BN;
  int64_t blocks = (int64_t)num_cus() * TC::per_cu(B_K);
  if (SPLIT) blocks = std::min<int64_t>(blocks, kSkPartElems / (TC::BMT * TC::BN));   // partial tiles in the workspace
  blocks = std::min(blocks, (int64_t)tm * tn * w.groups);
  blocks = (blocks + 7) / 8 * 8;
  hipLaunchKernelGGL(kern, dim3((unsigned)blocks), dim3(TC::NW * 64), shmem, s, p, tm, tn, w.groups);
  if constexpr (SPLIT) {
    const int nslot = (int)blocks / 8;   // a K-split last round has at most nslot / 4 tiles per XCD
    if (nslot >= 4 && p.ksplit)
      hipLaunchKernelGGL((gemm_wide_fixup_kernel<TC, EPI, ACT, CBLK>), dim3((unsigned)(8 * (nslot / 4) * TC::FM)),
                         dim3(TC::NW * 64), 0, s, p, tm, tn, w.groups, nslot);
  }
}

template <class TC, bool B_K, int EPI>
static void launch_wide_act(const WideCall& w, hipStream_t s) {
  switch (w.act) {
    case MOE_ACT_RELU: return launch_wide<TC, B_K, false, EPI, MOE_ACT_RELU, true>(w, s);
    case MOE_ACT_GELU_TANH: return launch_wide<TC, B_K, false, EPI, MOE_ACT_GELU_TANH, true>(w, s);
    case MOE_ACT_GELU_ERF: return launch_wide<TC, B_K, false, EPI, MOE_ACT_GELU_ERF, true>(w, s);
    default: return launch_wide<TC, B_K, false, EPI, MOE_ACT_IDENTITY, true>(w, s);
  }
}

// Ragged-M kinds on tile shape TC; ragged-K kinds on TCK.
template <class TC>
static void run_wide_m(const WideCall& w, hipStream_t s) {
  constexpr int ID = MOE_ACT_IDENTITY;
  switch (w.kind) {
    case WK_FWD1: return launch_wide_act<TC, true, EPI_FWD1>(w, s);
    case WK_NK: return launch_wide<TC, true, false, EPI_STORE, ID, false>(w, s);
    case WK_NK_RES: return launch_wide<TC, true, false, EPI_RES, ID, false>(w, s);
    case WK_DACT: return launch_wide_act<TC, false, EPI_DACT>(w, s);
    case WK_KN: return launch_wide<TC, false, false, EPI_STORE, ID, false>(w, s);
    default: return;
  }
}
template <class TCK>
static void run_wide_k(const WideCall& w, hipStream_t s) {
  constexpr int ID = MOE_ACT_IDENTITY;
  switch (w.kind) {
    case WK_DW: return launch_wide<TCK, false, true, EPI_STORE, ID, false>(w, s);
    case WK_DW_BLK: return launch_wide<TCK, false, true, EPI_STORE, ID, true>(w, s);
    case WK_WGF32: return launch_wide<TCK, false, true, EPI_WGF32, ID, false>(w, s);
    default: return;
  }
}

// One source file per tile shape (they compile in parallel).
void run_wide_256x256(const WideCall& w, hipStream_t s);
void run_wide_192x256(const WideCall& w, hipStream_t s);  // ragged-M products only
void run_wide_128x128(const WideCall& w, hipStream_t s);
void run_wide_64x128(const WideCall& w, hipStream_t s);   // ragged-M products only
void run_wide_64x64(const WideCall& w, hipStream_t s);    // ragged-M products only

}  // namespace lmoe
