// Top-k gate: logits = x Wg^T (+ bias), top-k selection and combine weights.
//
// The logits are a skinny product (tokens x E, E <= 64) computed on the fp64
// matrix cores: a block owns 16 * MT tokens and every expert, as MT x NT tiles
// of 16 x 16 doubles (v_mfma_f64_16x16x4).  Its NWV waves split d into
// interleaved chunks and meet in LDS, summing in wave order.  Because bf16 x bf16 (and
// f32 x f32) products are exact in double and the double sum is far more
// precise than float, the emitted float logit is the correctly rounded dot
// product except when the exact value lies within ~1e-15 relative of a float
// rounding boundary.  The top-k decision is taken on these float logits, so it
// matches any other evaluation that rounds the same values the same way.
//
// Operand mapping of one 16-byte load per lane: lane (i = lane & 15,
// q = lane >> 4) loads V consecutive elements of row i (a token of x, or an
// expert of Wg) at column 4V*c + V*q of the piece; MFMA j of chunk c then
// takes element j.  The product's k-index q therefore stands for the same
// column in both operands, which is all a dot product needs.
#include "internal.h"

namespace lmoe {

typedef double f64x4 __attribute__((ext_vector_type(4)));

// Order-preserving map of a float to uint32 (-0 treated as +0).
__device__ __forceinline__ uint32_t float_order_key(float f) {
  uint32_t u = __float_as_uint(f);
  if (u == 0x80000000u) u = 0u;
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
__device__ __forceinline__ float float_from_order_key(uint32_t o) {
  uint32_t u = (o & 0x80000000u) ? (o & 0x7fffffffu) : ~o;
  return __uint_as_float(u);
}

// Element j of a 16-byte vector as a double.
template <typename T> __device__ __forceinline__ double elem_f64(const u32x4& v, int j);
template <> __device__ __forceinline__ double elem_f64<uint16_t>(const u32x4& v, int j) {
  const uint32_t w = v[j >> 1];
  return (double)__uint_as_float((j & 1) ? (w & 0xffff0000u) : (w << 16));
}
template <> __device__ __forceinline__ double elem_f64<float>(const u32x4& v, int j) {
  return (double)__uint_as_float(v[j]);
}

constexpr int kGateGroup = 4;   // chunks whose loads are in flight together

template <typename T, int MT, int NT, int NWV, int KT>
__global__ __launch_bounds__(64 * NWV) void gate_topk_kernel(const T* __restrict__ x, const T* __restrict__ Wg,
                                                            const float* __restrict__ bias,
                                                            float* __restrict__ logits, int32_t* __restrict__ idx,
                                                            float* __restrict__ wout, int64_t T_tokens, int d,
                                                            int E, int k, int renorm) {
  constexpr int V = Vec<T>::N;          // elements per 16-byte load
  constexpr int CW = 4 * V;             // columns per chunk (four lane groups)
  constexpr int TM = 16 * MT;           // tokens per block
  __shared__ double red[NWV][MT * NT * 4 * kWave];
  __shared__ float lg[TM][kMaxE + 1];

  const int lane = threadIdx.x & 63;
  const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int i16 = lane & 15, q = lane >> 4;
  const int64_t t0 = (int64_t)blockIdx.x * TM;

  const T* xr[MT];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) {
    int64_t t = t0 + mt * 16 + i16;
    if (t >= T_tokens) t = T_tokens - 1;  // rows past the end are computed and discarded
    xr[mt] = x + t * d;
  }
  const T* wr[NT];
  bool wok[NT];
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) {
    const int e = nt * 16 + i16;
    wok[nt] = e < E;
    wr[nt] = Wg + (int64_t)(wok[nt] ? e : 0) * d;
  }

  f64x4 acc[MT][NT];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) acc[mt][nt] = f64x4{0.0, 0.0, 0.0, 0.0};

  // Wave wid takes chunks wid, wid + NWV, ...; kGateGroup of them per round,
  // loads first (unconditional, from a clamped column; masked after), then
  // the products, so the waits can retire one chunk at a time.
  const int nchunks = (d + CW - 1) / CW;
  for (int c0 = wid; c0 < nchunks; c0 += NWV * kGateGroup) {
    u32x4 xv[kGateGroup][MT], wv[kGateGroup][NT];
    bool ok[kGateGroup];
#pragma unroll
    for (int g = 0; g < kGateGroup; ++g) {
      const int col = (c0 + g * NWV) * CW + q * V;
      ok[g] = col < d;   // d is a multiple of V: a load is wholly inside or outside
      const int colc = ok[g] ? col : 0;
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) xv[g][mt] = *reinterpret_cast<const u32x4*>(xr[mt] + colc);
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) wv[g][nt] = *reinterpret_cast<const u32x4*>(wr[nt] + colc);
    }
    __builtin_amdgcn_sched_barrier(0);   // keep every load of the round ahead of the products
#pragma unroll
    for (int g = 0; g < kGateGroup; ++g) {
#pragma unroll
      for (int nt = 0; nt < NT; ++nt)
        if (!ok[g] || !wok[nt]) wv[g][nt] = u32x4{0u, 0u, 0u, 0u};
#pragma unroll
      for (int j = 0; j < V; ++j) {
        double a[MT], b[NT];
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) a[mt] = elem_f64<T>(xv[g][mt], j);
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) b[nt] = elem_f64<T>(wv[g][nt], j);
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
          for (int nt = 0; nt < NT; ++nt)
            acc[mt][nt] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[mt], b[nt], acc[mt][nt], 0, 0, 0);
      }
    }
  }

  // Wave sums meet in LDS and are added in wave order, every thread its share.
  // Accumulator element r of a lane holds row q + 4r, column i16 of its 16 x 16
  // tile: token mt*16 + q + 4r, expert nt*16 + i16.
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
      for (int r = 0; r < 4; ++r) red[wid][((mt * NT + nt) * 4 + r) * kWave + lane] = acc[mt][nt][r];
  __syncthreads();
  for (int o = threadIdx.x; o < MT * NT * 4 * kWave; o += 64 * NWV) {
    const int l = o & 63, r = (o >> 6) & 3, t = o >> 8;
    const int e = (t % NT) * 16 + (l & 15);
    if (e >= E) continue;
    double s = red[0][o];
#pragma unroll
    for (int w = 1; w < NWV; ++w) s += red[w][o];
    lg[(t / NT) * 16 + (l >> 4) + 4 * r][e] = (float)(s + (bias ? (double)bias[e] : 0.0));
  }
  __syncthreads();

  // Logits out: the block's rows are one contiguous run of [T][E].
  const int64_t ntok = (T_tokens - t0) < TM ? (T_tokens - t0) : TM;
  for (int i = threadIdx.x; i < ntok * E; i += blockDim.x) logits[t0 * E + i] = lg[i / E][i % E];

  // Top-k by (logit desc, expert asc): four lanes per token scan every fourth
  // expert into sorted lists of KT keys (distinct: the expert is part of the
  // key), which two exchanges merge, so each lane ends with the token's list.  Of
  // two sorted lists the larger of best[r] and other[KT - 1 - r] are the KT largest
  // keys, falling and then rising, which log2 KT rounds of exchanges sort: 20
  // comparisons for KT = 8 where inserting one by one takes 64 (1000 tokens, d 256,
  // 8 experts, k = 8 8.4 -> 6.9 us; k = 1 and 2 are the same).
  const int tl = threadIdx.x >> 2, l4 = threadIdx.x & 3;
  if (tl < ntok) {
    uint64_t best[KT];
#pragma unroll
    for (int r = 0; r < KT; ++r) best[r] = 0ull;
    auto insert = [&](uint64_t key) __attribute__((always_inline)) {
#pragma unroll
      for (int r = 0; r < KT; ++r) {
        const uint64_t hi = key > best[r] ? key : best[r];
        key = key > best[r] ? best[r] : key;
        best[r] = hi;
      }
    };
    for (int e = l4; e < E; e += 4)
      insert(((uint64_t)float_order_key(lg[tl][e]) << 32) | (uint64_t)(0xffffffffu - (uint32_t)e));
#pragma unroll
    for (int o = 1; o <= 2; o <<= 1) {
      uint64_t other[KT];
#pragma unroll
      for (int r = 0; r < KT; ++r) other[r] = __shfl_xor(best[r], o, kWave);
#pragma unroll
      for (int r = 0; r < KT; ++r) best[r] = best[r] > other[KT - 1 - r] ? best[r] : other[KT - 1 - r];
#pragma unroll
      for (int h = KT / 2; h > 0; h >>= 1)
#pragma unroll
        for (int r = 0; r < KT; ++r)
          if ((r & h) == 0) {
            const uint64_t lo = best[r] < best[r + h] ? best[r] : best[r + h];
            best[r] = best[r] < best[r + h] ? best[r + h] : best[r];
            best[r + h] = lo;
          }
    }
    const float m = float_from_order_key((uint32_t)(best[0] >> 32));
    float ex[KT], denom = 0.f;
#pragma unroll
    for (int r = 0; r < KT; ++r) {
      ex[r] = expf(float_from_order_key((uint32_t)(best[r] >> 32)) - m);
      if (r < k) denom += ex[r];
    }
    if (!renorm) {
      denom = 0.f;
      for (int e = l4; e < E; e += 4) denom += expf(lg[tl][e] - m);
      denom += __shfl_xor(denom, 1, kWave);
      denom += __shfl_xor(denom, 2, kWave);
    }
    const int64_t t = t0 + tl;
#pragma unroll
    for (int r = 0; r < KT; ++r) {
      if (r < k && (r & 3) == l4) {
        idx[t * k + r] = (int)(0xffffffffu - (uint32_t)(best[r] & 0xffffffffu));
        wout[t * k + r] = ex[r] / denom;
      }
    }
  }
}

template <typename T, int MT, int NT, int NWV, int KT>
static void launch_gate_k(const moe_cfg& c, const void* x, const void* Wg, const float* bias, float* logits,
                          int32_t* idx, float* w, hipStream_t s) {
  const int64_t blocks = (c.T + 16 * MT - 1) / (16 * MT);
  hipLaunchKernelGGL((gate_topk_kernel<T, MT, NT, NWV, KT>), dim3((unsigned)blocks), dim3(64 * NWV), 0, s,
                     (const T*)x, (const T*)Wg, bias, logits, idx, w, c.T, c.d_model, c.E, c.k, c.renorm);
}
// 32 tokens per block; 16 where that gives the CUs at most three blocks each (the
// kernel is then latency: loads, a short MFMA chain, the sums, the selection).
// One MI355X, with the wave sums spread over the block and four lanes per token
// selecting (before: one wave summing, one lane per token with a list of eight):
// 2048 tokens, d 768, 8 experts 11.3 -> 6.2 us; 8192 tokens, d 1024, 32 experts
// 22.5 -> 16.3; 32768 tokens, 64 experts 123 -> 101; 16384 tokens, d 2048, 8
// experts 28.6 -> 28.0 (fp64 matrix rate).  The line, 16- against 32-token blocks:
// 12000 tokens, d 4096, float, 24 experts 67 and 81 us, 64 experts 140 and 158; of
// 16000 tokens, where both are whole rounds and the smaller block reads Wg twice
// as often, 88 and 79, 187 and 160 (bf16 164 and 153).
template <typename T, int NT, int NWV, int KT>
static void launch_gate_m(const moe_cfg& c, const void* x, const void* Wg, const float* bias, float* logits,
                          int32_t* idx, float* w, hipStream_t s) {
  if (c.T <= (int64_t)16 * 3 * num_cus()) launch_gate_k<T, 1, NT, NWV, KT>(c, x, Wg, bias, logits, idx, w, s);
  else launch_gate_k<T, 2, NT, NWV, KT>(c, x, Wg, bias, logits, idx, w, s);
}
// KT: the top-k list's length, k rounded up to 1, 2, 4 or 8.
template <typename T, int NT, int NWV>
static void launch_gate_e(const moe_cfg& c, const void* x, const void* Wg, const float* bias, float* logits,
                          int32_t* idx, float* w, hipStream_t s) {
  if (c.k == 1) launch_gate_m<T, NT, NWV, 1>(c, x, Wg, bias, logits, idx, w, s);
  else if (c.k == 2) launch_gate_m<T, NT, NWV, 2>(c, x, Wg, bias, logits, idx, w, s);
  else if (c.k <= 4) launch_gate_m<T, NT, NWV, 4>(c, x, Wg, bias, logits, idx, w, s);
  else launch_gate_m<T, NT, NWV, 8>(c, x, Wg, bias, logits, idx, w, s);
}

// d is split over 8 waves (4 when four expert tiles already give each wave
// independent accumulators and more registers).
template <typename T>
static void launch_gate_t(const moe_cfg& c, const void* x, const void* Wg, const float* bias, float* logits,
                          int32_t* idx, float* w, hipStream_t s) {
  if (c.E <= 16) launch_gate_e<T, 1, 8>(c, x, Wg, bias, logits, idx, w, s);
  else if (c.E <= 32) launch_gate_e<T, 2, 8>(c, x, Wg, bias, logits, idx, w, s);
  else if (c.E <= 48) launch_gate_e<T, 3, 4>(c, x, Wg, bias, logits, idx, w, s);
  else launch_gate_e<T, 4, 4>(c, x, Wg, bias, logits, idx, w, s);
}

void launch_gate(const moe_cfg& c, const void* x, const void* Wg, const float* bias, float* logits,
                 int32_t* idx, float* w, hipStream_t s) {
  if (c.T == 0) return;
  if (c.dtype == MOE_BF16) launch_gate_t<uint16_t>(c, x, Wg, bias, logits, idx, w, s);
  else launch_gate_t<float>(c, x, Wg, bias, logits, idx, w, s);
}

}  // namespace lmoe
