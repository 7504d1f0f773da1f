// The wide bf16 kernel on 64 x 128 tiles (see gemm.hip for when it is chosen).
#include "gemm_wide.h"

namespace lmoe {

// 64 of K per step: with 8 MFMAs per wave and 32 K, a step is mostly LDS
// latency, barrier and scalar work, so two K halves share one (expert_out of
// 1531 tokens, d_model 768, 8 experts: 32 -> 26 us; a step of 32 K with more
// stages or one barrier per two steps measured no faster).
using Tile = Wide<64, 128, 4, 2, 2, 3, 3, 2, false>;

void run_wide_64x128(const WideCall& w, hipStream_t s) { run_wide_m<Tile>(w, s); }

}  // namespace lmoe
