// The wide bf16 kernel on 128 x 128 tiles (see gemm.hip for when it is chosen).
#include "gemm_wide.h"

namespace lmoe {

// Ragged-M: two blocks per CU.  Ragged-K: three stages and three blocks per CU
// (its tiles are short and end in a store; a third block covers the drain:
// dW of 2048 tokens, d_model 768, 8 experts 38 -> 32 us, of 3108 tokens 49 -> 44).
using Tile = Wide<128, 128, 4, 2, 1, 4, 4, 2, false>;
using TileK = Wide<128, 128, 4, 2, 1, 3, 3, 3, false>;

void run_wide_128x128(const WideCall& w, hipStream_t s) {
  if (w.kind < WK_DW) run_wide_m<Tile>(w, s);
  else run_wide_k<TileK>(w, s);
}

}  // namespace lmoe
