// The wide bf16 kernel on 256 x 256 tiles (see gemm.hip for when it is chosen).
#include "gemm_wide.h"

namespace lmoe {

using Tile = Wide<256, 256, 8, 4, 1, 4, 5, 2, true>;

void run_wide_256x256(const WideCall& w, hipStream_t s) {
  if (w.kind < WK_DW) run_wide_m<Tile>(w, s);
  else run_wide_k<Tile>(w, s);
}

}  // namespace lmoe
