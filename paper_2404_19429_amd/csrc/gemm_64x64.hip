// The wide bf16 kernel on 64 x 64 tiles (see gemm.hip for when it is chosen).
#include "gemm_wide.h"

namespace lmoe {

using Tile = Wide<64, 64, 4, 2, 2, 4, 4, 2, false>;

void run_wide_64x64(const WideCall& w, hipStream_t s) { run_wide_m<Tile>(w, s); }

}  // namespace lmoe
