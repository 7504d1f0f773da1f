// The wide bf16 kernel on 192 x 256 tiles (see gemm.hip for when it is chosen).
#include "gemm_wide.h"

namespace lmoe {

// The 256 x 256 kernel with a quarter of the rows left out of the tile (the LDS
// stage keeps its layout, and the loads of the left-out rows are issued and bring
// zeros): for row counts that end just past a multiple of 256.
using Tile = Wide<256, 256, 8, 4, 1, 4, 5, 2, false, 192>;

void run_wide_192x256(const WideCall& w, hipStream_t s) { run_wide_m<Tile>(w, s); }

}  // namespace lmoe
