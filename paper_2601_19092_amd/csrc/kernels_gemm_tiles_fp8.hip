// The small and medium tiles of gemm_tiles.h with fp8 inputs: unscaled, with fp32 scales, with E8M0 codes.
#include "gemm_tiles.h"

namespace axe {

hipError_t launch_gemm_tiles_fp8(int member, const GemmArgs& g, hipStream_t s) {
  if (!g.scale_a) return tiles::launch_family<2, 0>(member, g, s);
  return g.scale_e8m0 ? tiles::launch_family<2, 2>(member, g, s) : tiles::launch_family<2, 1>(member, g, s);
}

}  // namespace axe
