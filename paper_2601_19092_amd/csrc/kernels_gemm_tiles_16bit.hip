// The small and medium tiles of gemm_tiles.h with 16-bit inputs.
#include "gemm_tiles.h"

namespace axe {

hipError_t launch_gemm_tiles_16bit(int member, const GemmArgs& g, hipStream_t s) {
  return g.f16 ? tiles::launch_family<1, 0>(member, g, s) : tiles::launch_family<0, 0>(member, g, s);
}

}  // namespace axe
