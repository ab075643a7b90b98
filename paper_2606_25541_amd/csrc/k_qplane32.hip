// FP32 quarter-plane kernels of the operator apply (see qplane.hpp).
#include "qplane.hpp"

namespace psfd {

template void launch_qplane<float2, false, LD_VX, ST_PLAIN>(const TileArgs&, int, int, hipStream_t);
template void launch_qplane<float2, false, LD_VX_GIV, ST_PLAIN>(const TileArgs&, int, int, hipStream_t);
template void launch_qplane<float2, true, LD_PLAIN, ST_PLAIN>(const TileArgs&, int, int, hipStream_t);
template void launch_qplane<float2, true, LD_PLAIN, ST_AXPBY>(const TileArgs&, int, int, hipStream_t);

// 16 columns per pencil block, 8 at nz = 128 (16 would exceed a block's
// threads). 16 is faster everywhere else, also where 8 would fill more CUs:
// 32 x 32 x 32 FP64 apply 16.1 against 16.3 us, 64 x 64 x 32 FP32 19.2 against
// 20.7, 128 x 32 x 64 FP32 22.0 against 25.8, and, with the blocks that share the
// layout's 128-byte lines on one XCD, 128 x 128 x 64 FP32 52.2 against 59.5 and
// FP64 93.1 against 97.2 (the fixed work of a block is shared by twice the
// columns, and 8 columns take more than 80 registers: fewer resident wavefronts).
int qplane_bx(int nx, int ny, int nz, size_t esz) {
  if (!qplane_fits(ilog2i(nx), ilog2i(ny), esz) || nz < 8 || nz > 128) return 0;
  return nz == 128 ? 8 : 16;
}

}  // namespace psfd
