// FP32 quarter-plane kernels of an Arnoldi step that carry its Gram-Schmidt work:
// forward with the update of the previous column, inverse with the projections of
// the new vector (see qplane.hpp).
#include "qplane.hpp"

namespace psfd {

template void launch_qplane<float2, false, LD_UPD_VX, ST_PLAIN>(const TileArgs&, int, int, hipStream_t);
template void launch_qplane<float2, false, LD_UPD_SLOT, ST_PLAIN>(const TileArgs&, int, int, hipStream_t);
template void launch_qplane<float2, true, LD_PLAIN, ST_DOTS>(const TileArgs&, int, int, hipStream_t);

bool qplane_gs(int nx, int ny, int nz, size_t esz) {
  return qplane_bx(nx, ny, nz, esz) != 0 && qplane_gs_fits(ilog2i(nx), ilog2i(ny), esz) && nz <= 64;
}

}  // namespace psfd
