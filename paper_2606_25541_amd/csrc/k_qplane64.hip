// FP64 quarter-plane kernels of the operator apply (see qplane.hpp).
#include "qplane.hpp"

namespace psfd {

template void launch_qplane<double2, false, LD_VX, ST_PLAIN>(const TileArgs&, int, int, hipStream_t);
template void launch_qplane<double2, false, LD_VX_GIV, ST_PLAIN>(const TileArgs&, int, int, hipStream_t);
template void launch_qplane<double2, true, LD_PLAIN, ST_PLAIN>(const TileArgs&, int, int, hipStream_t);
template void launch_qplane<double2, true, LD_PLAIN, ST_AXPBY>(const TileArgs&, int, int, hipStream_t);

}  // namespace psfd
