// k_tile_reg in double precision, the shapes other than the default.
#include "tile_reg.hpp"

namespace qsv {
namespace dev {

hipError_t tile_reg_shapes_f64(void *psi, const TileArgs &ta, const RegOp *rops, const void *pool,
                               unsigned int *counter, hipStream_t s) {
    const int rb = ta.rb, tb = ta.m - ta.rb;
    if (tb == 8 && rb == 3) { QSV_TILE_REG(double, 3, 8) }
    if (tb == 8 && rb == 5) { QSV_TILE_REG(double, 5, 8) }
    if (tb == 9 && rb == 3) { QSV_TILE_REG(double, 3, 9) }
    if (tb == 9 && rb == 4) { QSV_TILE_REG(double, 4, 9) }
    return hipErrorInvalidValue;
}

}  // namespace dev
}  // namespace qsv
