// k_tile_reg and k_tile_reg_batch in single precision, default shape.
#include "tile_reg.hpp"

namespace qsv {
namespace dev {

hipError_t tile_reg_f32(void *psi, const TileArgs &ta, const RegOp *rops, const void *pool,
                        unsigned int *counter, hipStream_t s) {
    QSV_TILE_REG(float, 4, 8)
}

hipError_t tile_reg_batch_f32(int dg, void *states, const RegSeg *segs, int nseg, uint64_t items,
                              const TileArgs *tas, const RegOp *rops, const void *pool,
                              uint32_t img_max, hipStream_t s) {
    return dg == 0   ? launch_reg_batch_t<float, 0>(states, segs, nseg, items, tas, rops, pool, img_max, s)
           : dg == 1 ? launch_reg_batch_t<float, 1>(states, segs, nseg, items, tas, rops, pool, img_max, s)
                     : launch_reg_batch_t<float, 2>(states, segs, nseg, items, tas, rops, pool, img_max, s);
}

}  // namespace dev
}  // namespace qsv
