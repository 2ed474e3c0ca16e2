// Instantiations of the tile kernels (lbm_tile.hpp).
#include <hip/hip_runtime.h>

#include "lbm_tile.hpp"

namespace lbmk {

template <int BC>
static void fill_bc(TileTable& t) {
  t.fn[0][0][BC] = &k_tile<BC, true, false, 16, tile_max_waves(0)>;
  t.fn[0][1][BC] = &k_tile<BC, true, false, 32, tile_max_waves(0)>;
  t.fn[1][0][BC] = t.fn[1][1][BC] = &k_tile<BC, false, true, 16, tile_max_waves(1)>;
  t.fn[2][0][BC] = &k_tile<BC, true, true, 16, tile_max_waves(2)>;
  t.fn[2][1][BC] = &k_tile<BC, true, true, 32, tile_max_waves(2)>;
  t.fn[3][0][BC] = t.fn[3][1][BC] = &k_tile<BC, false, false, 16, tile_max_waves(3)>;
}

void tile_fill(TileTable& t) {
  fill_bc<LBM_PERIODIC>(t);
  fill_bc<LBM_DIRICHLET>(t);
}

}  // namespace lbmk
