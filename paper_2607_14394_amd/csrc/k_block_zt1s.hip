// Instances of the fused inverse + block epilogue kernel with one column tile
// (K_t <= 8) and one t group (N_t <= 16).
#include "block_zt.h"

namespace dtst {

const void* block_zt_kernel1s(int zp, int mt, int ncls, int kio) {
  if (zp == 4) return pick_mn<1, 1, 0, 0, 4>(mt, ncls, kio);
  return zp == 2 ? pick_mn<1, 1, 0, 0, 2>(mt, ncls, kio) : pick_mn<1, 1, 0, 0>(mt, ncls, kio);
}

}  // namespace dtst
