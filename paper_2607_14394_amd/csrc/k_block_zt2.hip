// Instances of the fused inverse + block epilogue kernel with two column
// tiles (8 < K_t <= 16), t not folded.
#include "block_zt.h"

namespace dtst {

const void* block_zt_kernel2(int th, int t32, int zp, int mt, int ncls, int kio) {
  if (th == 1) return zp == 2 ? pick_mn<2, 1, 0, 0, 2>(mt, ncls, kio) : pick_mn<2, 1, 0, 0>(mt, ncls, kio);
  return t32 ? pick_mn<2, 2, 0, 1>(mt, ncls, kio) : pick_mn<2, 2, 0, 0>(mt, ncls, kio);
}

}  // namespace dtst
