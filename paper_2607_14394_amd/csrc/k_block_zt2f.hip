// Instances of the fused inverse + block epilogue kernel with two column
// tiles (8 < K_t <= 16), t folded.
#include "block_zt.h"

namespace dtst {

const void* block_zt_kernel2f(int t32, int mt, int ncls, int kio) {
  return t32 ? pick_mn<2, 2, 1, 1>(mt, ncls, kio) : pick_mn<2, 2, 1, 0>(mt, ncls, kio);
}

}  // namespace dtst
