// Instances of the fused inverse + block epilogue kernel with one column tile
// (K_t <= 8) and N_t = 32.
#include "block_zt.h"

namespace dtst {

const void* block_zt_kernel1(int mt, int ncls, int kio) { return pick_mn<1, 2, 0, 1>(mt, ncls, kio); }

}  // namespace dtst
