// rfa_pair_4x1.hip -- two-step kernel, 4 waves of 1 voxel per lane, nz <= 96.
#include "rfa_pair_kernel.h"

namespace rfa {

RFA_PAIR_LAUNCH(launch_pair_4x1) {
  return launch_store<256, 1, 96>(s, g, b, K, mode, hi_mid, store, st);
}

}  // namespace rfa
