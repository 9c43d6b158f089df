// rfa_pair_16x2.hip -- two-step kernel, 16 waves of 2 voxels per lane, nz <= 256.
#include "rfa_pair_kernel.h"

namespace rfa {

RFA_PAIR_LAUNCH(launch_pair_16x2) {
  return launch_store<1024, 2, 256>(s, g, b, K, mode, hi_mid, store, st);
}

}  // namespace rfa
